// The top-b end of an event (Algorithm 1's explicit lambda = 0 branch): from the ordered keys of a head's scores in the
// registers of a workgroup of 256 threads to its lists and kept rows.  Used by the kernel that reads the scores and by the
// scorer that computes them.
#pragma once
#include "kvr_dense_common.hpp"

namespace kvr {

constexpr int kTopbThreads = 256;
constexpr int kTopbMaxB = 1024;

struct TopbArgs {
  const char* K; const char* V; const float* s_in;
  int32_t* idx_sorted; int32_t* pick_order; float* pick_gain;
  char* K_out; char* V_out;
  long long stride_head, stride_tok;   // elements (bf16 when K_out / V_out are given)
  int n, b;
  const int32_t* b_h;                  // per-head budgets <= b (output rows stay b apart), or null
};

constexpr int topb_smem_bytes(int slots, int b) { return (16 + 2 * slots * (kTopbThreads / 64) + 4 * b) * 4; }

// key[k]: of token 256 * k + thread, 0 past the head's end.  smem_i: topb_smem_bytes(S, a.b) of LDS, 16-byte aligned.
template <int S>
__device__ __forceinline__ void topb_finish(const TopbArgs& a, int32_t* smem_i, const uint32_t (&key)[S], int h, int tid, int lane, int w) {
  constexpr int NT = kTopbThreads, W = NT / 64;
  int32_t* cnt_l = smem_i;                       // [2][W] counts of a search round
  int32_t* tab_a = smem_i + 16;                  // [S][W] per (slot, wave) counts
  int32_t* tab_b = tab_a + S * W;                // [S][W]
  uint32_t* sel_key = reinterpret_cast<uint32_t*>(tab_b + S * W);   // [b]
  int32_t* sel_tok = reinterpret_cast<int32_t*>(sel_key) + a.b;    // [b] = sort(S)
  int32_t* order_l = sel_tok + a.b;                                 // [b]
  float* gain_l = reinterpret_cast<float*>(order_l + a.b);          // [b]
  const int bs = a.b;                                               // rows of the outputs per head

  const int n = a.n;
  const int b = a.b_h ? min(max(a.b_h[h], 0), bs) : bs;             // the head's own budget
  // ---- 1. tau = the largest key value with at least b keys >= it; or, as soon as some value has exactly b keys at or above it,
  // the one below that value (no key is between the two then, and nothing is equal to tau that counts): half the rounds of
  // the full search on scores without ties
  int par = 0;
  uint32_t tau = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = tau | (1u << bit);
    const int c_w = count_slots_ge<S>(key, cand);
    if (lane == 0) cnt_l[par * W + w] = c_w;
    lds_barrier();
    const int4 c4 = *reinterpret_cast<const int4*>(cnt_l + par * W);
    const int c = __builtin_amdgcn_readfirstlane(c4.x + c4.y + c4.z + c4.w);
    par ^= 1;
    if (c == b) { tau = cand - 1u; break; }
    if (c > b) tau = cand;
  }
  // ---- 2. selected tokens in token order: token order is slot-major, then wave, then lane
  unsigned long long above[S], equal[S];
  masks_ge<S>(key, tau, equal);
  if (tau != 0xffffffffu) masks_ge<S>(key, tau + 1u, above);
#pragma unroll
  for (int k = 0; k < S; ++k) {
    if (tau == 0xffffffffu) above[k] = 0;
    equal[k] &= ~above[k];
    if (lane == 0) { tab_a[k * W + w] = __popcll(above[k]); tab_b[k * W + w] = __popcll(equal[k]); }
  }
  lds_barrier();
  // counts over the (slot, wave) cells before each: a prefix sum in registers, cell c of 64 in lane c (both counts in one
  // word, at most 8192 each), instead of one LDS read after the other
  constexpr int CELLS = S * W, BLK = (CELLS + 63) / 64;
  uint32_t pre[BLK], total = 0;
#pragma unroll
  for (int q = 0; q < BLK; ++q) {
    const int c = q * 64 + lane;
    const uint32_t own = c < CELLS ? static_cast<uint32_t>(tab_a[c]) | (static_cast<uint32_t>(tab_b[c]) << 16) : 0u;
    int v = static_cast<int>(own);
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    pre[q] = static_cast<uint32_t>(v) - own + total;
    total += static_cast<uint32_t>(__builtin_amdgcn_readlane(v, 63));
  }
  const int need_eq = b - static_cast<int>(total & 0xffffu);          // >= 0 by the choice of tau
  // position of this lane's tokens: selected tokens before them
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const uint32_t before = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(pre[k * W / 64]), (k * W) % 64 + w));
    const int eq_rank = static_cast<int>(before >> 16) + __popcll(equal[k] & below);       // this token's rank among the equal ones
    const bool is_above = (above[k] >> lane) & 1ull, is_equal = (equal[k] >> lane) & 1ull;
    if (is_above || (is_equal && eq_rank < need_eq)) {
      const int eq_taken = eq_rank < need_eq ? eq_rank : need_eq;        // equal tokens before it that are selected
      const int p = static_cast<int>(before & 0xffffu) + __popcll(above[k] & below) + eq_taken;
      sel_key[p] = key[k];
      sel_tok[p] = k * NT + tid;
    }
  }
  lds_barrier();
  // ---- 3. rank among the selected: (score descending, index ascending); the list is in index order.  With a budget
  // of up to 64 the four waves share the comparisons of an entry (two shares for up to 128 cost more than they save: 7168 heads,
  // b = 128, 215 us against 207).
  const int parts = b <= 64 ? 4 : 1;
  const int step = NT / parts, part = __builtin_amdgcn_readfirstlane(tid / step);
  if (parts > 1) {
    const int e = tid - part * step;
    int32_t* rank_l = order_l;                     // [b] partial ranks add up here before the lists take its place
    if (tid < b) rank_l[tid] = 0;
    lds_barrier();
    const uint32_t ke = e < b ? sel_key[e] : 0u;
    const int f0 = part * ((b + parts - 1) / parts), f1 = min(b, f0 + (b + parts - 1) / parts);
    int rank = 0;
    for (int f = f0; f < f1; ++f) {
      const uint32_t kf = sel_key[f];
      rank += (kf > ke || (kf == ke && f < e)) ? 1 : 0;
    }
    if (e < b) atomicAdd(&rank_l[e], rank);
    lds_barrier();
    const int r = tid < b ? rank_l[tid] : 0;
    const int tok = tid < b ? sel_tok[tid] : 0;
    const float g = tid < b ? key_to_float(ke) : 0.f;   // (threads below b are the first part: ke is their own entry's)
    lds_barrier();
    if (tid < b) { order_l[r] = tok; gain_l[r] = g; }
  } else {
    for (int e = tid; e < b; e += NT) {
      const uint32_t ke = sel_key[e];
      int rank = 0;
      for (int f = 0; f < b; ++f) {
        const uint32_t kf = sel_key[f];
        rank += (kf > ke || (kf == ke && f < e)) ? 1 : 0;
      }
      order_l[rank] = sel_tok[e];
      gain_l[rank] = key_to_float(ke);
    }
  }
  lds_barrier();
  // ---- 4. outputs
  const long long ob = static_cast<long long>(h) * bs;
  for (int u = tid; u < bs; u += NT) {                              // entries past the head's budget are padding
    a.idx_sorted[ob + u] = u < b ? sel_tok[u] : -1;
    if (a.pick_order) a.pick_order[ob + u] = u < b ? order_l[u] : -1;
    if (a.pick_gain) a.pick_gain[ob + u] = u < b ? gain_l[u] : -INFINITY;
  }
  if ((a.K_out || a.V_out) && b > 0)
    compact_rows<4>(a.K, a.V, a.K_out, a.V_out, h * a.stride_head * 2, a.stride_tok, sel_tok, n, b, ob, tid, NT);
}

}  // namespace kvr
