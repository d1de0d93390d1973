// Greedy selection (paper Sec. 4.1, Algorithm 1) for bf16 heads of 4097 to 8192 tokens with budgets up to 1024,
// followed by the compaction of the kept rows.
//
// Exact greedy with lazily refreshed penalties, in epochs as in select_lazy_kernel (a gain computed from an out-of-date
// running maximum m of Eq. 2 is an upper bound, so a token needs an update only when its bound matters):
//   1. the 128 best fresh unselected tokens form the pool (each wave contributes its best sixteen); the best gain of any
//      token outside it, fresh or stale, is the bound of the epoch;
//   2. the pool's rows are gathered into LDS and their cosine triangle is computed on bf16 MFMA;
//   3. one wave runs Algorithm 1 inside the pool for as long as the pool's best (gain, lower index) beats the bound;
//   4. every wave brings the quarter of its tokens with the highest bounds up to date (the first epoch: every token).
// What differs is where the rows of the picks are: a thousand of them do not fit LDS, so step 4 streams them, 128 at a
// time and shared by all waves, past the 128 rows that every wave holds as operands.  Every token carries the 16-pick tile up to
// which its m covers the picks; a wave's list holds its stale tokens first, the least covered ones in front, and its fresh ones,
// which need the last epoch's picks only, after them, and every 64 entries start at the first block of 64 picks that one of them
// has yet to meet.  (So an entry meets up to 63 picks again, more beside less covered neighbours.  Their cosines are the ones that
// m has seen but for the last bit: the triangle multiplies a sum by the norms of its two tokens in their order, the pass by
// the pick's first.)
//
// Why lazily here too: with all of V read after every epoch 256 heads of 8192 tokens with b = 1024 fetched 13.2 GB and took
// 2770 us, here 4.6 GB in 1620-1700 us (by the memory counters, 24.6 and 8.6 times V's 0.54 GB: the listed rows, the rows of
// the pools and of the picks, which every round streams again, and spilled registers).  A pool of 192 and an eighth of the
// tokens per pass are faster (1300 us), but then the epochs are others than those of a full refresh, other cosines come out of
// the pool's triangle, and among 7840 heads two kept another token; with
// a quarter of the tokens fresh the pools are nearly always those of a full refresh (none did).  Asking for that in
// every epoch, with passes until no stale bound reaches a wave's best seventeen, costs more than it saves (2250 us).
//
// Layout: one workgroup of eight wave64s per head, token j = 1024*w + 64*k + lane in wave w, lane `lane`, slot k; m
// and covered tile of a token stay in its lane's registers, its inverse norm in LDS.
#define KVR_BOUNDS_FILE 4   // ids 4xx of the debug build's bounds checks (kvr_bounds.hpp)
#include "kvr_dense_common.hpp"
#include "kvr_kernels.hpp"
#include <type_traits>

namespace kvr {

constexpr int kLgW = 8;             // waves
constexpr int kLgThreads = 64 * kLgW;
constexpr int kLgPool = 128;        // pool size, a multiple of 64
constexpr int kLgMaxB = 1024;       // largest budget
constexpr int kLgPitch = 272;       // bytes per pool row and per row of a wave's stage (256 + 16)
// 64 picked rows as operands of the 16x16x32 products: 16-byte piece p of row r of a tile sits in plane p & 3 at r * 80 +
// (p >> 2) * 16, the planes 1280 bytes apart.  Lane (row c, k-group kg) reads piece 4 ks + kg in step ks: the sixteen lanes
// of a k-group cover all banks and the four k-groups hit the same ones, which is what a 128-bit LDS read needs to run
// at full rate.  The order over k is the natural one, that of the Gram's 32x32x16 products, whose sums then come out in the same bits.
constexpr int kLgPlaneRow = 80;
constexpr int kLgPlane = 16 * kLgPlaneRow;
constexpr int kLgTile = 4 * kLgPlane;
constexpr int kLgChunk = 128;               // picked rows per chunk
constexpr int kLgTiles = kLgChunk / 16;
constexpr int kLgChunkBytes = kLgTiles * kLgTile;
constexpr int kLgGroup = 128;       // rows of a list that a wave holds as operands at once
constexpr int kLgNone = 255;        // (no group)
constexpr int kLgSelBits = 16;      // leading bits of a gain's ordered key used to choose the pool

struct LargeArgs {
  const char* K; const char* V; const float* s_in;
  int32_t* idx_sorted; int32_t* pick_order; float* pick_gain;
  char* K_out; char* V_out;
  long long stride_head, stride_tok;   // elements
  int n, b;
  float lambda, eps;
  const int32_t* b_h;                  // per-head budgets <= b (output rows stay b apart), or null
};

template <int S> struct LargeCfg {
  static constexpr int TPW = 64 * S;
  static constexpr int CAP = TPW / 2;             // entries of a wave's list (the first epoch's pass takes two lists)
  static constexpr int kStage = 16 * kLgPitch;    // per wave: 16 rows on their way into operands
  static constexpr int kScratch = 1024 + 512;     // per wave: exchange of 64 entries' maxima | 128 squared norms
  static constexpr int kPass = 2 * kLgChunkBytes;
  static_assert(kLgW * kStage <= kPass, "the stages fit the chunks' area");
  static constexpr int kTriBytes = padded_tri_floats(kLgPool) * 4;
  static constexpr int kRowBytes = kLgPool * kLgPitch;
  static constexpr int kCounts = 16 * 64;         // per wave, while its list is built: stale entries by class and lane
  static constexpr int kMax2 = kTriBytes > kRowBytes ? kTriBytes : kRowBytes;
  static constexpr int kUnion = ((kPass > kMax2 ? kPass : kMax2) + 15) & ~15;
  static_assert(kRowBytes + kLgW * kCounts * 4 <= kUnion && kRowBytes % 16 == 0, "the counters of the lists fit above the pool's rows");
  // floats: slots 64 | shared 16 | wcount 16 | first 64 picks needed by every 64 list entries 8*8 |
  //         pool_tok,r,s,m,picked 5*P | inverse norms 64*S*W | lists W*CAP (at the end the sorted indices) |
  //         order, gain, pick_r 3*bcap ; then the waves' scratch and the union area (pool rows -> triangle -> stages -> chunks -> pick flags)
  static constexpr int kTables = 160;
  static constexpr int kFixedFloats = kTables + 5 * kLgPool + TPW * kLgW;
  static constexpr int kListFloats = kLgW * CAP;
  static_assert(kListFloats >= kLgMaxB, "the sorted indices fit the lists");
  static_assert(TPW * kLgW * 4 <= kUnion, "the pick flags of the read-out fit the union area");
  static_assert(kFixedFloats % 4 == 0 && kListFloats % 4 == 0 && kStage % 16 == 0 && kScratch % 16 == 0, "16-byte areas");
  static constexpr int bcap(int b) { return (b + 63) & ~63; }
  static constexpr int smem_bytes(int b) { return (kFixedFloats + kListFloats + 3 * bcap(b)) * 4 + kLgW * kScratch + kUnion; }
};

// BUD: per-head budgets are read from a.b_h.  FAR: a head spans 2 GiB or more (byte offsets of 64 bits).
template <int S, bool BUD, bool FAR>
__global__ __launch_bounds__(kLgThreads, 1) void select_large_kernel(LargeArgs a) {
  using Cfg = LargeCfg<S>;
  constexpr int W = kLgW, P = kLgPool, NT = kLgThreads;
  constexpr int TPW = Cfg::TPW, CAP = Cfg::CAP;
  constexpr int Q = P / W;                         // pool members contributed per wave
  constexpr int KR = TPW / 4;                      // tokens a wave aims to refresh per pass
  constexpr int NB = P / 32, NTRI = NB * (NB + 1) / 2, NTILE = (NTRI + W - 1) / W;
  constexpr int NQ = P / 64;                       // pool slots per lane in the race
  static_assert(P % 64 == 0 && Q <= 64 && KR <= CAP && CAP % kLgGroup == 0, "pool and list sizes");
  extern __shared__ __align__(16) float smem[];
  float* slot_gain = smem;                                       // [2][16]
  int32_t* slot_idx = reinterpret_cast<int32_t*>(smem + 32);     // [2][16]
  int32_t* shared_i = reinterpret_cast<int32_t*>(smem + 64);     // [16] np, t, stop reason
  int32_t* wcount = reinterpret_cast<int32_t*>(smem + 80);       // [16]
  int32_t* gstart = reinterpret_cast<int32_t*>(smem + 96);       // [W][8] first 64 picks (by number / 64) that 64 entries of the wave's list need, kLgNone past the last
  int32_t* pool_tok = reinterpret_cast<int32_t*>(smem + Cfg::kTables);    // [P] token of the member, -1 = none
  float* pool_r = smem + Cfg::kTables + P;
  float* pool_s = smem + Cfg::kTables + 2 * P;
  float* pool_m = smem + Cfg::kTables + 3 * P;
  int32_t* pool_picked = reinterpret_cast<int32_t*>(smem + Cfg::kTables + 4 * P);
  float* r_l = smem + Cfg::kTables + 5 * P;                               // [64 S W] inverse norms by token
  float* lr_all = smem + Cfg::kFixedFloats;                      // [W][CAP] refresh lists / results
  int32_t* idxs_l = reinterpret_cast<int32_t*>(lr_all);          // [b] sorted indices (the lists are dead by then)
  const int bcap = Cfg::bcap(a.b);
  int32_t* order_l = reinterpret_cast<int32_t*>(lr_all + Cfg::kListFloats);
  float* gain_l = lr_all + Cfg::kListFloats + bcap;
  float* pick_r = lr_all + Cfg::kListFloats + 2 * bcap;          // inverse norms of the picks, 0 past the last
  char* wave_scratch = reinterpret_cast<char*>(lr_all + Cfg::kListFloats + 3 * bcap);
  char* uni = wave_scratch + W * Cfg::kScratch;
  char* prow = uni;                                              // [P][272 B] pool rows (gather, Gram) ...
  float* tri = reinterpret_cast<float*>(uni);                    // ... then the padded P x P cosine triangle (race) ...
  char* chunk = uni;                                             // ... then the waves' stages, then two chunks of picked rows (pass) ...
  int32_t* flag = reinterpret_cast<int32_t*>(uni);               // ... and at the end [n padded] pick flags

  const int h = blockIdx.x;
  int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // What the phases compute from the lane number is computed where it is used: hoisted out of the epochs, as the compiler
  // would, it takes a hundred registers and comes back from scratch memory, whose loads wait for every row in flight.
  auto fresh_lane = [&]() { asm volatile("" : "+v"(lane), "+v"(tid)); };
  const int n = a.n;
  const int b = BUD ? min(max(a.b_h[blockIdx.x], 0), a.b) : a.b;      // a scalar load: the index is uniform
  const long long head_off = h * a.stride_head * 2;             // bytes
  const char* Vh = a.V + head_off;
  using Off = std::conditional_t<FAR, unsigned long long, uint32_t>;
  const Off pitch_b = static_cast<Off>(a.stride_tok) * 2u;      // bytes between tokens
  const int base = w * TPW;
  char* stage = uni + w * Cfg::kStage;
  float* scratch = reinterpret_cast<float*>(wave_scratch + w * Cfg::kScratch);   // [256] exchange of 64 entries' maxima
  float* norm_x = scratch + 256;                                 // [128] squared norms of the group's rows
  float* lrw = lr_all + w * CAP;                          // tokens to refresh, then their raw maxima
  int32_t* lrw_i = reinterpret_cast<int32_t*>(lrw);

  // Kept in registers: m, two packed tables and bit masks.  The scores are read from memory again in every epoch (they are
  // needed for the choice of the pool and the list only).  All 256 registers are in use all the same, and 22 to 24 of them spill: 176
  // bytes of scratch per lane, some 0.86 of the 1.0 GB that 256 heads of 8192 tokens write.
  float s[S], m[S];
  uint32_t dead = 0;             // bit k: token past the head, below the score bound or picked (its score counts as -inf)
  uint32_t place[S / 2];         // 16 bits each: 0 = none, 1 + pool slot of this token in the current epoch, or 0x8000 + position in the wave's refresh list
  uint32_t cov[S / 4];           // bytes: 16-pick tile from which m[k] has yet to meet the picks (those before are covered)
  uint32_t fresh = 0xffffffffu;  // bit k: m[k] covers every pick made so far
  auto tok_of = [&](int k) -> int { return base + 64 * k + lane; };
  auto get_place = [&](int k) -> uint32_t { return (place[k >> 1] >> (16 * (k & 1))) & 0xffffu; };
  auto set_place = [&](int k, uint32_t v) { place[k >> 1] = (place[k >> 1] & (0xffffu << (16 * (1 - (k & 1))))) | (v << (16 * (k & 1))); };
  const float* const sh = a.s_in + static_cast<long long>(h) * n;
  auto load_scores = [&]() {
#pragma unroll
    for (int k = 0; k < S; ++k) s[k] = sh[min(tok_of(k), n - 1)];
  };
  auto mask_scores = [&]() {
#pragma unroll
    for (int k = 0; k < S; ++k) s[k] = ((dead >> k) & 1u) ? -INFINITY : s[k];
  };
#pragma unroll
  for (int k = 0; k < S; ++k) {
    if (tok_of(k) >= n) dead |= 1u << k;
    m[k] = 0.f;
    r_l[base + 64 * k + lane] = 0.f;
  }
#pragma unroll
  for (int k = 0; k < S / 2; ++k) place[k] = 0u;
#pragma unroll
  for (int k = 0; k < S / 4; ++k) cov[k] = 0u;
  load_scores();
  mask_scores();
  for (int u = tid; u < bcap; u += NT) pick_r[u] = 0.f;
  const float nlam = -a.lambda;
  int par = 0;
  int t = 0;
  int kbits = kLgSelBits;        // leading key bits the pool choice looks at (uniform)
  uint32_t tau_prev = 0;         // the wave's pool threshold of the last epoch (0: none)
  bool starved = false;
  float delta = -1.f;            // refresh threshold: this far below the wave's best outside gain (< 0: not yet known)

  // workgroup argmax over av (per slot); ibest carries bit 30 when the winner's slot has a stale m
  auto wg_argmax = [&](const float (&av)[S], float& gbest, int& ibest, float& amax_w) {
    float best = av[0];
#pragma unroll
    for (int k = 1; k < S; ++k) best = hw_max(best, av[k]);
    amax_w = wave_max_uniform(best);
    int i_w = -1;
#pragma unroll
    for (int k = S - 1; k >= 0; --k) {
      const unsigned long long eq = __ballot(av[k] == amax_w);
      if (eq) {
        const int l0 = __ffsll(static_cast<long long>(eq)) - 1;
        const int fr = (__builtin_amdgcn_readlane(static_cast<int>(fresh), l0) >> k) & 1;
        i_w = (base + 64 * k + l0) | (fr ? 0 : (1 << 30));
      }
    }
    if (lane == 0) { slot_gain[par * 16 + w] = amax_w; slot_idx[par * 16 + w] = i_w; }
    lds_barrier();
    const float g = lane < W ? slot_gain[par * 16 + lane] : -INFINITY;
    const int ii = lane < W ? slot_idx[par * 16 + lane] : -1;
    par ^= 1;
    gbest = wave_max_uniform(g);
    const unsigned long long eqw = __ballot(lane < W && g == gbest);
    ibest = eqw ? __builtin_amdgcn_readlane(ii, __ffsll(static_cast<long long>(eqw)) - 1) : -1;
  };

  if (b == 1) {
    float gmax, dummy; int i;
    wg_argmax(s, gmax, i, dummy);
    if (!(gmax > -INFINITY)) starved = true;
    else { if (tid == 0) { order_l[0] = i & 0x3fffffff; gain_l[0] = gmax; } t = 1; }
  } else {
    bool have_r = false;
    // Exact candidate reduction: a token with s_j < s_(b) - lambda never wins Eq. 3 (while fewer than b tokens are
    // selected one of the b best-scored is free and gains at least s_(b) - lambda, and a token gains at most its
    // score).  Such tokens get the score -inf: never a pool member, a pick or in a list, and their rows are never
    // read.  Nothing can go when the finite scores spread by less than lambda; one min/max settles that first.
    {
      float hi = -INFINITY, lo = INFINITY;
#pragma unroll
      for (int k = 0; k < S; ++k) {
        if (s[k] > -INFINITY && s[k] < INFINITY) { hi = hw_max(hi, s[k]); lo = fminf(lo, s[k]); }
      }
      hi = wave_max_uniform(hi);
      lo = -wave_max_uniform(-lo);
      if (lane == 0) { slot_gain[par * 16 + w] = hi; slot_gain[32 + w] = lo; }   // (smem 32.. is slot_idx: free until the first argmax)
      lds_barrier();
      float ghi = -INFINITY, glo = INFINITY;
#pragma unroll
      for (int u = 0; u < W; ++u) { ghi = hw_max(ghi, slot_gain[par * 16 + u]); glo = fminf(glo, slot_gain[32 + u]); }
      par ^= 1;
      const bool wide = __builtin_amdgcn_readfirstlane(ghi - glo > a.lambda ? 1 : 0) != 0;   // false also when no score is finite
      lds_barrier();                                 // the min/max slots are rewritten below
      if (wide) {
        uint32_t key[S];
#pragma unroll
        for (int k = 0; k < S; ++k) key[k] = tok_of(k) < n ? ordered_key(s[k] + 0.0f) : 0u;
        uint32_t T = 0;                              // s_(b) from the leading 16 bits: at most s_(b), the bound only loosens
        for (int bit = 31; bit >= 16; --bit) {
          const uint32_t cand = T | (1u << bit);
          int c = 0;
#pragma unroll
          for (int k = 0; k < S; ++k) c += __popcll(__ballot(key[k] >= cand));
          if (lane == 0) slot_idx[par * 16 + w] = c;
          lds_barrier();
          int tot = 0;
#pragma unroll
          for (int u = 0; u < W; ++u) tot += slot_idx[par * 16 + u];
          par ^= 1;
          if (tot >= b) T = cand;
        }
        const float sb = key_to_float(T);
        const float thr = sb - a.lambda * 1.00001f - 1e-5f * fabsf(sb);   // fp32 cosines may exceed 1 by a few ulp
#pragma unroll
        for (int k = 0; k < S; ++k)
          if (s[k] < thr) { s[k] = -INFINITY; dead |= 1u << k; }   // (a NaN threshold or score leaves the token in)
      }
    }
    // sum of squares of a row whose 16-byte pieces sit in the 16 lanes of a DPP row; every lane gets it
    auto sum_sq = [](const uint4& x) -> float {
      const float e[8] = {bf16_lo(x.x), bf16_hi(x.x), bf16_lo(x.y), bf16_hi(x.y),
                          bf16_lo(x.z), bf16_hi(x.z), bf16_lo(x.w), bf16_hi(x.w)};
      float ss = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) ss = fmaf(e[q], e[q], ss);
      KVR_DPP_ADD(ss, 0x128, 0xf) KVR_DPP_ADD(ss, 0x124, 0xf) KVR_DPP_ADD(ss, 0x122, 0xf) KVR_DPP_ADD(ss, 0x121, 0xf)
      return ss;
    };

    int idle = 0;                                    // epochs in a row without a pick
    while (t < b) {
      fresh_lane();
      // ================= 1. pool = the best Q fresh unselected tokens of every wave =================
      // Keys are cut to their leading kbits bits: the pool only has to be a good guess (the race against the outside
      // bound keeps the picks exact).  When the cut keys cannot tell a wave's best tokens apart the best one may be
      // left outside and the epoch ends without a pick; it is then repeated on the full keys.
      float go[S];                                   // gains; then the bounds of the tokens left outside
      uint32_t ekey[S];                              // key + 1 of a fresh token, 0 of a stale one (never a member)
#pragma unroll
      for (int k = 0; k < S; ++k) {
        go[k] = fmaf(nlam, m[k], s[k]);
        const uint32_t k1 = (ordered_key(go[k]) >> (32 - kbits)) + 1u;   // (wraps to 0 for an all-ones key, which only a NaN with full keys has)
        ekey[k] = ((fresh >> k) & 1u) ? k1 : 0u;
      }
      uint32_t tau = 0;                              // largest value with at least Q fresh keys >= it
      auto at_least_q = [&](uint32_t x) -> bool {
        int c = 0;
#pragma unroll
        for (int k = 0; k < S; ++k) c += __popcll(__ballot(ekey[k] >= x));
        return c >= Q;
      };
      if (kbits == kLgSelBits && tau_prev != 0) {
        // bracketed from the last epoch's value with doubling steps, then bisected
        constexpr uint32_t kTop = (1u << kLgSelBits) + 1u;   // no key + 1 reaches this
        uint32_t lo, hi;                             // at_least_q(lo), !at_least_q(hi)
        if (at_least_q(tau_prev)) {
          lo = tau_prev;
          for (uint32_t d = 1;; d <<= 1) {
            hi = lo + d;
            if (hi >= kTop) { hi = kTop; break; }
            if (!at_least_q(hi)) break;
            lo = hi;
          }
        } else {
          hi = tau_prev;
          for (uint32_t d = 1;; d <<= 1) {
            lo = hi > d ? hi - d : 0u;               // (every key is >= 0)
            if (lo == 0u || at_least_q(lo)) break;
            hi = lo;
          }
        }
        while (hi - lo > 1u) {
          const uint32_t mid = (lo + hi) >> 1;
          if (at_least_q(mid)) lo = mid; else hi = mid;
        }
        tau = lo;
      } else {
        for (int bit = kbits; bit >= 0; --bit) {
          if (bit == 32) continue;                   // keys + 1 of full-width keys are searched over 32 bits
          const uint32_t cand = tau | (1u << bit);
          if (at_least_q(cand)) tau = cand;
        }
      }
      tau_prev = tau;
      if (tau == 0) tau = 1;                         // fewer than Q fresh tokens: all of them join
      int taken = 0;                                 // members with key > tau come first, ties in token order
#pragma unroll
      for (int k = 0; k < S; ++k) taken += __popcll(__ballot(ekey[k] > tau));
      int need_eq = Q - taken;                       // how many of the key == tau tokens join
      int rank_base = 0;
#pragma unroll
      for (int k = 0; k < S; ++k) {
        const bool above = ekey[k] > tau, equal = ekey[k] == tau;
        const unsigned long long eqm = __ballot(equal);
        const int eq_before = __popcll(eqm & ((1ull << lane) - 1ull));
        const bool in = above || (equal && eq_before < need_eq);
        const unsigned long long inm = __ballot(in);
        const int slot = w * Q + kvr_ix_if(in, rank_base + __popcll(inm & ((1ull << lane) - 1ull)), Q, 401);   // 401: a member's place in the wave's share
        set_place(k, in ? static_cast<uint32_t>(slot + 1) : 0u);
        if (in) {
          pool_tok[slot] = tok_of(k) < n ? tok_of(k) : -1;
          pool_s[slot] = s[k];
          pool_m[slot] = m[k];
        }
        if (in) go[k] = -INFINITY;
        rank_base += __popcll(inm);
        const int eq_in = __popcll(eqm);
        need_eq -= eq_in < need_eq ? eq_in : need_eq;
      }
      if (lane >= rank_base && lane < Q) {           // fewer fresh tokens than the wave's share: empty slots
        const int slot = w * Q + lane;
        pool_tok[slot] = -1; pool_s[slot] = -INFINITY; pool_m[slot] = 0.f;
      }
      float gout, gmax_w; int jout_f;
      wg_argmax(go, gout, jout_f, gmax_w);           // barrier inside: the pool tables are complete
      const int jout = jout_f < 0 ? -1 : (jout_f & 0x3fffffff);
      const bool jout_stale = jout_f >= 0 && (jout_f & (1 << 30));

      fresh_lane();
      // the pool's rows are requested now; the refresh list is built while they are on their way
      constexpr int kGat = P * 16 / NT;              // rows per thread
      constexpr int kGatRows = NT / 16;              // rows per round
      const int gat_row = tid >> 4, gat_piece = tid & 15;
      uint4 x[kGat];
#pragma unroll
      for (int k = 0; k < kGat; ++k) {
        const int tk = pool_tok[k * kGatRows + gat_row];
        const int tkc = kvr_ix(tk < 0 ? 0 : tk, n, 403);   // an empty slot reads row 0 and stores zeros (403: token of a pool member)
        x[k] = *reinterpret_cast<const uint4*>(Vh + (static_cast<Off>(tkc) * pitch_b + gat_piece * 16u));
      }
      if (tid < P) {
        const int tk = pool_tok[tid];
        if (have_r) pool_r[tid] = tk < 0 ? 0.f : r_l[kvr_ix(tk, TPW * W, 405)];   // (in the first epoch the gather finds it; 405: token of a pool member)
        pool_picked[tid] = 0;
      }
      // ---- the wave's refresh list for this epoch's pass: outside tokens whose bound lies within delta of the wave's
      // best one.  delta is steered so that about KR tokens qualify: a few bisection steps around the previous
      // epoch's value.  In the first epoch every outside token that can still be picked is refreshed, in two lists.
      const int t0 = t;                              // picks that fresh tokens cover
      int cnt_r = 0;                                 // entries of the list
      bool split = false;                            // the list takes two turns: the wave's lower slots, then the others
      float thr_r = -INFINITY;
      // Stale entries come first, ordered by the 64 picks from which they have yet to meet the picks (their class), those of a
      // class by lane and slot, then the fresh ones in token order.  The order decides which entries share a start, so it must not
      // depend on the order in which the hardware serves lanes: every lane counts its entries of a class in a counter of its own, and
      // a prefix sum over (class, lane) gives each counter its first position.
      auto build_list = [&](auto member) {
        fresh_lane();
        int wu = w;
        asm volatile("" : "+s"(wu));                 // (likewise: no addresses kept over the epochs)
        int32_t* const counts = reinterpret_cast<int32_t*>(uni + Cfg::kRowBytes) + wu * Cfg::kCounts;   // [16][64], above the pool's rows, which other waves may be storing
        int32_t* const mine = counts + lane;
        auto class_of = [&](int k) -> int { return static_cast<int>((cov[k >> 2] >> (8 * (k & 3) + 2)) & 0xfu); };
        int4* const share = reinterpret_cast<int4*>(counts + lane * 16);   // sixteen counters of a class, four lanes a class
#pragma unroll
        for (int u = 0; u < 4; ++u) share[u] = make_int4(0, 0, 0, 0);
        wave_lds_sync();
        int place_in[S];
#pragma unroll
        for (int k = 0; k < S; ++k) {
          place_in[k] = 0;
          if (member(k) && !((fresh >> k) & 1u)) place_in[k] = atomicAdd(&mine[64 * class_of(k)], 1);
        }
        wave_lds_sync();
        int incl;
        {
          int4 c[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) c[u] = share[u];
          int own = 0;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int x = c[u].x, y = c[u].y, z = c[u].z, q = c[u].w;
            c[u] = make_int4(own, own + x, own + x + y, own + x + y + z);
            own += x + y + z + q;
          }
          incl = own;                                // inclusive prefix sums over the lanes' shares
          incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, false);
          incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, false);
          incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, false);
          incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, false);
          incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);
          incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xc, 0xf, false);
          const int at = incl - own;
#pragma unroll
          for (int u = 0; u < 4; ++u) share[u] = make_int4(c[u].x + at, c[u].y + at, c[u].z + at, c[u].w + at);
        }
        int off = __builtin_amdgcn_readlane(incl, 63);
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < S; ++k)                  // (all the reads before the first write)
          place_in[k] += mine[64 * class_of(k)];
#pragma unroll
        for (int k = 0; k < S; ++k) {
          const bool mem = member(k), fr = (fresh >> k) & 1u;
          const unsigned long long mm = __ballot(mem && fr);
          if (mem) {
            const int pos = kvr_ix(fr ? off + __popcll(mm & ((1ull << lane) - 1ull)) : place_in[k], CAP, 402);   // 402: position in the refresh list
            lrw_i[pos] = tok_of(k);
            set_place(k, 0x8000u + static_cast<uint32_t>(pos));
          }
          off += __popcll(mm);
        }
        cnt_r = off;
        int first = kLgNone;                         // lane g: of entry 64 g
#pragma unroll
        for (int g = 0; g < CAP / 64; ++g) {
          const int c = __popcll(__ballot((lane & 3) == 3 && incl <= 64 * g));
          const int f = g * 64 < cnt_r ? (c < 16 ? min(c, t0 >> 6) : t0 >> 6) : kLgNone;
          first = lane == g ? f : first;
        }
        if (lane < 8) gstart[w * 8 + lane] = first;
        // pad to whole groups with a valid row (its results are never read)
        const int padded = max((cnt_r + kLgGroup - 1) & ~(kLgGroup - 1), kLgGroup);
        for (int u = cnt_r + lane; u < padded; u += 64) lrw_i[u] = min(base, n - 1);
      };
      // A group's rows: as they come from memory (sub-block, row (lane >> 4) + 4 q of it), then as operands.
      uint4 rows[8][4];
      auto fetch = [&](int gi, int sub) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = kvr_ix(lrw_i[gi * kLgGroup + sub * 16 + (lane >> 4) + 4 * q], n, 404);   // 404: token of a list entry
          rows[sub][q] = *reinterpret_cast<const uint4*>(Vh + (static_cast<Off>(row) * pitch_b + (lane & 15) * 16u));
        }
      };
      if (have_r && gmax_w > -INFINITY) {
        auto count_ge = [&](float thr) -> int {
          int c = 0;
#pragma unroll
          for (int k = 0; k < S; ++k) c += __popcll(__ballot(go[k] >= thr && go[k] > -INFINITY));
          return c;
        };
        float lo_d, hi_d;
        int steps;
        if (delta < 0.f) {
          float gmin = INFINITY;
#pragma unroll
          for (int k = 0; k < S; ++k) if (go[k] > -INFINITY) gmin = fminf(gmin, go[k]);
          gmin = -wave_max_uniform(-gmin);
          lo_d = 0.f; hi_d = gmax_w - gmin; steps = 8;
        } else {
          lo_d = 0.5f * delta; hi_d = 2.0f * delta; steps = 3;
        }
        int c_lo = 1;                                // tokens within lo_d of the best (not counted for the first guess)
        bool above = false;                          // some count exceeded KR: more than KR tokens lie within hi_d
        for (int it = 0; it < steps; ++it) {         // count(delta) grows with delta
          const float mid = 0.5f * (lo_d + hi_d);
          const int c = count_ge(gmax_w - mid);
          if (c > KR) { hi_d = mid; above = true; } else { lo_d = mid; c_lo = c; }
        }
        // the lower end of the bracket: at most KR tokens, always including the wave's best outside token
        delta = lo_d;
        thr_r = gmax_w - delta;
        if (4 * c_lo < KR) {
          // The guess has collapsed or run away: a full search next time.  When the bracket could not split a crowd of
          // bounds and the last epoch ended without a pick, the whole crowd is refreshed, or the epochs would crawl
          // through it a few tokens at a time.
          if (above && idle > 0) thr_r = gmax_w - hi_d;
          delta = -1.f;
        }
        // A token with a score of +inf is outside, and distances from an infinite bound say nothing (inf - inf is a NaN, which
        // would list no token: none of them fresh again, none ever picked).  The list takes exactly these tokens.
        if (gmax_w == INFINITY) { thr_r = 3.402823466e38f; delta = -1.f; }
        split = count_ge(thr_r) > CAP;
      }
      if (!have_r) split = true;
      build_list([&](int k) { return go[k] >= thr_r && go[k] > -INFINITY && (!split || k < S / 2); });
      wave_lds_sync();                               // the list was written by other lanes of this wave
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) fetch(0, sub);   // (they travel while the pool's triangle is computed and raced ...

      fresh_lane();
      // ================= 2. pool rows -> LDS, cosine triangle on MFMA (written over the rows) =================
#pragma unroll
      for (int k = 0; k < kGat; ++k) {
        const int slot = k * kGatRows + gat_row;
        if (pool_tok[slot] < 0) x[k] = make_uint4(0u, 0u, 0u, 0u);   // (only here: a select between the loads would make each wait for the one before)
        *reinterpret_cast<uint4*>(prow + slot * kLgPitch + gat_piece * 16) = x[k];
      }
      if (!have_r) {
#pragma unroll
        for (int k = 0; k < kGat; ++k) {
          const int slot = k * kGatRows + gat_row;
          const float ss = sum_sq(x[k]);
          if (gat_piece == 0) {
            const float r = 1.0f / (sqrtf(ss) + a.eps);
            pool_r[slot] = pool_tok[slot] < 0 ? 0.f : r;
            if (pool_tok[slot] >= 0) r_l[pool_tok[slot]] = r;
          }
        }
      }
      lds_barrier();
      {
        const int hf = lane >> 5;
        f32x16 acc[NTILE];
#pragma unroll
        for (int q = 0; q < NTILE; ++q) {
          const int tile = w + q * W;                  // lower-triangular 32x32 tiles of the P x P matrix
          acc[q] = f32x16{0};
          if (tile < NTRI) {
            int I = 0;
            while ((I + 1) * (I + 2) / 2 <= tile) ++I;
            const int J = tile - I * (I + 1) / 2;
            const char* pa = prow + (I * 32 + (lane & 31)) * kLgPitch + hf * 16;
            const char* pb = prow + (J * 32 + (lane & 31)) * kLgPitch + hf * 16;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
              acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(pb + ks * 32),
                                                               *reinterpret_cast<const bf16x8*>(pa + ks * 32), acc[q], 0, 0, 0);
          }
        }
        lds_barrier();                                 // every wave has read its rows: the triangle takes their place
#pragma unroll
        for (int q = 0; q < NTILE; ++q) {
          const int tile = w + q * W;
          if (tile < NTRI) {
            int I = 0;
            while ((I + 1) * (I + 2) / 2 <= tile) ++I;
            const int J = tile - I * (I + 1) / 2;
            write_cos_tile_padded(tri, pool_r, acc[q], I, J, lane);   // the diagonal holds +inf: the row of a pick retires it
          }
        }
      }
      lds_barrier();
      fresh_lane();
#pragma unroll
      for (int sub = 4; sub < 8; ++sub) fetch(0, sub);   // ... the second half while it is raced: beside the Gram's accumulators there is no room)
      // ================= 3. Algorithm 1 inside the pool, against the outside bound =================
      if (w == 0) {
        // Pool slots lane, lane + 64, .. live in lane `lane` (slots are in token order, so the lowest slot is the lowest
        // token).  A pick is parked in lane np of two registers, at most 64 picks a turn.
        const int tri0 = static_cast<int>(reinterpret_cast<uintptr_t>(
            (__attribute__((address_space(3))) const char*)reinterpret_cast<const char*>(tri)));
        float sq[NQ], mq[NQ];
        int tja[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int p = lane + 64 * q;
          sq[q] = pool_s[p];
          mq[q] = pool_m[p];
          tja[q] = padded_row_start(p) * 4 + tri0;         // start of the slot's row
        }
        const int jb = __builtin_amdgcn_readfirstlane(jout < 0 ? 0x7fffffff : jout);
        const float gout_u = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(gout)));
        const bool no_out = __builtin_amdgcn_readfirstlane(jout) < 0;
        const int room = __builtin_amdgcn_readfirstlane(min(b - t, P));
        int done = 0, stop = 0;                      // stop: 1 = bound wins, 2 = nothing finite left
        while (done < room && stop == 0) {
          const int turn = __builtin_amdgcn_readfirstlane(min(room - done, 64));
          int np = 0;
          int rec_i = 0, rec_g = 0;
          int until = turn;
          float bound = gout_u;
          while (np < turn) {
            float amax; int i4;
            np = race_loop<NQ, true>(mq, sq, tja, lane, nlam, np, until, bound, rec_i, rec_g, amax, i4, tri0, Cfg::kTriBytes / 4);
            if (np == until) { until = turn; bound = gout_u; continue; }
            // rare: the bound wins, a tie with it, or nothing finite
            if (!(amax > -INFINITY)) { stop = no_out ? 2 : 1; break; }
            if (!(amax == gout_u && __builtin_amdgcn_readfirstlane(pool_tok[i4 >> 2]) < jb)) { stop = 1; break; }
            until = np + 1;                          // a tie that the pool's lower token wins: this one pick passes
            bound = -INFINITY;
          }
          rec_i >>= 2;
          if (lane < np) {
            const int ri = kvr_ix(rec_i, P, 406);                 // 406: pool slot of a pick
            const int tp = kvr_ix(t + done + lane, bcap, 407);    // 407: number of a pick
            order_l[tp] = pool_tok[ri]; gain_l[tp] = __int_as_float(rec_g);
            pick_r[tp] = pool_r[ri]; pool_picked[ri] = 1;
          }
          done += np;
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) pool_m[lane + 64 * q] = mq[q];   // the pool's m is authoritative
        t += done;
        if (lane == 0) { shared_i[0] = done; shared_i[1] = t; shared_i[2] = stop; }
      }
      lds_barrier();
      const int np = shared_i[0];
      t = shared_i[1];
      const int stop = shared_i[2];
      fresh_lane();
      // pool members: m from the race (it covers every pick so far), picked members leave
#pragma unroll
      for (int k = 0; k < S; ++k) {
        const uint32_t pl = get_place(k);
        if (pl != 0u && pl < 0x8000u) {
          m[k] = pool_m[pl - 1];
          if (pool_picked[pl - 1]) dead |= 1u << k;
        }
      }
      if (t >= b) break;
      if (stop == 2 || (np == 0 && !(gout > -INFINITY))) { starved = true; break; }
      if (np == 0) {
        // The bound won at once.  A stale token carried it: its wave lists it or, in a crowd, other stale tokens, which
        // are fresh from then on, so the fresh set grows with every such epoch (at most n of them in a row).  A fresh
        // one: the cut keys left it outside the pool, full keys from here on; under full keys every wave's best
        // fresh tokens are members, so a fresh token can only block on non-finite gains, and then nothing would ever change.
        if (!jout_stale) {
          if (kbits == 32) { starved = true; break; }
          kbits = 32;
        }
        if (++idle > n + 8) { starved = true; break; }   // (never reached without a NaN, by the count above)
      } else {
        idle = 0;
      }
      lds_barrier();                               // everyone is done with the triangle and the pool tables
      fresh_lane();
      // ================= 4. the wave's refresh list against the picks its tokens do not cover =================
      const int kg = lane >> 4;
      const int tiles = kvr_ix((t + 15) >> 4, kLgMaxB / 16 + 1, 410);   // 16-row operands of picked rows (410)
      const int nchunks = (tiles + kLgTiles - 1) / kLgTiles;
      uint32_t now = 0;                              // bit k: this epoch brought m[k] up to date
      for (int turn = 0;; ++turn) {
        // rounds: group g of every wave's list at once; a round starts at the first picks that any wave's group needs
        const int gs_own = gstart[w * 8 + (lane & 7)];
        int gs = gstart[lane];                       // (eight waves of eight entries)
        gs = min(gs, __shfl_xor(gs, 8));
        gs = min(gs, __shfl_xor(gs, 16));
        gs = min(gs, __shfl_xor(gs, 32));
        const int rounds = (__popcll(__ballot(lane < 8 && gs != kLgNone)) + 1) >> 1;
        auto start_of = [&](int g) -> int { return __builtin_amdgcn_readlane(gs, 2 * g) >> 1; };   // first chunk (they ascend with the group)
        uint4 cx[4];                                 // this thread's share of the next chunk
        auto load_chunk = [&](int c) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int tk = kvr_ix(order_l[min(c * kLgChunk + q * (NT / 16) + (tid >> 4), t - 1)], n, 411);   // 411: token of a pick
            cx[q] = *reinterpret_cast<const uint4*>(Vh + (static_cast<Off>(tk) * pitch_b + (tid & 15) * 16u));
          }
        };
        int buf = 0;
        if (rounds > 0 && start_of(0) < nchunks) load_chunk(start_of(0));
        for (int g = 0; g < rounds; ++g) {
          const int c0 = start_of(g);                // (the same in every wave)
          const int q0 = __builtin_amdgcn_readlane(gs_own, 2 * g), q1 = __builtin_amdgcn_readlane(gs_own, 2 * g + 1);
          float part[8];                             // per 16-row sub-block: max over my four picks of every operand
#pragma unroll
          for (int sub = 0; sub < 8; ++sub) {
            part[sub] = 0.f;                         // the floor of Eq. 2
            if ((sub < 4 ? q0 : q1) != kLgNone) {
              wave_lds_sync();
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const uint4 y = rows[sub][q];
                *reinterpret_cast<uint4*>(stage + ((lane >> 4) + 4 * q) * kLgPitch + (lane & 15) * 16) = y;
                if (!have_r) {                       // row (lane >> 4) + 4q of the sub-block is list entry 16*sub + row of the group
                  const float ss = sum_sq(y);
                  if ((lane & 15) == 0) norm_x[sub * 16 + (lane >> 4) + 4 * q] = ss;
                }
              }
              wave_lds_sync();
              const char* fp = stage + (lane & 15) * kLgPitch + kg * 16;
#pragma unroll
              for (int ks = 0; ks < 4; ++ks) rows[sub][ks] = *reinterpret_cast<const uint4*>(fp + ks * 64);
            }
          }
          lds_barrier();                             // the chunks take the stages' place
          for (int c = c0; c < nchunks; ++c) {
            char* cb = chunk + buf * kLgChunkBytes;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int r = q * (NT / 16) + (tid >> 4), pc = tid & 15;
              const uint4 z = make_uint4(0u, 0u, 0u, 0u);       // rows past the last pick are zeros
              *reinterpret_cast<uint4*>(cb + (r >> 4) * kLgTile + (pc & 3) * kLgPlane + (r & 15) * kLgPlaneRow + (pc >> 2) * 16) =
                  c * kLgChunk + r < t ? cx[q] : z;
            }
            const int cn = c + 1 < nchunks ? c + 1 : (g + 1 < rounds ? start_of(g + 1) : nchunks);
            if (cn < nchunks) load_chunk(cn);
            lds_barrier();                           // (the buffer written next was last read before the previous barrier)
            auto tile_products = [&](auto quads_c, int tl0, int tl1) {
              constexpr int quads = decltype(quads_c)::value;
              const char* ap = cb + (tl0 - c * kLgTiles) * kLgTile + kg * kLgPlane + (lane & 15) * kLgPlaneRow;
              const float* pr = pick_r + tl0 * 16 + 4 * kg;
#pragma unroll 1
              for (int tl = tl0; tl < tl1; ++tl, ap += kLgTile, pr += 16) {
                bf16x8 av[4];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) av[ks] = *reinterpret_cast<const bf16x8*>(ap + ks * 16);
                const float4 p0 = *reinterpret_cast<const float4*>(pr);
                f32x4 acc[4 * quads];
#pragma unroll
                for (int v = 0; v < quads; ++v) {
#pragma unroll
                  for (int u = 0; u < 4; ++u) acc[4 * v + u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                      acc[4 * v + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[ks], __builtin_bit_cast(bf16x8, rows[4 * v + u][ks]), acc[4 * v + u], 0, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < 4 * quads; ++u)
                  part[u] = max3(max3(part[u], acc[u][0] * p0.x, acc[u][1] * p0.y), acc[u][2] * p0.z, acc[u][3] * p0.w);
              }
            };
            // the first 64 entries' tiles of this chunk before the others join, then the tiles that all of them meet
            const int tE = min((c + 1) * kLgTiles, tiles);
            const int tA = max(c * kLgTiles, 4 * q0), tB = max(c * kLgTiles, 4 * q1);
            tile_products(std::integral_constant<int, 1>{}, tA, min(tB, tE));
            tile_products(std::integral_constant<int, 2>{}, tB, tE);
            buf ^= 1;
          }
          // lane (col, kg) holds partial maxima of row col of sub-block 0..3; list entry 16*sub + col of the 64 is
          // finished by lane (col, kg = sub).  Exchange through the wave's scratch: [sub][kg][col].
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            if ((v ? q1 : q0) != kLgNone) {
              wave_lds_sync();
#pragma unroll
              for (int sub = 0; sub < 4; ++sub) scratch[sub * 64 + kg * 16 + (lane & 15)] = part[4 * v + sub];
              wave_lds_sync();
              const float* sp = scratch + kg * 64 + (lane & 15);
              const float mx = hw_max(hw_max(sp[0], sp[16]), hw_max(sp[32], sp[48]));
              const int e = g * kLgGroup + v * 64 + lane;
              if (!have_r && e < cnt_r) r_l[kvr_ix(lrw_i[e], TPW * W, 412)] = 1.0f / (sqrtf(norm_x[v * 64 + lane]) + a.eps);   // 412: token of a list entry
              lrw[e] = mx;                           // (the list entries of this group have been consumed)
            }
          }
          if (g + 1 < rounds) lds_barrier();         // the stages take the chunks' place
          if (g + 1 < rounds && (g + 1) * kLgGroup < cnt_r) {
#pragma unroll
            for (int sub = 0; sub < 8; ++sub) fetch(g + 1, sub);
          }
        }
        fresh_lane();
        load_scores();                               // (for the second list, or the next epoch)
        wave_lds_sync();
        // refreshed tokens take their new m
#pragma unroll
        for (int k = 0; k < S; ++k) {
          const uint32_t pl = get_place(k);
          if (pl >= 0x8000u) {
            const int pos = kvr_ix(static_cast<int>(pl - 0x8000u), CAP, 413);   // 413: list position of a refreshed token
            m[k] = hw_max(m[k], lrw[pos] * r_l[tok_of(k)]);
          }
          if (pl != 0u) {                            // pool members left the race up to date
            now |= 1u << k;
            cov[k >> 2] = (cov[k >> 2] & ~(0xffu << (8 * (k & 3)))) | (static_cast<uint32_t>(t >> 4) << (8 * (k & 3)));
          }
        }
#pragma unroll
        for (int k = 0; k < S / 2; ++k) place[k] = 0u;
        mask_scores();
        if (turn == 1) break;
        if (tid == 0) shared_i[4 + par] = 0;
        lds_barrier();                               // the lists' tables are read
        if (split && lane == 0) shared_i[4 + par] = 1;
        cnt_r = 0;
        if (split) {
          build_list([&](int k) {
            const float gk = fmaf(nlam, m[k], s[k]);
            return k >= S / 2 && !((now >> k) & 1u) && gk >= thr_r && gk > -INFINITY;
          });
          wave_lds_sync();
#pragma unroll
          for (int sub = 0; sub < 8; ++sub) fetch(0, sub);
        } else if (lane < 8) {
          gstart[w * 8 + lane] = kLgNone;
        }
        lds_barrier();
        const bool more = shared_i[4 + par] != 0;    // some wave's list takes a second turn
        par ^= 1;
        if (!more) break;
      }
      fresh = np > 0 ? now : (fresh | now);
      have_r = true;
      lds_barrier();                               // stages and chunks are dead: the next epoch reuses the union
    }
  }

  // ---- sort(S): flag the picked tokens, ascending indices by prefix counts
  lds_barrier();
#pragma unroll
  for (int k = 0; k < S; ++k) flag[base + 64 * k + lane] = 0;
  lds_barrier();
  for (int u = tid; u < t; u += NT) flag[kvr_ix(order_l[u], 64 * S * W, 414)] = 1;   // 414: token of a pick
  lds_barrier();
  if (starved) {
    if (tid == 0) {                                  // non-finite input only: lowest unpicked tokens fill up
      int j = 0;
      for (int u = t; u < b; ++u) {
        while (j < n - 1 && flag[j]) ++j;
        order_l[u] = j; gain_l[u] = -INFINITY; flag[j] = 1;
      }
    }
    lds_barrier();
  }
  {
    unsigned long long sel[S];
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < S; ++k) {
      sel[k] = __ballot(tok_of(k) < n && flag[tok_of(k)] != 0);
      cnt += __popcll(sel[k]);
    }
    if (lane == 0) wcount[w] = cnt;
    lds_barrier();
    int off = 0;
    for (int u = 0; u < w; ++u) off += wcount[u];
#pragma unroll
    for (int k = 0; k < S; ++k) {
      if ((sel[k] >> lane) & 1ull) {
        const int rank = off + __popcll(sel[k] & ((1ull << lane) - 1ull));
        if (rank < b) idxs_l[rank] = tok_of(k);
      }
      off += __popcll(sel[k]);
    }
  }
  lds_barrier();
  const int bs = a.b;
  const long long ob = static_cast<long long>(h) * bs;
  for (int u = tid; u < b; u += NT) {
    a.idx_sorted[ob + u] = idxs_l[u];
    if (a.pick_order) a.pick_order[ob + u] = order_l[u];
    if (a.pick_gain) a.pick_gain[ob + u] = gain_l[u];
  }
  if constexpr (BUD) {
    for (int u = b + tid; u < bs; u += NT) {                   // entries past the head's budget are padding
      a.idx_sorted[ob + u] = -1;
      if (a.pick_order) a.pick_order[ob + u] = -1;
      if (a.pick_gain) a.pick_gain[ob + u] = -INFINITY;
    }
  }
  if ((a.K_out || a.V_out) && (!BUD || b > 0))
    compact_rows<4>(a.K, a.V, a.K_out, a.V_out, head_off, a.stride_tok, idxs_l, n, b, ob, tid, NT);
}

KVR_BOUNDS_TU(large)

bool large_supported(const Layout& lay, int b) {
  return lay.dtype == DT_BF16 && lay.n > 4096 && lay.n <= 8192 && b <= kLgMaxB;
}

hipError_t launch_select_large(const void* K, const void* V, const float* s, const Layout& lay, int b,
                               float lambda, float eps, int32_t* idx_sorted, int32_t* pick_order,
                               float* pick_gain, void* K_out, void* V_out, hipStream_t st, const int32_t* b_h) {
  LargeArgs a;
  a.b_h = b_h;
  a.K = static_cast<const char*>(K); a.V = static_cast<const char*>(V); a.s_in = s;
  a.idx_sorted = idx_sorted; a.pick_order = pick_order; a.pick_gain = pick_gain;
  a.K_out = static_cast<char*>(K_out); a.V_out = static_cast<char*>(V_out);
  a.stride_head = lay.stride_head; a.stride_tok = lay.stride_tok;
  a.n = lay.n; a.b = b; a.lambda = lambda; a.eps = eps;
  auto go = [&](auto kern, int smem) -> hipError_t {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(lay.heads), dim3(kLgThreads), smem, st, a);
    return hipGetLastError();
  };
  auto by_shape = [&](auto bud) -> hipError_t {
    constexpr bool BUD = decltype(bud)::value;
    if (static_cast<long long>(lay.n) * lay.stride_tok * 2 >= (1ll << 31))
      return go(&select_large_kernel<16, BUD, true>, LargeCfg<16>::smem_bytes(b));
    return go(&select_large_kernel<16, BUD, false>, LargeCfg<16>::smem_bytes(b));
  };
  return b_h ? by_shape(std::true_type{}) : by_shape(std::false_type{});
}

}  // namespace kvr
