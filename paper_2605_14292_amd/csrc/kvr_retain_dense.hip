// Fused retention step for heads with n <= 256 bf16 tokens: from HBM to the compacted rows in one launch.
//
//   score    (optional, G <= 8)  logits Q K^T on bf16 MFMA, softmax over the
//            tokens per query, mean over queries             (base-score stand-in)
//   norms    r_j = 1/(||V_j|| + eps) from the Gram diagonal  (paper Eq. 1)
//   Gram     lower-triangular 32x32 tiles of V V^T on bf16 MFMA with fp32
//            accumulation, scaled to cosines and parked in LDS as a packed or padded
//            triangle of fp32                                (Algorithm 1, Sims)
//   greedy   one wave keeps s, m and the alive set in registers (token j lives
//            in lane j%64) and runs the race of kvr_dense_common.hpp   (Eq. 2-3, Alg. 1)
//   compact  rows at the ascending picks are copied to the dense outputs
//
// The raw bf16 rows go through the MFMA un-normalised (bf16 x bf16 products are
// exact in fp32); the cosine is dot * r_i * r_j in fp32.  Rounding normalised
// rows to bf16 first would put ~4e-3 on every cosine.
//
// Persistent workgroups, each a pipeline over its heads: while wave 0 runs the pick chain of head h, the other waves
// write out head h-1 and prepare head h+1: its scores (wave 1, K straight into operand registers), its V rows (the waves
// after it, in registers).  When the chain is done the rows are staged over the dead triangle, all waves compute the Gram
// tiles and the norms and write the next triangle, and the next chain starts.
// The order of the sums decides near-ties, so the norms come from the Gram's diagonal, as in retain_dense16_kernel (a head's
// picks are the same bits in both), and the softmax denominators are summed as four groups of blocks.  Norms from
// dot products of the rows in registers, off the chain, were 1-2 % faster at 128 and 192 tokens (nothing at 256) but moved
// the cosines' last bits, and 2 of 37632 heads (n=251, b=101) kept another token.  Norms off the chain from products of
// the blocks with themselves, V loaded as operands: the same bits, but up to 8 % slower at 128 tokens.
//
// What bounds it is the chain of dependent picks, which uses one wave, times the heads a CU holds at once: one of 256
// tokens (the triangle takes 132 of the CU's 160 KB of LDS), two of 192 (75 KB), three of 128 and four of 64 tokens
// (registers).  Measured with one phase after the other and the compiler's race -> this pipeline, scores from 7 queries: 4096 heads:
// n=192, b=64 213 -> 155, n=128, b=64 175 -> 111; 8192 heads, n=64, b=48 234 -> 123; one head, n=128, b=64 19.0 -> 15.5, 256
// heads 20.5 -> 17.  Scores far below lambda given: 4096 heads, n=128, b=64 153 -> 84.
//
// Heads of more than 192 tokens: between two chains of such a head stand 0.6 us of staging, 1.8 of Gram and 1.9 of triangle beside 14.1
// of chain (n = 251, b = 101), and only the triangle needs the place of the one before.  So under AHEAD the waves 2 .. 7 stage the next head's rows a
// quarter of their columns at a time in the 16 KB beside the triangle, run the Gram and scale it to cosines while the chain runs (they meet at
// a counter, the chain's wave is not asked), and what is left between two chains is the stores (6 700 cycles with the scaling among them, 4 600 now, beside
// 32 500 of chain and 900 of sorting).  2688 heads of 251 tokens, b=101 414 us one phase after the other, 220 with the Gram between the chains, 209 with the packed triangle,
// 194 beside them; 8192 of 250, b=128, tight scores given 785 -> 696; 257 of 256, b=128 54.8 -> 51.2.  With short chains there is nothing to hide behind:
// gram_ahead_pays.
// Tried: the Gram beside the chain with its operands loaded from memory in the MFMA layout: the 450 gathered loads of a head of 256 tokens take
// 12 us whatever the prefetch depth or the bytes per row and request, the address unit spending 64 cycles on each (239 us); and no triangle
// at all, the cosines of 32 candidates at a time from rows of V held as operands in registers, three heads per CU (238 us: twelve waves'
// instructions per pick are more than the idle SIMDs have room for).
// The roles are separate loops with matching barriers, not one loop with branches: registers of one role are not carried
// through the other.
#include "kvr_dense_common.hpp"
#include "kvr_kernels.hpp"

namespace kvr {

constexpr int kMaxB = 256;
struct DenseArgs {
  const char* K; const char* V; const char* Q; const float* s_in;
  float* s_out; int32_t* idx_sorted; int32_t* pick_order; float* pick_gain;
  char* K_out; char* V_out;
  long long stride_head, stride_tok;   // elements
  int n, b, G, heads;
  float lambda, eps;
  int only_marked;                     // process only heads whose idx_sorted[h*b] is -1
  const int32_t* b_h;                  // per-head budgets <= b (rows of the outputs stay b apart), or null
};

template <int NT, bool GRAM_AHEAD = false> struct DenseCfg {
  static constexpr int W = NT == 8 ? 8 : 4;           // waves
  static constexpr int OCC = NT == 8 ? 1 : (NT == 6 ? 2 : (NT == 4 ? 3 : 4));   // heads per CU; up to 128 tokens the registers set it, above LDS
  static constexpr int N32 = NT * 32;
  static constexpr int OFFD = NT * (NT - 1) / 2;      // tiles of the lower triangle off its diagonal
  // One head per CU: the Gram of the next head can run beside the chain as well, on the waves 2 .. 7, its rows staged a quarter of their columns
  // at a time in the 16 KB that the triangle leaves (gram_ahead_pays says when).
  static constexpr bool AHEAD = GRAM_AHEAD;
  static_assert(!AHEAD || NT == 8, "one head per CU");
  static constexpr int GW = 6, GT = NT * (NT + 1) / 2 / GW;   // (then) waves with tiles, tiles of each
  static constexpr int kQuarter = AHEAD ? N32 * 64 : 0, kMet = AHEAD ? 16 : 0;
  static_assert(!AHEAD || GT * GW == NT * (NT + 1) / 2, "equal shares");
  static constexpr int MAXD = (NT + W - 1) / W, MAXO = (OFFD + W - 1) / W;   // Gram tiles per wave, on the diagonal and off it
  static constexpr int ROWS = (N32 * 16 + 64 * (W - 2) - 1) / (64 * (W - 2));   // 16-byte row pieces per thread of waves 2 ..
  static constexpr int bcap(int b) { return (b + 63) & ~63; }
  // The triangle: packed, or with rows padded to 16-byte stores.  Padded rows are written faster and read with bank conflicts (a pick of 256
  // tokens 24 cycles longer).  One head per CU waits for its picks: 2688 heads of 251 tokens, b = 101 220 us padded, 209 packed; 257 of 256, b = 128 54.8
  // and 52.5.  Several heads share the LDS's store rate: 4096 of 192, b = 64 156 and 159, of 128 110 and 111; 8192 of 64 122 and 125.
  static constexpr bool PACKED = NT == 8;
  static constexpr int kTriBytes = PACKED ? dense_tri_floats(NT) * 4 : padded_tri_floats(N32) * 4;
  static constexpr int region = !AHEAD && N32 * kRowPitch > kTriBytes ? N32 * kRowPitch : kTriBytes;   // (AHEAD: rows are not staged there)
  // triangle or staged rows | quarter of the rows | s_l[2][N32] | rinv[N32] | met (AHEAD) | lists [2][order, gain][bcap] | [2][idx][bcap], 16 bits each: with 32
  // two heads of 192 tokens and more than 128 picks do not fit a CU (4096 heads, n=192, b=160 412 us; now 244, and 377 before the lists came in pairs)
  static constexpr int smem_bytes(int b) { return region + kQuarter + N32 * 3 * 4 + kMet + 2 * bcap(b) * (4 + 4 + 2); }
  static_assert(OCC * (region + kQuarter + N32 * 3 * 4 + kMet + 2 * N32 * (4 + 4 + 2)) <= 160 * 1024, "OCC heads fit a CU at every budget");
};

template <int NT, bool GRAM_AHEAD>
__global__ __launch_bounds__(64 * DenseCfg<NT>::W, DenseCfg<NT>::W * DenseCfg<NT>::OCC / 4) void retain_dense_kernel(DenseArgs a) {
  using C = DenseCfg<NT, GRAM_AHEAD>;
  constexpr int N32 = C::N32, NQ = NT / 2, W = C::W, ROWS = C::ROWS;
  extern __shared__ __align__(16) char smem[];
  char* stage = smem;
  float* tri = reinterpret_cast<float*>(smem);
  char* quarter = smem + C::region;                     // [N32][64 B]
  float* s_all = reinterpret_cast<float*>(quarter + C::kQuarter);   // [2][N32]
  float* rinv = s_all + 2 * N32;                        // inverse norms of the head whose triangle is being built
  const int bcap = C::bcap(a.b);
  int32_t* met = reinterpret_cast<int32_t*>(rinv + N32);     // [4] how often the waves with tiles have met (AHEAD)
  int32_t* lists = met + C::kMet / 4;                   // [2][2][bcap]: picks in order, gains
  uint16_t* idx_all = reinterpret_cast<uint16_t*>(lists + 4 * bcap);   // [2][bcap]: ascending indices

  int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = a.n, b = a.b;
  const bool diverse = a.lambda != 0.0f;
  const bool need_v = diverse && b > 1;
  // First head at or after h0 on this workgroup's stride that is to be processed.  With only_marked set, an earlier kernel
  // has already finished every head it did not mark; 64 marks are looked at per round trip to memory.
  auto next_head = [&](int h0) -> int {
    if (!a.only_marked) return h0;
    for (long long base = h0; base < a.heads; base += 64ll * gridDim.x) {
      const long long hh = base + static_cast<long long>(lane) * gridDim.x;
      const unsigned long long m = __ballot(hh < a.heads && a.idx_sorted[hh * a.b] == -1);
      if (m) return static_cast<int>(base) + (__ffsll(static_cast<long long>(m)) - 1) * static_cast<int>(gridDim.x);
    }
    return a.heads;
  };
  auto budget = [&](int h) -> int { return a.b_h ? __builtin_amdgcn_readfirstlane(min(max(a.b_h[h], 0), b)) : b; };
  // Staged rows -> triangle, by all waves.  A wave takes its diagonal tiles first, then its share of the others, row by row:
  // the norms (Eq. 1, from the diagonal of the Gram) are worked out under the products of its first other tile.
  auto build_triangle = [&]() __attribute__((always_inline)) {
    lds_barrier();                                      // the rows are staged
    const int o0 = wave * C::OFFD / W, cnt = (wave + 1) * C::OFFD / W - o0;
    int I0 = 1;
    while (I0 * (I0 + 1) / 2 <= o0) ++I0;
    f32x16 accd[C::MAXD], acc[C::MAXO];
    if (need_v) {
      bf16x8 fi[8];
#pragma unroll
      for (int d = 0; d < C::MAXD; ++d) {
        accd[d] = f32x16{0};
        if (wave + W * d < NT) {
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) fi[ks] = frag_at(stage, wave + W * d, ks, lane);
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) accd[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fi[ks], fi[ks], accd[d], 0, 0, 0);
        }
      }
      int I = I0, J = o0 - I0 * (I0 - 1) / 2;
      if (cnt > 0) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) fi[ks] = frag_at(stage, I, ks, lane);
      }
#pragma unroll
      for (int sl = 0; sl < C::MAXO; ++sl) {
        acc[sl] = f32x16{0};
        if (sl < cnt) {
#pragma unroll
          for (int ks = 0; ks < 8; ++ks)
            acc[sl] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_at(stage, J, ks, lane), fi[ks], acc[sl], 0, 0, 0);
          if (++J == I) {
            ++I; J = 0;
            if (sl + 1 < cnt) {
#pragma unroll
              for (int ks = 0; ks < 8; ++ks) fi[ks] = frag_at(stage, I, ks, lane);
            }
          }
        }
        if (sl == 0) {
#pragma unroll
          for (int d = 0; d < C::MAXD; ++d) {
            if (wave + W * d < NT) {
              // element r of lane (l32, hf) is row 8 (r / 4) + 4 hf + r % 4 of the tile: row l32 sits in one of its two lanes
              auto pick = [](int bit, float one, float zero) { return bit ? one : zero; };   // (by value: a choice between two elements would put the array in memory)
              float v8[8], v4[4];
#pragma unroll
              for (int k = 0; k < 8; ++k) v8[k] = pick(l32 & 1, accd[d][2 * k + 1], accd[d][2 * k]);
#pragma unroll
              for (int k = 0; k < 4; ++k) v4[k] = pick(l32 & 2, v8[2 * k + 1], v8[2 * k]);
              const float ss = pick(l32 & 16, pick(l32 & 8, v4[3], v4[2]), pick(l32 & 8, v4[1], v4[0]));
              if (((l32 >> 2) & 1) == hf) rinv[(wave + W * d) * 32 + l32] = 1.0f / (sqrtf(ss) + a.eps);
            }
          }
        }
      }
    }
    lds_barrier();                                      // every wave has read its rows: the triangle takes their place
    if (need_v) {
      auto write_tile = [&](const f32x16& t, int I, int J) {
        if constexpr (C::PACKED) write_cos_tile_rows(tri, rinv, t, I, J, lane);
        else write_cos_tile_padded(tri, rinv, t, I, J, lane);
      };
#pragma unroll
      for (int d = 0; d < C::MAXD; ++d)
        if (wave + W * d < NT) write_tile(accd[d], wave + W * d, wave + W * d);
      int I = I0, J = o0 - I0 * (I0 - 1) / 2;
#pragma unroll
      for (int sl = 0; sl < C::MAXO; ++sl) {
        if (sl < cnt) write_tile(acc[sl], I, J);
        if (++J == I) { ++I; J = 0; }
      }
    }
    lds_barrier();                                      // triangle and scores are complete: the chain starts
  };
  // The tiles of the waves 2 .. 7 under AHEAD, row by row: tile I (I + 1) / 2 + J is row block I, column block J.
  f32x16 acc6[C::AHEAD ? C::GT : 1];
  int mt = 0;                                           // how often this wave should have been met
  auto meet = [&]() __attribute__((always_inline)) {                                   // among the waves 2 .. 7, which all come here equally often
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (lane == 0) __hip_atomic_fetch_add(met, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    mt += C::GW;
    while (__hip_atomic_load(met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < mt) __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");
  };
  // Rows in registers -> cosines in acc6.  Sixteen rows' pieces of one number lie on sixteen different bank groups.
  auto gram_ahead = [&](auto store_quarter) __attribute__((always_inline)) {
    const int first = (wave - 2) * C::GT;
    int I0 = 0;
    while ((I0 + 1) * (I0 + 2) / 2 <= first) ++I0;
    const int J0 = first - I0 * (I0 + 1) / 2;
#pragma unroll
    for (int k = 0; k < C::GT; ++k) acc6[k] = f32x16{0};
    auto piece = [&](int block, int p) __attribute__((always_inline)) -> bf16x8 {
      const int row = block * 32 + l32;
      return *reinterpret_cast<const bf16x8*>(quarter + row * 64 + ((p ^ (row >> 2)) & 3) * 16);
    };
#pragma unroll 1
    for (int kq = 0; kq < 4; ++kq) {
      store_quarter(kq);
      meet();                                           // the quarter is staged
      int I = I0, J = J0, held = -1;
      bf16x8 fi[2];
#pragma unroll
      for (int k = 0; k < C::GT; ++k) {
        if (I != held) { fi[0] = piece(I, hf); fi[1] = piece(I, 2 + hf); held = I; }
        acc6[k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece(J, hf), fi[0], acc6[k], 0, 0, 0);
        acc6[k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece(J, 2 + hf), fi[1], acc6[k], 0, 0, 0);
        if (++J > I) { ++I; J = 0; }
      }
      meet();                                           // ... and read
    }
    int I = I0, J = J0;
#pragma unroll
    for (int k = 0; k < C::GT; ++k) {
      if (I == J) {                                     // (as in build_triangle)
        auto pick = [](int bit, float one, float zero) { return bit ? one : zero; };
        float v8[8], v4[4];
#pragma unroll
        for (int q = 0; q < 8; ++q) v8[q] = pick(l32 & 1, acc6[k][2 * q + 1], acc6[k][2 * q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) v4[q] = pick(l32 & 2, v8[2 * q + 1], v8[2 * q]);
        const float ss = pick(l32 & 16, pick(l32 & 8, v4[3], v4[2]), pick(l32 & 8, v4[1], v4[0]));
        if (((l32 >> 2) & 1) == hf) rinv[I * 32 + l32] = 1.0f / (sqrtf(ss) + a.eps);
      }
      if (++J > I) { ++I; J = 0; }
    }
    meet();                                             // the norms are complete
    I = I0; J = J0;
#pragma unroll
    for (int k = 0; k < C::GT; ++k) {
      scale_cos_tile(rinv, acc6[k], I, J, lane);
      if (++J > I) { ++I; J = 0; }
    }
  };
  // Between two chains under AHEAD: the tiles into the triangle's place.
  auto write_ahead = [&]() __attribute__((always_inline)) {
    lds_barrier();                                      // the triangle is dead
    if (wave >= 2 && need_v) {
      const int first = (wave - 2) * C::GT;
      int I = 0;
      while ((I + 1) * (I + 2) / 2 <= first) ++I;
      int J = first - I * (I + 1) / 2;
#pragma unroll
      for (int k = 0; k < C::GT; ++k) {
        store_cos_tile(tri, acc6[k], I, J, lane);
        if (++J > I) { ++I; J = 0; }
      }
    }
    lds_barrier();                                      // triangle and scores are complete: the chain starts
  };
  int h = next_head(blockIdx.x);
  if (h >= a.heads) return;                             // (uniform over the workgroup)
  if constexpr (C::AHEAD) {
    if (tid == 0) met[0] = 0;
    lds_barrier();
  }

  if (wave == 0) {
    // ---------------------------------------------------------------- the chain
    if constexpr (C::AHEAD) write_ahead(); else build_triangle();
    for (int par = 0; h < a.heads; par ^= 1) {
      const int h_next = next_head(h + gridDim.x);
      const int bh = budget(h), brun = bh < 1 ? 1 : bh;
      int32_t* order_l = lists + par * 2 * bcap;
      float* s_l = s_all + par * N32;
      __builtin_amdgcn_s_setprio(3);                    // the waves that share its SIMD have time to spare
      pick_chain<NQ, !C::PACKED>(s_l, tri, order_l, reinterpret_cast<float*>(order_l + bcap), n, brun, a.lambda, diverse, lane);
      sort_picks<NQ>(order_l, idx_all + par * bcap, reinterpret_cast<int32_t*>(s_l), brun, lane, nullptr);   // (the scores are dead by now)
      __builtin_amdgcn_s_setprio(0);
      h = h_next;
      if constexpr (C::AHEAD) {
        if (h < a.heads) write_ahead(); else lds_barrier();   // the triangle of h is dead
      } else {
        lds_barrier();                                  // the triangle of h is dead
        if (h < a.heads) build_triangle();
      }
    }
    return;
  }

  // ---------------------------------------------------------------- everything else
  constexpr int nthr = 64 * (W - 1);
  int t0 = tid - 64;
  const long long tok_bytes = a.stride_tok * 2;
  auto score = [&](int hh, float* s_l) {                // wave 1 only
    if (!a.Q) {
#pragma unroll
      for (int k = 0; k < (N32 + 63) / 64; ++k) {
        const int j = lane + 64 * k;
        s_l[j] = j < n ? a.s_in[static_cast<long long>(hh) * n + min(j, n - 1)] : -INFINITY;   // padding never competes
      }
      return;
    }
    const char* Kh = a.K + hh * a.stride_head * 2;
    auto load_block = [&](int blk, bf16x8 (&f)[8]) {    // rows past n: the last row again (masked below)
      const char* p = Kh + min(blk * 32 + l32, n - 1) * tok_bytes + hf * 16;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const uint4 x = *reinterpret_cast<const uint4*>(p + ks * 32);
        f[ks] = *reinterpret_cast<const bf16x8*>(&x);
      }
    };
    constexpr int KD = NT <= 4 ? 2 : 4;                 // blocks of K in flight
    bf16x8 qf[8], kf[KD][8];
    {
      const char* qp = a.Q + (static_cast<long long>(hh) * a.G + min(l32, a.G - 1)) * kD * 2 + hf * 16;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const uint4 x = *reinterpret_cast<const uint4*>(qp + ks * 32);
        qf[ks] = *reinterpret_cast<const bf16x8*>(&x);  // (rows past G repeat the last query; their results are not used)
      }
    }
    float z[NT][4];                                     // lane (token l32 of block I, hf): queries hf*4 + r
#pragma unroll
    for (int I = 0; I < KD; ++I) load_block(I, kf[I]);
    const float scale = 0.08838834764831845f;           // 1/sqrt(128)
    float zmax[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int I = 0; I < NT; ++I) {
      f32x16 d = {0};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], kf[I % KD][ks], d, 0, 0, 0);
      if (I + KD < NT) load_block(I + KD, kf[I % KD]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z[I][r] = I * 32 + l32 < n ? d[r] * scale : -INFINITY;
        zmax[r] = fmaxf(zmax[r], z[I][r]);
      }
    }
    const float invG = 1.0f / static_cast<float>(a.G);
    float w[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float v = half_max_at_31(zmax[r]);
      zmax[r] = __shfl(v, lane | 31, kWave);
      // The denominator in four sums, of the blocks I % 4, added in that order.  (The order is kept as the scores' last bits,
      // and with them near-ties at the budget's edge, depend on it.)
      float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int I = 0; I < NT; ++I) { z[I][r] = __expf(z[I][r] - zmax[r]); sum[I & 3] += z[I][r]; }   // exp(-inf) = 0: padding
      half_sums_at_31(sum);
      v = __shfl(sum[0] + sum[1] + sum[2] + sum[3], lane | 31, kWave);
      w[r] = hf * 4 + r < a.G ? invG / v : 0.f;
    }
#pragma unroll
    for (int I = 0; I < NT; ++I) {
      float p = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) p = fmaf(z[I][r], w[r], p);
      p += __shfl_xor(p, 32, kWave);                    // queries 0-3 live in lanes 0-31, 4-7 in 32-63
      const int j = I * 32 + l32;
      if (hf == 0) {
        s_l[j] = j < n ? p : -INFINITY;
        if (j < n && a.s_out) a.s_out[static_cast<long long>(hh) * n + j] = p;
      }
    }
  };
  // V rows of head hh: 16 threads a row; rows past n are the last row again (never picked)
  constexpr int NR = 64 * (W - 2);
  int r0 = tid - 128;
  uint4 vrow[ROWS];
  auto fetch = [&](int hh) {
    const char* Vh = a.V + hh * a.stride_head * 2 + (r0 & 15) * 16;
#pragma unroll
    for (int k = 0; k < ROWS; ++k)
      vrow[k] = *reinterpret_cast<const uint4*>(Vh + min((r0 >> 4) + k * (NR / 16), n - 1) * tok_bytes);
  };
  auto store_stage = [&]() __attribute__((always_inline)) {
    if (!need_v || wave == 1) return;
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int row = (r0 >> 4) + k * (NR / 16);
      if (row < N32) *reinterpret_cast<uint4*>(stage + row * kRowPitch + (r0 & 15) * 16) = vrow[k];
    }
  };
  auto output = [&](int hh, int par) {
    const int bh = budget(hh);
    const int32_t* order_l = lists + par * 2 * bcap;
    const uint16_t* idx_l = idx_all + par * bcap;
    const long long ob = static_cast<long long>(hh) * b;
    for (int t = t0; t < b; t += nthr) {                // entries past the head's budget are padding
      a.idx_sorted[ob + t] = t < bh ? idx_l[t] : -1;
      if (a.pick_order) a.pick_order[ob + t] = t < bh ? order_l[t] : -1;
      if (a.pick_gain) a.pick_gain[ob + t] = t < bh ? reinterpret_cast<const float*>(order_l)[bcap + t] : -INFINITY;
    }
    if ((a.K_out || a.V_out) && bh > 0)
      compact_rows<4>(a.K, a.V, a.K_out, a.V_out, hh * a.stride_head * 2, a.stride_tok, idx_l, n, bh, ob, t0, nthr);
  };

  auto prepare = [&](int hh, float* s_l) {
    if (wave == 1) {
      score(hh, s_l);
      // (defined here by nothing: the row registers are not carried through the scores)
#pragma unroll
      for (int k = 0; k < ROWS; ++k) asm volatile("" : "=v"(vrow[k].x), "=v"(vrow[k].y), "=v"(vrow[k].z), "=v"(vrow[k].w));
    } else if (need_v) {
      fetch(hh);
    }
  };
  // (AHEAD) the threads that hold pieces of quarter kq of the rows put them down
  auto store_quarter = [&](int kq) __attribute__((always_inline)) {
    if (((r0 & 15) >> 2) != kq) return;
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int row = (r0 >> 4) + k * (NR / 16);
      if (row < N32) *reinterpret_cast<uint4*>(quarter + row * 64 + ((r0 ^ (row >> 2)) & 3) * 16) = vrow[k];
    }
  };
  auto next_triangle = [&]() __attribute__((always_inline)) {
    if constexpr (C::AHEAD) {
      if (need_v && wave >= 2) gram_ahead(store_quarter);
      write_ahead();
    } else {
      store_stage();
      build_triangle();
    }
  };
  prepare(h, s_all);
  next_triangle();
  int h_prev = -1;
  for (int par = 0; h < a.heads; par ^= 1) {
    const int h_next = next_head(h + gridDim.x);
    // (opaque once per head: otherwise every per-lane address of the body is loop-invariant and lives in registers)
    asm volatile("" : "+v"(tid));
    lane = tid & 63; hf = lane >> 5; l32 = lane & 31; t0 = tid - 64; r0 = tid - 128;
    if (h_prev >= 0) output(h_prev, par ^ 1);
    if (h_next < a.heads) {
      prepare(h_next, s_all + (par ^ 1) * N32);
      if constexpr (!C::AHEAD) lds_barrier();           // the chain of h is done, its triangle dead
      next_triangle();
    } else {
      lds_barrier();
      output(h, par);
    }
    h_prev = h;
    h = h_next;
  }
}

bool dense_supported(const Layout& lay, int b, int G, bool has_q) {
  return lay.dtype == DT_BF16 && lay.n <= 256 && b <= kMaxB && (!has_q || G <= 8);
}

// Whether the Gram of a workgroup's next head runs beside the chain (DenseCfg::AHEAD) or between two chains, heads of 193-256 tokens.  Beside it,
// six waves instead of eight meet eight times a head, and a workgroup's first head has no chain to hide that behind: it pays where the
// chain is long, and with queries (whose scores need one wave the longest) sooner.  Between / beside, us:
//   scores given, 2688 heads of 256, b = 2 / 32 / 64 / 80:  104 / 138, 126 / 153, 172 / 173, 197 / 186;  of 200, b = 64:  171 / 166
//   ... at most two heads per CU, 257 of 200, b = 24 / 64 / 128:  25.7 / 30.6, 36.4 / 38.2, 55.5 / 56.7;  512 of 224, b = 128: 0.989x beside; 700: 1.011x
//   7 queries, 700 heads of 200, b = 24 / 48 / 56 / 64 / 80:  36.7 / 40.0, 42.4 / 44.7, 45.4 / 45.9, 48.7 / 47.4, 55.5 / 52.7
//   ... at most two heads per CU, 257 of 240, b = 24 / 48 / 56:  23.0 / 25.3, 29.0 / 29.0, 31.1 / 30.1
// With queries and short chains the event is bound by its reads once K and V exceed the memory-side cache, and beside the chain they are requested
// sooner: 3072 heads (1 / 4 / 7 queries alike) of 256, b = 2 / 24 / 40: 1.08x, 1.06x, 1.03x beside; of 193, b = 24 / 40: 1.00x, 0.96x;
// inside the cache, 1536 of 256, b = 24: 0.96x.
bool gram_ahead_pays(int heads, int n, int b, bool queries, int cus) {
  const bool few = heads <= 2 * cus;
  if (b >= (queries && few ? 56 : 64)) return queries || !few;
  const bool past_cache = static_cast<long long>(heads) * n * (2 * kD * 2) >= 256ll << 20;
  return queries && past_cache && (n >= 240 || b <= 24);
}

hipError_t launch_retain_dense(const void* K, const void* V, const void* Q, int G, const float* s_in,
                               const Layout& lay, int b, float lambda, float eps, float* s_out,
                               int32_t* idx_sorted, int32_t* pick_order, float* pick_gain,
                               void* K_out, void* V_out, hipStream_t st, bool only_marked, const int32_t* b_h) {
  DenseArgs a;
  a.only_marked = only_marked ? 1 : 0;
  a.b_h = b_h;
  a.K = static_cast<const char*>(K); a.V = static_cast<const char*>(V);
  a.Q = static_cast<const char*>(Q); a.s_in = s_in; a.s_out = s_out;
  a.idx_sorted = idx_sorted; a.pick_order = pick_order; a.pick_gain = pick_gain;
  a.K_out = static_cast<char*>(K_out); a.V_out = static_cast<char*>(V_out);
  a.stride_head = lay.stride_head; a.stride_tok = lay.stride_tok;
  a.n = lay.n; a.b = b; a.G = G; a.heads = lay.heads; a.lambda = lambda; a.eps = eps;
  const int cus = cu_count();
  auto go = [&](auto kern, int smem, int threads, int most) -> hipError_t {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    // persistent workgroups: as many as fit the chip at once (LDS-limited), never more than heads
    int per_cu = 160 * 1024 / smem;
    per_cu = per_cu < 1 ? 1 : (per_cu > most ? most : per_cu);
    const int blocks = lay.heads < cus * per_cu ? lay.heads : cus * per_cu;
    dim3 grid(blocks);
    hipLaunchKernelGGL(kern, grid, dim3(threads), smem, st, a);
    return hipGetLastError();
  };
  auto launch = [&](auto kern, auto cfg) -> hipError_t {
    using C = decltype(cfg);
    return go(kern, C::smem_bytes(b), 64 * C::W, C::OCC);
  };
  if (lay.n <= 64) return launch(&retain_dense_kernel<2, false>, DenseCfg<2>{});
  if (lay.n <= 128) return launch(&retain_dense_kernel<4, false>, DenseCfg<4>{});
  if (lay.n <= 192) return launch(&retain_dense_kernel<6, false>, DenseCfg<6>{});
  if (gram_ahead_pays(lay.heads, lay.n, b, Q != nullptr, cus)) return launch(&retain_dense_kernel<8, true>, DenseCfg<8, true>{});
  return launch(&retain_dense_kernel<8, false>, DenseCfg<8>{});
}

}  // namespace kvr
