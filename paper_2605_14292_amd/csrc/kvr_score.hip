// Base scores: s_i = (1/G) sum_g softmax_i(q_g . k_i / sqrt(d)).
// (Stand-in for the external scorer of paper Sec. 4.1, which takes s as given.)
//
// One workgroup per head.  A group of 16 lanes owns one K row per step (16
// bytes of bf16 or 32 bytes of fp32 per lane, so a wave reads four whole rows
// with one coalesced request); the query slices a lane needs stay in
// registers.  The logits of the head are kept in LDS when G*n floats fit, so K
// is read from HBM exactly once; otherwise the logits are recomputed in a
// second pass.
#include "kvr_kernels.hpp"
#include "kvr_topb.hpp"

namespace kvr {

constexpr int kScoreThreads = 256;
constexpr int kGT = 8;                       // queries handled per register tile
constexpr int kZMaxFloats = 16384;           // logits kept in LDS (64 KB)

template <int DT>
__device__ __forceinline__ void row_logits(const char* Kh, long long stride_tok, int j, int c,
                                           const float (&q)[kGT][8], int gcount, float scale,
                                           float (&z)[kGT]) {
  float k[8];
  load8<DT>(Kh + (static_cast<long long>(j) * stride_tok + c * 8) * elem_bytes<DT>(), k);
#pragma unroll
  for (int g = 0; g < kGT; ++g) {
    float acc = 0.f;
    if (g < gcount) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(k[e], q[g][e], acc);
      acc = group16_sum(acc) * scale;
    }
    z[g] = acc;
  }
}

template <int DT, bool ZFITS>
__global__ __launch_bounds__(kScoreThreads) void score_kernel(const void* __restrict__ K,
                                                              const void* __restrict__ Q, int G,
                                                              Layout lay,
                                                              float* __restrict__ s_out) {
  extern __shared__ float smem[];
  // smem: zbuf[G*n] (ZFITS) | acc[n] ; then red[2*kGT*4]
  const int n = lay.n;
  float* zbuf = smem;                                 // ZFITS: [G][n]
  float* acc = smem + (ZFITS ? G * n : 0);            // [n] running mean
  float* red = acc + n;                               // [4 waves][kGT] x2
  const int h = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15;                            // 16-byte chunk of the row
  const int rsub = tid >> 4;                          // row within a step (0..15)
  const char* Kh = static_cast<const char*>(K) + h * lay.stride_head * elem_bytes<DT>();
  const char* Qh = static_cast<const char*>(Q) +
                   static_cast<long long>(h) * G * kD * elem_bytes<DT>();
  const float scale = 0.08838834764831845f;           // 1/sqrt(128)
  const float invG = 1.0f / static_cast<float>(G);

  for (int j = tid; j < n; j += kScoreThreads) acc[j] = 0.f;

  for (int g0 = 0; g0 < G; g0 += kGT) {
    const int gcount = min(kGT, G - g0);
    float q[kGT][8];
#pragma unroll
    for (int g = 0; g < kGT; ++g) {
      if (g < gcount) {
        load8<DT>(Qh + (static_cast<long long>(g0 + g) * kD + c * 8) * elem_bytes<DT>(), q[g]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) q[g][e] = 0.f;
      }
    }
    // pass A: logits, running max per query
    float zmax[kGT];
#pragma unroll
    for (int g = 0; g < kGT; ++g) zmax[g] = -INFINITY;
    for (int j0 = 0; j0 < n; j0 += kScoreThreads / 16) {
      const int j = j0 + rsub;
      if (j < n) {
        float z[kGT];
        row_logits<DT>(Kh, lay.stride_tok, j, c, q, gcount, scale, z);
#pragma unroll
        for (int g = 0; g < kGT; ++g) {
          zmax[g] = fmaxf(zmax[g], z[g]);
          if (ZFITS && c == 0 && g < gcount) zbuf[(g0 + g) * n + j] = z[g];
        }
      }
    }
    // block max per query
#pragma unroll
    for (int g = 0; g < kGT; ++g) {
      float v = zmax[g];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
      if (lane == 0) red[wave * kGT + g] = v;
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kGT; ++g)
      zmax[g] = fmaxf(fmaxf(red[g], red[kGT + g]), fmaxf(red[2 * kGT + g], red[3 * kGT + g]));
    __syncthreads();
    // pass B: sum of exp per query
    float zsum[kGT];
#pragma unroll
    for (int g = 0; g < kGT; ++g) zsum[g] = 0.f;
    if (ZFITS) {
      for (int j = tid; j < n; j += kScoreThreads) {
#pragma unroll
        for (int g = 0; g < kGT; ++g)
          if (g < gcount) {
            const float e = __expf(zbuf[(g0 + g) * n + j] - zmax[g]);
            zbuf[(g0 + g) * n + j] = e;
            zsum[g] += e;
          }
      }
    } else {
      for (int j0 = 0; j0 < n; j0 += kScoreThreads / 16) {
        const int j = j0 + rsub;
        if (j < n) {
          float z[kGT];
          row_logits<DT>(Kh, lay.stride_tok, j, c, q, gcount, scale, z);
          if (c == 0) {
#pragma unroll
            for (int g = 0; g < kGT; ++g)
              if (g < gcount) zsum[g] += __expf(z[g] - zmax[g]);
          }
        }
      }
    }
#pragma unroll
    for (int g = 0; g < kGT; ++g) {
      float v = zsum[g];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
      if (lane == 0) red[wave * kGT + g] = v;
    }
    __syncthreads();
    float rinv[kGT];
#pragma unroll
    for (int g = 0; g < kGT; ++g)
      rinv[g] = 1.0f / (red[g] + red[kGT + g] + red[2 * kGT + g] + red[3 * kGT + g]);
    __syncthreads();
    // pass C: accumulate the mean of the softmax rows
    if (ZFITS) {
      for (int j = tid; j < n; j += kScoreThreads) {
        float a = acc[j];
#pragma unroll
        for (int g = 0; g < kGT; ++g)
          if (g < gcount) a = fmaf(zbuf[(g0 + g) * n + j], rinv[g] * invG, a);
        acc[j] = a;
      }
    } else {
      for (int j0 = 0; j0 < n; j0 += kScoreThreads / 16) {
        const int j = j0 + rsub;
        if (j < n) {
          float z[kGT];
          row_logits<DT>(Kh, lay.stride_tok, j, c, q, gcount, scale, z);
          if (c == 0) {
            float a = acc[j];
#pragma unroll
            for (int g = 0; g < kGT; ++g)
              if (g < gcount) a = fmaf(__expf(z[g] - zmax[g]), rinv[g] * invG, a);
            acc[j] = a;
          }
        }
      }
    }
    __syncthreads();
  }
  float* so = s_out + static_cast<long long>(h) * n;
  for (int j = tid; j < n; j += kScoreThreads) so[j] = acc[j];
}

// ---------------------------------------------------------------------------
// bf16, G <= 32 (GQ = 8 or 32 query rows of the MFMA's 32-row operand in use): the logits are a thin dense contraction ([G x d] x [d x n]), so
// they go through the matrix cores.  K is streamed from HBM once, straight into MFMA
// operand registers.  The logits of the head wait in LDS for the softmax.

// One head's scores on a workgroup of NW waves; finish(score_at) is called when they are there: score_at(j) is token j's.
template <int GQ, int NW, class Finish>
__device__ __forceinline__ void score_head(const char* __restrict__ K, const char* __restrict__ Q, int G, const Layout& lay,
                                           char* smem_raw, Finish finish) {
  float* zbuf = reinterpret_cast<float*>(smem_raw);                         // [G][n]
  const int n = lay.n;
  float* red = zbuf + G * n;                                                // [2][NW][GQ]
  const int h = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const char* Kh = K + h * lay.stride_head * 2;
  bf16x8 qf[8];
  {
    const int g = lane & 31;
    const char* qp = Q + (static_cast<long long>(h) * G + g) * kD * 2 + hf * 16;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      uint4 w = make_uint4(0u, 0u, 0u, 0u);
      if (g < G) w = *reinterpret_cast<const uint4*>(qp + ks * 32);
      qf[ks] = *reinterpret_cast<bf16x8*>(&w);
    }
  }
  // Wave w takes the 32-token tiles w, w+NW, ...: the rows go straight into the registers in the
  // MFMA operand layout (lane l: token l % 32, eight consecutive k at 8 * (l / 32) per step; the
  // two halves of a row are 32 contiguous bytes per request), the next tile is in flight while
  // the current one is multiplied, and no wave waits for another until the softmax.
  const int ntiles = (n + 31) >> 5;
  const long long tok_bytes = lay.stride_tok * 2;
  bf16x8 kf[8], kn[8];
  auto fetch = [&](int t, bf16x8 (&dst)[8]) {
    const char* p = Kh + min(t * 32 + (lane & 31), n - 1) * tok_bytes + hf * 16;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint4 w = *reinterpret_cast<const uint4*>(p + ks * 32);
      dst[ks] = *reinterpret_cast<const bf16x8*>(&w);
    }
  };
  const float scale = 0.08838834764831845f;
  float zm[GQ / 2];                                   // maxima of this lane's logits (a tile past the head's end repeats its last token)
#pragma unroll
  for (int r = 0; r < GQ / 2; ++r) zm[r] = -INFINITY;
  if (wave < ntiles) fetch(wave, kf);
  for (int t = wave; t < ntiles; t += NW) {
    if (t + NW < ntiles) fetch(t + NW, kn);
    f32x16 acc = {0};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], kf[ks], acc, 0, 0, 0);
    const int j = t * 32 + (lane & 31);
    // lane (token, hf) holds query rows (r/4)*8 + hf*4 + r%4 of the 32x32 tile
#pragma unroll
    for (int r = 0; r < GQ / 2; ++r) {
      const float z = acc[r] * scale;
      zm[r] = hw_max(zm[r], z);
      const int g = (r >> 2) * 8 + hf * 4 + (r & 3);
      if (g < G && j < n) zbuf[g * n + j] = z;
    }
    if (t + NW < ntiles) {
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) kf[ks] = kn[ks];
    }
  }
  // softmax over the tokens for each query, then the mean over queries
#pragma unroll
  for (int r = 0; r < GQ / 2; ++r) {
    const float v = half_max_at_31(zm[r]);
    if ((lane & 31) == 31) red[wave * GQ + (r >> 2) * 8 + hf * 4 + (r & 3)] = v;
  }
  float zmax[GQ], zsum[GQ];
#pragma unroll
  for (int g = 0; g < GQ; ++g) zsum[g] = 0.f;
  __syncthreads();
#pragma unroll
  for (int g = 0; g < GQ; ++g) {
    float v = red[g];
#pragma unroll
    for (int u = 1; u < NW; ++u) v = fmaxf(v, red[u * GQ + g]);
    zmax[g] = v;
  }
  for (int j = tid; j < n; j += 64 * NW)
#pragma unroll
    for (int g = 0; g < GQ; ++g)
      if (g < G) {
        const float e = __expf(zbuf[g * n + j] - zmax[g]);
        zbuf[g * n + j] = e;
        zsum[g] += e;
      }
#pragma unroll
  for (int g = 0; g < GQ; ++g) {
    const float v = butterfly_sum(zsum[g]);
    if (lane == 0) red[(NW + wave) * GQ + g] = v;
  }
  __syncthreads();
  const float invG = 1.0f / static_cast<float>(G);
  float wgt[GQ];
#pragma unroll
  for (int g = 0; g < GQ; ++g) {
    float v = red[NW * GQ + g];
#pragma unroll
    for (int u = 1; u < NW; ++u) v += red[(NW + u) * GQ + g];
    wgt[g] = invG / v;
  }
  finish([&](int j) -> float {
    float p = 0.f;
#pragma unroll
    for (int g = 0; g < GQ; ++g)
      if (g < G) p = fmaf(zbuf[g * n + j], wgt[g], p);
    return p;
  });
}

// Waves per SIMD asked for: what the registers allow anyway (124 and 149), told to the compiler, which then spends all of them on the
// tile in flight; against no bound: 7168 heads of 300 tokens, 7 queries, 104.0 -> 101.1 us, of 1024 332.7 -> 331.0, 1024 of 900
// with 32 queries 101.7 -> 100.8; 2048 of 4096 and 112 of 1024 or 4000 tokens do not change.
template <int GQ, int NW>
__global__ __launch_bounds__(64 * NW, GQ == 8 ? 4 : 3) void score_mfma_kernel(const char* __restrict__ K,
                                                                   const char* __restrict__ Q, int G,
                                                                   Layout lay,
                                                                   float* __restrict__ s_out) {
  extern __shared__ __align__(16) char smem_raw[];
  float* so = s_out + static_cast<long long>(blockIdx.x) * lay.n;
  score_head<GQ, NW>(K, Q, G, lay, smem_raw, [&](auto score_at) {
    for (int j = threadIdx.x; j < lay.n; j += 64 * NW) so[j] = score_at(j);
  });
}

// The whole lambda = 0 event: scores, top-b, kept rows.  The search and the copies of one workgroup run beside the streams of K of
// the others on its CU; as a kernel of its own (select_topb_kernel) the 7168 heads of a call search and copy at the same
// time, at 4 TB/s: 7168 heads of 1024 tokens, b = 64, 476 us in two launches, 443 in one; of 300, b = 17, 178 and 147.  (Four
// workgroups per CU instead of three are better up to 512 tokens only: 156 -> 147 us at 300, 443 -> 450 at 1024.)
template <int S>
__global__ __launch_bounds__(kTopbThreads, S <= 2 ? 4 : 1) void score_topb_kernel(const char* __restrict__ K, const char* __restrict__ Q, int G,
                                                                  Layout lay, float* __restrict__ s_out, TopbArgs a) {
  extern __shared__ __align__(16) char smem_raw[];
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* so = s_out + static_cast<long long>(h) * lay.n;
  uint32_t key[S];
  score_head<8, kTopbThreads / 64>(K, Q, G, lay, smem_raw, [&](auto score_at) {
#pragma unroll
    for (int k = 0; k < S; ++k) {
      const int j = k * kTopbThreads + tid;
      key[k] = 0u;
      if (j < lay.n) {
        const float p = score_at(j);
        so[j] = p;
        key[k] = ordered_key(p + 0.0f);
      }
    }
  });
  lds_barrier();                                      // the logits are dead: the tables of the selection take their place
  topb_finish<S>(a, reinterpret_cast<int32_t*>(smem_raw), key, h, tid, lane, w);
}

// LDS of a four-wave scorer with its logits; where it leaves room for three workgroups per CU or more, four waves score a head
static int score_smem_four(const Layout& lay, int G) { return (G * lay.n + 2 * 4 * 8) * 4; }

bool score_topb_supported(const Layout& lay, int b, float lambda, int G) {
  return topb_supported(lay, b, lambda) && lay.dtype == DT_BF16 && G <= 8 && lay.n <= 16 * kTopbThreads &&
         3 * score_smem_four(lay, G) <= 160 * 1024;
}

hipError_t launch_score_topb(const void* K, const void* V, const void* Q, int G, const Layout& lay, int b, float* s_out,
                             int32_t* idx_sorted, int32_t* pick_order, float* pick_gain, void* K_out, void* V_out,
                             hipStream_t st) {
  TopbArgs a;
  a.b_h = nullptr;
  a.K = static_cast<const char*>(K); a.V = static_cast<const char*>(V); a.s_in = nullptr;
  a.idx_sorted = idx_sorted; a.pick_order = pick_order; a.pick_gain = pick_gain;
  a.K_out = static_cast<char*>(K_out); a.V_out = static_cast<char*>(V_out);
  a.stride_head = lay.stride_head; a.stride_tok = lay.stride_tok;
  a.n = lay.n; a.b = b;
  auto go = [&](auto kern, int slots) -> hipError_t {
    const int s1 = score_smem_four(lay, G), s2 = topb_smem_bytes(slots, b), smem = s1 > s2 ? s1 : s2;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(lay.heads), dim3(kTopbThreads), smem, st, static_cast<const char*>(K),
                       static_cast<const char*>(Q), G, lay, s_out, a);
    return hipGetLastError();
  };
  if (lay.n <= 2 * kTopbThreads) return go(&score_topb_kernel<2>, 2);
  if (lay.n <= 4 * kTopbThreads) return go(&score_topb_kernel<4>, 4);
  if (lay.n <= 8 * kTopbThreads) return go(&score_topb_kernel<8>, 8);
  return go(&score_topb_kernel<16>, 16);
}

hipError_t launch_score(const void* K, const void* Q, int G, const Layout& lay, float* s_out,
                        hipStream_t st) {
  // the logits of a head (G x n floats) wait in LDS
  const bool fits = static_cast<long long>(G) * lay.n <= (G <= 8 ? 24576 : 31488);
  // Logits that fill a CU's LDS: one workgroup of sixteen waves per CU still reads K once where score_wide_kernel reads it twice.
  // Few heads leave CUs idle here, while the other kernel splits a head over several (hence the two heads to five CUs).  Two passes / one, us, 4 queries: 256 heads of 8192
  // tokens 196 / 101, 448 354 / 180, 128 86 / 68, 112 75 / 67, 96 65 / 67, 32 32 / 67; 256 of 5500 with 7 queries 136 / 72.  (Scores' error against 64
  // bits, 2-norm, 256 heads of 8192: 3.6e-7 / 1.3e-7.)
  // The line at 4096 tokens is not one of speed: shorter heads whose logits fill the LDS (7 queries from 3513 tokens on, 8 from 3073) would gain as
  // well, 256 heads of 4096 with 7 queries 78 / 48, 112 44.0 / 39.7, 256 of 3300 with 8 62 / 43, 64 of 4096 30.9 / 31.0.  Their scores keep the bits that two passes give.
  const bool whole_cu = !fits && lay.n > 4096 && G <= 8 && (G * lay.n + 2 * 16 * 8) * 4 <= 160 * 1024 && 5 * lay.heads > 2 * cu_count();
  if (lay.dtype == DT_BF16 && G <= 32 && (fits || whole_cu)) {
    const int gq = G <= 8 ? 8 : 32;
    // The logit buffer sets how many workgroups share a CU; when it leaves room for two or fewer, eight waves per
    // workgroup keep as many rows in flight as four waves do with a small buffer.
    const int smem_one = (G * lay.n + 8 * gq) * 4;
    const bool big = 3 * smem_one > 160 * 1024;
    const int nw = whole_cu ? 16 : (big ? 8 : 4);
    const int smem_m = (G * lay.n + 2 * nw * gq) * 4;
    auto go_m = [&](auto kern) -> hipError_t {
      const hipError_t em = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, smem_m);
      if (em != hipSuccess) return em;
      hipLaunchKernelGGL(kern, dim3(lay.heads), dim3(64 * nw), smem_m, st,
                         static_cast<const char*>(K), static_cast<const char*>(Q), G, lay, s_out);
      return hipGetLastError();
    };
    if (whole_cu) return go_m(&score_mfma_kernel<8, 16>);
    if (big) return gq == 8 ? go_m(&score_mfma_kernel<8, 8>) : go_m(&score_mfma_kernel<32, 8>);
    return gq == 8 ? go_m(&score_mfma_kernel<8, 4>) : go_m(&score_mfma_kernel<32, 4>);
  }
  if (score_wide_supported(lay, G)) return launch_score_wide(K, Q, G, lay, s_out, st);
  const bool zfits = static_cast<long long>(G) * lay.n <= kZMaxFloats;
  const size_t smem = (static_cast<size_t>(zfits ? G * lay.n : 0) + lay.n + 2 * kGT * 4) * 4;
  dim3 grid(lay.heads), block(kScoreThreads);
  auto go = [&](auto kern) -> hipError_t {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             static_cast<int>(smem));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, smem, st, K, Q, G, lay, s_out);
    return hipSuccess;
  };
  hipError_t e;
  if (lay.dtype == DT_BF16) e = zfits ? go(&score_kernel<DT_BF16, true>) : go(&score_kernel<DT_BF16, false>);
  else e = zfits ? go(&score_kernel<DT_F32, true>) : go(&score_kernel<DT_F32, false>);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace kvr
