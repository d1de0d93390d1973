// The whole retention event (paper Sec. 4.1: scores -> Eq. 1 signatures -> Algorithm 1 ->
// kept rows) for bf16 heads of 128 < n <= 256 tokens when the call has so few heads that every
// workgroup gets a CU to itself (a decode-time event of one sequence: layers x KV heads <= CUs).
// Throughput is then the latency of one head, so the parallel phases -- rows, logits, Gram,
// cosine triangle, outputs -- are spread over sixteen wave64s instead of four; the b dependent
// picks stay on one wave.  Same arithmetic and same helpers as
// retain_dense_kernel, which remains the kernel for batched calls (several heads per CU).
//
// What is not the chain is a row of latencies, so it is cut where it can be.  Both tensors and the queries are requested at once and staged
// side by side (the triangle takes their place).  Waves 0-3 work out the scores while waves 4-15 run the Gram, two row blocks
// by two column blocks each, so that an operand read from LDS meets two others (one tile at a time the Gram was bound by its LDS
// reads); the second half of the softmax runs beside the writing of the triangle.  The triangle is the packed one: in padded rows
// (16-byte stores) it is written as fast, but a pick reads its columns with bank conflicts (24 cycles of 302).
// 112 heads, n = 256, b = 128, cycles of a head: rows in LDS 4 500, Gram until 8 400, triangle until 12 900, picks until 51 600,
// outputs until 57 500.  Before, with K staged first, then the scores, V and the Gram: chain from 20 200 on, 65 300 in all; the call 29.4 -> 26.5 us,
// n = 192, b = 64 17.8 -> 15.7.
#include "kvr_dense_common.hpp"
#include "kvr_kernels.hpp"

namespace kvr {

constexpr int kD16Threads = 1024;
constexpr int kD16Waves = kD16Threads / 64;
constexpr int kD16MaxB = 256;

constexpr int kD16MaxG = 8;

// staged rows of V, then of K; the triangle takes their place | s_l[N32] | rinv[N32] | max [8 queries][4], sum [8][8] |
// queries [8][272 B] | met [4] | idx_l | order_l | gain_l
__host__ __device__ constexpr int dense16_area(int NT) {
  const int rows = 2 * NT * 32 * kRowPitch, tri = dense_tri_floats(NT) * 4;
  return rows > tri ? rows : tri;
}
__host__ __device__ constexpr int dense16_smem_bytes(int NT) {
  return dense16_area(NT) + NT * 32 * 4 * 2 + 2 * kD16MaxG * 8 * 4 + kD16MaxG * kRowPitch + 16 + kD16MaxB * 4 * 3;
}

struct Dense16Args {
  const char* K; const char* V; const char* Q; const float* s_in;
  float* s_out; int32_t* idx_sorted; int32_t* pick_order; float* pick_gain;
  char* K_out; char* V_out;
  long long stride_head, stride_tok;   // elements
  int n, b, G;
  float lambda, eps;
  const int32_t* b_h;                  // per-head budgets <= b (rows of the outputs stay b apart), or null
};

template <int NT>
__global__ __launch_bounds__(kD16Threads, 1) void retain_dense16_kernel(Dense16Args a) {
  constexpr int N32 = NT * 32;
  constexpr int NQ = NT / 2;
  constexpr int UNITS = NT / 2 * (NT / 2 + 1) / 2;    // pairs of row blocks by pairs of column blocks in the lower triangle
  constexpr int kIters = N32 * 16 / kD16Threads;      // 16-byte pieces of the head's rows per thread
  static_assert(NT % 2 == 0 && NT >= 4 && UNITS <= kD16Waves - 4, "a wave per unit");
  extern __shared__ __align__(16) char smem[];
  char* stage = smem;                                // staged rows of V ...
  char* stage_k = smem + N32 * kRowPitch;            // ... and of K
  float* tri = reinterpret_cast<float*>(smem);       // ... later the cosine triangle
  float* s_l = reinterpret_cast<float*>(smem + dense16_area(NT));
  float* rinv = s_l + N32;
  float* red = rinv + N32;                           // maxima [8 queries][4 waves], sums [8 queries][8 blocks]
  char* stage_q = reinterpret_cast<char*>(red + 2 * kD16MaxG * 8);
  int32_t* met = reinterpret_cast<int32_t*>(stage_q + kD16MaxG * kRowPitch);   // [4] waves that have their maxima
  int32_t* idx_l = met + 4;
  int32_t* order_l = idx_l + kD16MaxB;
  float* gain_l = reinterpret_cast<float*>(order_l + kD16MaxB);

  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x;
  const int n = a.n, b = a.b;
  const int bh = a.b_h ? min(max(a.b_h[h], 0), b) : b;  // the head's own budget
  const bool diverse = a.lambda != 0.0f;
  const bool need_v = diverse && b > 1;
  const long long head_off = h * a.stride_head * 2;   // bytes
  const int chunk = tid & 15, r0 = tid >> 4;          // 64 rows per step of the row loops

  // everything starts its trip from memory at once; rows past n are the last one again (never picked).  (Vector types, not the
  // struct uint4: the arrays of those ended up in scratch memory)
  {
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    const long long tok_bytes = a.stride_tok * 2, off = head_off + chunk * 16;
    u32x4 kreg[kIters], vreg[kIters], q = {0u, 0u, 0u, 0u};
    if (tid < 4) met[tid] = 0;
    if (a.Q) {
#pragma unroll
      for (int k = 0; k < kIters; ++k) kreg[k] = *reinterpret_cast<const u32x4*>(a.K + off + min(r0 + 64 * k, n - 1) * tok_bytes);
      // (rows past G are the last query again; their results are not used)
      if (wave < 2) q = *reinterpret_cast<const u32x4*>(a.Q + (static_cast<long long>(h) * a.G + min(r0, a.G - 1)) * kD * 2 + chunk * 16);
    }
    if (need_v) {
#pragma unroll
      for (int k = 0; k < kIters; ++k) vreg[k] = *reinterpret_cast<const u32x4*>(a.V + off + min(r0 + 64 * k, n - 1) * tok_bytes);
    }
    if (a.Q) {
#pragma unroll
      for (int k = 0; k < kIters; ++k) *reinterpret_cast<u32x4*>(stage_k + (r0 + 64 * k) * kRowPitch + chunk * 16) = kreg[k];
      if (wave < 2) *reinterpret_cast<u32x4*>(stage_q + r0 * kRowPitch + chunk * 16) = q;
    } else if (tid < N32) {
      s_l[tid] = tid < n ? a.s_in[static_cast<long long>(h) * n + tid] : -INFINITY;
    }
    if (need_v) {
#pragma unroll
      for (int k = 0; k < kIters; ++k) *reinterpret_cast<u32x4*>(stage + (r0 + 64 * k) * kRowPitch + chunk * 16) = vreg[k];
    }
  }
  lds_barrier();

  if (wave >= 4) {
    // ------------------------------------------------ Gram -> packed cosines: waves 4-15, a pair of row blocks by a pair of column blocks each
    if (need_v && wave - 4 < UNITS) {
      int P = wave - 4, Q = P;                        // the pairs on the diagonal first (two diagonal tiles and the one between them)
      if (P >= NT / 2) {
        const int o = P - NT / 2;
        P = 1;
        while (P * (P + 1) / 2 <= o) ++P;
        Q = o - P * (P - 1) / 2;
      }
      // Four operands from LDS make four tiles.  (One tile at a time the Gram was bound by the LDS: 16 reads a tile.)
      f32x16 t00 = {0}, t01 = {0}, t10 = {0}, t11 = {0};   // tile (2P + first, 2Q + second)
      if (P == Q) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          const bf16x8 i0 = frag_at(stage, 2 * P, ks, lane), i1 = frag_at(stage, 2 * P + 1, ks, lane);
          t00 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(i0, i0, t00, 0, 0, 0);
          t11 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(i1, i1, t11, 0, 0, 0);
          t10 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(i0, i1, t10, 0, 0, 0);
        }
        // squared norms: element r of lane (l32, hf) is column 8 (r / 4) + 4 hf + r % 4 of the tile, so row l32's own sits in one of its two lanes
        auto norms = [&](const f32x16& t, int block) {
          auto pick = [](int bit, float one, float zero) { return bit ? one : zero; };
          float v8[8], v4[4];
#pragma unroll
          for (int k = 0; k < 8; ++k) v8[k] = pick(l32 & 1, t[2 * k + 1], t[2 * k]);
#pragma unroll
          for (int k = 0; k < 4; ++k) v4[k] = pick(l32 & 2, v8[2 * k + 1], v8[2 * k]);
          const float ss = pick(l32 & 16, pick(l32 & 8, v4[3], v4[2]), pick(l32 & 8, v4[1], v4[0]));
          if (((l32 >> 2) & 1) == hf) rinv[block * 32 + l32] = 1.0f / (sqrtf(ss) + a.eps);
        };
        norms(t00, 2 * P);
        norms(t11, 2 * P + 1);
      } else {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          const bf16x8 i0 = frag_at(stage, 2 * P, ks, lane), i1 = frag_at(stage, 2 * P + 1, ks, lane);
          const bf16x8 j0 = frag_at(stage, 2 * Q, ks, lane), j1 = frag_at(stage, 2 * Q + 1, ks, lane);
          t00 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(j0, i0, t00, 0, 0, 0);
          t01 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(j1, i0, t01, 0, 0, 0);
          t10 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(j0, i1, t10, 0, 0, 0);
          t11 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(j1, i1, t11, 0, 0, 0);
        }
      }
      lds_barrier();                                  // staged rows are dead from here on, the norms complete
      if constexpr (NT > 6) {                         // (26.5 -> 25.8 us; with six blocks, three units fewer, 15.7 -> 16.3)
        scale_cos_tile(rinv, t00, 2 * P, 2 * Q, lane);
        scale_cos_tile(rinv, t10, 2 * P + 1, 2 * Q, lane);
        scale_cos_tile(rinv, t11, 2 * P + 1, 2 * Q + 1, lane);
        if (P != Q) scale_cos_tile(rinv, t01, 2 * P, 2 * Q + 1, lane);
        store_cos_tile(tri, t00, 2 * P, 2 * Q, lane);
        store_cos_tile(tri, t10, 2 * P + 1, 2 * Q, lane);
        store_cos_tile(tri, t11, 2 * P + 1, 2 * Q + 1, lane);
        if (P != Q) store_cos_tile(tri, t01, 2 * P, 2 * Q + 1, lane);
      } else {
        write_cos_tile_rows(tri, rinv, t00, 2 * P, 2 * Q, lane);
        write_cos_tile_rows(tri, rinv, t10, 2 * P + 1, 2 * Q, lane);
        write_cos_tile_rows(tri, rinv, t11, 2 * P + 1, 2 * Q + 1, lane);
        if (P != Q) write_cos_tile_rows(tri, rinv, t01, 2 * P, 2 * Q + 1, lane);
      }
    } else {
      lds_barrier();
    }
  } else {
    // ---------------------------------------------------------------- scores: wave w takes the token blocks w and w + 4
    if (a.Q) {
      __builtin_amdgcn_s_setprio(2);                  // (ahead of the tiles of the waves on the same SIMD)
      const float scale = 0.08838834764831845f;      // 1/sqrt(128)
      float z[2][4];                                  // lane (token, hf): the logits of queries hf*4 .. hf*4+3
      {
        f32x16 d0 = {0}, d1 = {0};
        const int second = wave + 4 < NT ? wave + 4 : wave;   // (no second block: the first again, its logits are -inf)
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          const bf16x8 q = *reinterpret_cast<const bf16x8*>(stage_q + min(l32, kD16MaxG - 1) * kRowPitch + ks * 32 + hf * 16);
          d0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q, frag_at(stage_k, wave, ks, lane), d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q, frag_at(stage_k, second, ks, lane), d1, 0, 0, 0);
        }
        const bool live0 = wave * 32 + l32 < n, live1 = wave + 4 < NT && wave * 32 + 128 + l32 < n;
#pragma unroll
        for (int r = 0; r < 4; ++r) { z[0][r] = live0 ? d0[r] * scale : -INFINITY; z[1][r] = live1 ? d1[r] * scale : -INFINITY; }
      }
      {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = hw_max(z[0][r], z[1][r]);
        half_maxes_at_31(v);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (l32 == 31) red[(hf * 4 + r) * 4 + wave] = v[r];
      }
      // This exchange is among the four waves only (a barrier would wait for the tiles of the others): each adds itself to a counter and
      // waits until all four have.  (None of them waits for anything in between.)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (lane == 0) __hip_atomic_fetch_add(met, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      while (__hip_atomic_load(met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < 4) {}
      asm volatile("" ::: "memory");
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float4 x = *reinterpret_cast<const float4*>(red + (hf * 4 + r) * 4);
        const float zmax = fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w));
        z[0][r] = __expf(z[0][r] - zmax);             // exp(-inf) = 0 for padded tokens
        z[1][r] = __expf(z[1][r] - zmax);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float v[4] = {z[u][0], z[u][1], z[u][2], z[u][3]};
        half_sums_at_31(v);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (l32 == 31) red[kD16MaxG * 4 + (hf * 4 + r) * 8 + wave + 4 * u] = v[r];
      }
      __builtin_amdgcn_s_setprio(0);
      lds_barrier();                                  // the sums are there; staged rows are dead
      const float invG = 1.0f / static_cast<float>(a.G);
      float p[2] = {0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* rs = red + kD16MaxG * 4 + (hf * 4 + r) * 8;
        const float4 x = *reinterpret_cast<const float4*>(rs), y = *reinterpret_cast<const float4*>(rs + 4);
        const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
        float tot = 0.f;                              // (the blocks' sums in their order)
#pragma unroll
        for (int u = 0; u < NT; ++u) tot += v[u];
        const float wt = hf * 4 + r < a.G ? invG / tot : 0.f;
        p[0] = fmaf(z[0][r], wt, p[0]);
        p[1] = fmaf(z[1][r], wt, p[1]);
      }
      p[0] += __shfl_xor(p[0], 32, kWave);           // queries 0-3 live in lanes 0-31, 4-7 in 32-63
      p[1] += __shfl_xor(p[1], 32, kWave);
      const int j = wave * 32 + l32 + 128 * hf;       // lane (token, hf) stores the token of block wave + 4 hf
      const float pj = hf ? p[1] : p[0];
      if (j < N32) {
        s_l[j] = j < n ? pj : -INFINITY;              // padding never competes
        if (j < n && a.s_out) a.s_out[static_cast<long long>(h) * n + j] = pj;
      }
    }
    if (!a.Q) lds_barrier();
  }
  lds_barrier();

  // ---------------------------------------------------------------- greedy
  if (wave == 0) {
    const int brun = bh < 1 ? 1 : bh;
    pick_chain<NQ>(s_l, tri, order_l, gain_l, n, brun, a.lambda, diverse, lane);
    sort_picks<NQ>(order_l, idx_l, reinterpret_cast<int32_t*>(rinv), brun, lane, nullptr);   // rinv is dead by now
  }
  lds_barrier();

  // ------------------------------------------------- outputs and compaction
  const long long ob = static_cast<long long>(h) * b;
  for (int t = tid; t < b; t += kD16Threads) {                   // entries past the head's budget are padding
    a.idx_sorted[ob + t] = t < bh ? idx_l[t] : -1;
    if (a.pick_order) a.pick_order[ob + t] = t < bh ? order_l[t] : -1;
    if (a.pick_gain) a.pick_gain[ob + t] = t < bh ? gain_l[t] : -INFINITY;
  }
  if ((a.K_out || a.V_out) && bh > 0)
    compact_rows<4>(a.K, a.V, a.K_out, a.V_out, head_off, a.stride_tok, idx_l, n, bh, ob, tid, kD16Threads);
}

bool dense16_supported(const Layout& lay, int b, int G, bool has_q, int cus) {
  return lay.dtype == DT_BF16 && lay.n > 128 && lay.n <= 256 && b <= kD16MaxB && (!has_q || G <= 8) &&
         lay.heads <= cus;
}

hipError_t launch_retain_dense16(const void* K, const void* V, const void* Q, int G, const float* s_in,
                                 const Layout& lay, int b, float lambda, float eps, float* s_out,
                                 int32_t* idx_sorted, int32_t* pick_order, float* pick_gain, void* K_out,
                                 void* V_out, hipStream_t st, const int32_t* b_h) {
  Dense16Args a;
  a.K = static_cast<const char*>(K); a.V = static_cast<const char*>(V);
  a.Q = static_cast<const char*>(Q); a.s_in = s_in; a.s_out = s_out;
  a.idx_sorted = idx_sorted; a.pick_order = pick_order; a.pick_gain = pick_gain;
  a.K_out = static_cast<char*>(K_out); a.V_out = static_cast<char*>(V_out);
  a.stride_head = lay.stride_head; a.stride_tok = lay.stride_tok;
  a.n = lay.n; a.b = b; a.G = G; a.lambda = lambda; a.eps = eps; a.b_h = b_h;
  auto go = [&](auto kern, int smem) -> hipError_t {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(lay.heads), dim3(kD16Threads), smem, st, a);
    return hipGetLastError();
  };
  if (lay.n <= 192) return go(&retain_dense16_kernel<6>, dense16_smem_bytes(6));
  return go(&retain_dense16_kernel<8>, dense16_smem_bytes(8));
}

}  // namespace kvr
