// Algorithm 1 (paper Sec. 4.1, Eq. 1-3) for heads of n <= 256 tokens whose rows are fp32: the
// flat-signature mode, whose signature rows are means over layers and heads and so are not
// bf16 numbers, and fp32 caches.  One workgroup of sixteen wave64s per head (such launches have
// few heads, so the latency of one head is what counts):
//
//   rows     staged in LDS as fp32, 132-float pitch (16-byte aligned rows; sixteen consecutive rows
//            cover the banks with their 16-byte pieces)
//   Gram     lower-triangular 16x16 tiles on the fp32 MFMA (16x16x4, fp32 products and sums, one after the other in the order of
//            the lanes' four k-groups).  The sums run over k = 0, 64, 1, 65, ..: MFMA t takes k = 2t, 64 + 2t, 2t + 1, 65 + 2t,
//            and the rows are staged in the order [k / 64][k % 2][k % 64 / 2], so that a lane reads 32 consecutive floats of
//            its row.  (32x32x2 MFMAs give the same bits at the same rate, but their tiles hold more of the upper triangle
//            and 21 of them do not divide by four SIMDs: n = 192, 24 600 cycles at best, 20 000 now.  One head, n = 192, b = 64
//            27.9 -> 25.2 us with the triangle's stores from one base address and the score bound's search only where it can
//            drop a token; 32 heads of 130, b = 40 25.1 -> 22.3; n = 256, b = 128 44.6 -> 43.7)
//   norms    r_j = 1/(||V_j|| + eps) from the Gram diagonal              (Eq. 1)
//   cosines  packed fp32 triangle in the space the rows were staged in   (Algorithm 1, Sims)
//   greedy   the single-wave pick loop of the bf16 kernels                (Eq. 2-3)
//
// With Q the kernel also computes the base scores (up to 16 queries), and with K_out / V_out it
// copies the kept rows: a single fp32 head is then one launch instead of three.
#include "kvr_dense_common.hpp"
#include "kvr_kernels.hpp"

namespace kvr {

constexpr int kF32Pitch = 132;                 // floats per staged row
constexpr int kF32MaxB = 256;
constexpr int kF32Threads = 1024;
constexpr int kF32Waves = kF32Threads / 64;

__host__ __device__ constexpr int f32_region_a(int NT) {
  const int tri = dense_tri_floats(NT) * 4, stage = NT * 32 * kF32Pitch * 4;
  return ((tri > stage ? tri : stage) + 15) & ~15;
}
__host__ __device__ constexpr int f32_smem_bytes(int NT) {
  // region A | s_l[N32] | rinv[N32] | idx_l | order_l | gain_l | tok_c[N32] | meta[4]
  return f32_region_a(NT) + NT * 32 * 4 * 2 + kF32MaxB * 4 * 3 + NT * 32 * 4 + 16;
}

struct F32Args {
  const float* V; const float* s;
  int32_t* idx_sorted; int32_t* pick_order; float* pick_gain;
  long long stride_head, stride_tok;   // elements
  int n, b;
  float lambda, eps;
  // optional: the scores are computed here from K and Q (then `s` is unused and s_out receives them),
  // and the kept rows are written here
  const float* K; const float* Q; int G; float* s_out;
  float* K_out; float* V_out;
};

template <int NT>
__global__ __launch_bounds__(kF32Threads, 1) void select_dense_f32_kernel(F32Args a) {
  constexpr int N32 = NT * 32;
  constexpr int NQ = NT / 2;
  constexpr int NTILES = NT * (2 * NT + 1);           // 16x16 tiles of the lower triangle
  constexpr int MAXT = (NTILES + kF32Waves - 1) / kF32Waves;
  extern __shared__ __align__(16) char smem[];
  float* stage = reinterpret_cast<float*>(smem);
  float* tri = reinterpret_cast<float*>(smem);
  float* s_l = reinterpret_cast<float*>(smem + f32_region_a(NT));
  float* rinv = s_l + N32;
  int32_t* idx_l = reinterpret_cast<int32_t*>(rinv + N32);
  int32_t* order_l = idx_l + kF32MaxB;
  float* gain_l = reinterpret_cast<float*>(order_l + kF32MaxB);
  int32_t* tok_c = reinterpret_cast<int32_t*>(gain_l + kF32MaxB);     // [N32] tokens of the reduced problem
  int32_t* meta = tok_c + N32;                                         // [0] its size, 0 = not reduced

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x;
  const int n = a.n, b = a.b;
  const bool diverse = a.lambda != 0.0f && b > 1;

  // The rows start their trip from memory before anything else, those of V behind those of K and the first query: 32 threads per
  // row (float4 each), rows past n read as zero.  (One head, n = 192, b = 64: 29.0 us with V requested after the scores and
  // their sums exchanged through LDS, 27.8 now.)
  float4 kr[NT], xr[NT], q0 = make_float4(0.f, 0.f, 0.f, 0.f);
  const float* Qh = a.Q + static_cast<long long>(h) * a.G * kD + (tid & 31) * 4;
  if (a.Q) {
    q0 = *reinterpret_cast<const float4*>(Qh);
    const float* Kh = a.K + h * a.stride_head;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int r = (tid >> 5) + 32 * k;
      kr[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (r < n) kr[k] = *reinterpret_cast<const float4*>(Kh + r * a.stride_tok + (tid & 31) * 4);
    }
  }
  if (diverse) {
    const float* Vh = a.V + h * a.stride_head;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int r = (tid >> 5) + 32 * k;
      xr[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (r < n) xr[k] = *reinterpret_cast<const float4*>(Vh + r * a.stride_tok + (tid & 31) * 4);
    }
  }
  if (a.Q) {
    // Base scores (the stand-in for the paper's external scorer): s_i = (1/G) sum_g softmax_i(q_g . k_i / sqrt(d)).
    // 32 threads per row (float4 each) take the dot products in fp32, one wave per query takes its softmax.
    float* zl = stage;                                 // [G][N32] logits, then probabilities (the stage is free until the rows arrive)
    const float scale = 0.08838834764831845f;          // 1/sqrt(128)
    for (int g = 0; g < a.G; ++g) {
      const float4 qv = q0;
      if (g + 1 < a.G) q0 = *reinterpret_cast<const float4*>(Qh + (g + 1) * kD);
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        const float p = half_butterfly_sum(fmaf(kr[k].x, qv.x, fmaf(kr[k].y, qv.y, fmaf(kr[k].z, qv.z, kr[k].w * qv.w))));
        const int r = (tid >> 5) + 32 * k;
        if ((tid & 31) == 0) zl[g * N32 + r] = r < n ? p * scale : -INFINITY;
      }
    }
    __syncthreads();
    if (wave < a.G) {
      float v[NQ];
      float mx = -INFINITY;
#pragma unroll
      for (int q = 0; q < NQ; ++q) { v[q] = zl[wave * N32 + lane + 64 * q]; mx = fmaxf(mx, v[q]); }
      mx = wave_max_uniform(mx);
      float sum = 0.f;
#pragma unroll
      for (int q = 0; q < NQ; ++q) { v[q] = __expf(v[q] - mx); sum += v[q]; }   // exp(-inf) = 0 for padding
      sum = butterfly_sum(sum);
      const float inv = 1.0f / sum;
#pragma unroll
      for (int q = 0; q < NQ; ++q) zl[wave * N32 + lane + 64 * q] = v[q] * inv;
    }
    __syncthreads();
    if (tid < N32) {
      float p = 0.f;
      for (int g = 0; g < a.G; ++g) p += zl[g * N32 + tid];
      p /= static_cast<float>(a.G);
      s_l[tid] = tid < n ? p : -INFINITY;                // padding never competes
      if (tid < n && a.s_out) a.s_out[static_cast<long long>(h) * n + tid] = p;
    }
    __syncthreads();                                     // the stage is free again
  } else {
    if (tid < N32) s_l[tid] = tid < n ? a.s[static_cast<long long>(h) * n + tid] : -INFINITY;
  }
  if (tid == 0) meta[0] = 0;
  f32x4 acc[MAXT];
  int ns = 0;                                       // size of the reduced problem, 0 = all n tokens
  if (diverse) {
    // Exact candidate reduction for heads of more than 128 tokens: a token with s_j < s_(b) - lambda
    // never wins Eq. 3 (while fewer than b tokens are selected one of the b best-scored is free and
    // gains at least s_(b) - lambda; the token itself gains at most s_j).  When at most 128 tokens
    // remain, the head shrinks to them: fewer Gram tiles, two tokens per lane in the pick loop.
    // The survivors keep their order, so ties break as before.
    if constexpr (NT > 4) {
      __syncthreads();
      if (wave == 0) {
        float sv[NQ];
        uint32_t key[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          sv[q] = s_l[lane + 64 * q];
          key[q] = lane + 64 * q < n ? ordered_key(sv[q] + 0.0f) : 0u;
        }
        // (nothing can go when the finite scores spread by no more than lambda: softmax means always do)
        float hi = -INFINITY, lo = INFINITY;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          if (sv[q] > -INFINITY && sv[q] < INFINITY) { hi = hw_max(hi, sv[q]); lo = fminf(lo, sv[q]); }
        hi = wave_max_uniform(hi);
        lo = -wave_max_uniform(-lo);
        const bool wide = __builtin_amdgcn_readfirstlane(hi - lo > a.lambda ? 1 : 0) != 0;   // false also when no score is finite
        // s_(b) from the leading 16 bits of the ordered keys: at most s_(b), so the bound only loosens
        uint32_t T = 0;
        for (int bit = 31; wide && bit >= 16; --bit) {
          const uint32_t cand = T | (1u << bit);
          const int cnt = count_slots_ge<NQ>(key, cand);
          if (cnt >= b) T = cand;
        }
        const float sb = key_to_float(T);
        const float thr = sb - a.lambda * 1.00001f - 1e-5f * fabsf(sb);   // cosines may exceed 1 by a few ulp
        unsigned long long keep[NQ];
        int cnt = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          keep[q] = __ballot(lane + 64 * q < n && !(sv[q] < thr));
          cnt += __popcll(keep[q]);
        }
        if (wide && cnt >= b && cnt <= 128) {
          wave_lds_sync();                            // every lane holds its scores before s_l is rewritten
          int base = 0;
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            const bool kept = (keep[q] >> lane) & 1ull;
            const int c = base + __popcll(keep[q] & ((1ull << lane) - 1ull));
            if (kept) {
              tok_c[c] = lane + 64 * q;
              s_l[c] = sv[q];
            }
            idx_l[lane + 64 * q] = kept ? c : -1;        // where the token's row goes (idx_l is free until the sort)
            base += __popcll(keep[q]);
          }
          for (int c = cnt + lane; c < 128; c += kWave) s_l[c] = -INFINITY;   // padding never competes
          if (lane == 0) meta[0] = cnt;
        }
      }
      __syncthreads();
      ns = meta[0];
    }
    // rows -> LDS: at their own position, or at their position in the reduced problem
    const int perm = (tid & 31) * 4, at = (perm & 64) + (perm & 63) / 2;   // k = perm .. + 3 go to at, at + 32, at + 1, at + 33
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int r = (tid >> 5) + 32 * k;
      const int dst = ns ? idx_l[r] : r;
      if (dst >= 0) {
        *reinterpret_cast<float2*>(stage + dst * kF32Pitch + at) = make_float2(xr[k].x, xr[k].z);
        *reinterpret_cast<float2*>(stage + dst * kF32Pitch + at + 32) = make_float2(xr[k].y, xr[k].w);
      }
    }
    if (ns)                                           // rows between the survivors and the end of their last block
      for (int r = ns + (tid >> 5); r < ((ns + 15) & ~15); r += kF32Threads / 32)
        *reinterpret_cast<float4*>(stage + r * kF32Pitch + (tid & 31) * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    // the tiles of the lower triangle (row block I, column block J <= I, only the blocks in use), row by row, in sixteen equal shares
    const int nblk = ns ? (ns + 15) >> 4 : 2 * NT;
    const int ntiles = nblk * (nblk + 1) / 2;
    const int c = lane & 15, kg = lane >> 4;
    const int first = wave * ntiles / kF32Waves, count = (wave + 1) * ntiles / kF32Waves - first;
    int I0 = 0;
    while ((I0 + 1) * (I0 + 2) / 2 <= first) ++I0;
    const float* const op = stage + c * kF32Pitch + (kg & 1) * 64 + (kg >> 1) * 32;   // lane (row c, k-group kg) of an operand
    float4 xi[8];
    {
      int I = I0, J = first - I0 * (I0 + 1) / 2, held = -1;
#pragma unroll
      for (int sl = 0; sl < MAXT; ++sl) {
        acc[sl] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (sl < count) {
          if (I != held) {                            // (the row block's operand stays for the tiles of its row)
#pragma unroll
            for (int q = 0; q < 8; ++q) xi[q] = *reinterpret_cast<const float4*>(op + I * 16 * kF32Pitch + 4 * q);
            held = I;
          }
          const float* pj = op + J * 16 * kF32Pitch;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float4 xj = *reinterpret_cast<const float4*>(pj + 4 * q);
            acc[sl] = __builtin_amdgcn_mfma_f32_16x16x4f32(xj.x, xi[q].x, acc[sl], 0, 0, 0);
            acc[sl] = __builtin_amdgcn_mfma_f32_16x16x4f32(xj.y, xi[q].y, acc[sl], 0, 0, 0);
            acc[sl] = __builtin_amdgcn_mfma_f32_16x16x4f32(xj.z, xi[q].z, acc[sl], 0, 0, 0);
            acc[sl] = __builtin_amdgcn_mfma_f32_16x16x4f32(xj.w, xi[q].w, acc[sl], 0, 0, 0);
          }
          // lane (row c of block I, kg) holds columns 4 kg .. + 3 of block J: the squared norm of row c sits in lane (c, c / 4)
          if (I == J && (c >> 2) == kg) {
            auto pick = [](int bit, float one, float zero) { return bit ? one : zero; };   // (by value: a choice between two elements would put the array in memory)
            const float ss = pick(c & 2, pick(c & 1, acc[sl][3], acc[sl][2]), pick(c & 1, acc[sl][1], acc[sl][0]));
            rinv[I * 16 + c] = 1.0f / (sqrtf(ss) + a.eps);
          }
          if (++J > I) { ++I; J = 0; }
        }
      }
    }
    __syncthreads();                                  // staged rows are dead from here on, the norms complete
    {
      int I = I0, J = first - I0 * (I0 + 1) / 2;
#pragma unroll
      for (int sl = 0; sl < MAXT; ++sl) {
        if (sl < count) {
          const int row = I * 16 + c;
          const float rrow = rinv[row];
          const float4 rc = *reinterpret_cast<const float4*>(rinv + J * 16 + 4 * kg);
          const float v[4] = {acc[sl][0] * rrow * rc.x, acc[sl][1] * rrow * rc.y, acc[sl][2] * rrow * rc.z, acc[sl][3] * rrow * rc.w};
          float* dst = tri + row * (row + 1) / 2 + J * 16 + 4 * kg;
          if (I != J) {
#pragma unroll
            for (int q = 0; q < 4; ++q) dst[q] = v[q];
          } else {                                    // (reading the row of a pick retires it)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (4 * kg + q <= c) dst[q] = 4 * kg + q == c ? INFINITY : v[q];
          }
          if (++J > I) { ++I; J = 0; }
        }
      }
    }
  }
  __syncthreads();

  if (wave == 0) {
    if (ns) {                                           // the reduced problem: indices go back through tok_c
      pick_chain<2>(s_l, tri, order_l, gain_l, ns, b, a.lambda, diverse, lane);
      sort_picks<2>(order_l, idx_l, reinterpret_cast<int32_t*>(rinv), b, lane, tok_c);
    } else {
      pick_chain<NQ>(s_l, tri, order_l, gain_l, n, b, a.lambda, diverse, lane);
      sort_picks<NQ>(order_l, idx_l, reinterpret_cast<int32_t*>(rinv), b, lane, nullptr);
    }
  }
  __syncthreads();
  const long long ob = static_cast<long long>(h) * b;
  for (int t = tid; t < b; t += kF32Threads) {
    a.idx_sorted[ob + t] = idx_l[t];
    if (a.pick_order) a.pick_order[ob + t] = order_l[t];
    if (a.pick_gain) a.pick_gain[ob + t] = gain_l[t];
  }
  // kept rows: 32 threads per row, four rows per thread in flight
  if (a.K_out || a.V_out) {
    const int c4 = (tid & 31) * 4;
    for (int t0 = 0; t0 < b; t0 += 128) {
      float4 xk[4], xv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int t = min(t0 + (tid >> 5) + 32 * k, b - 1);
        const long long src = h * a.stride_head + min(max(idx_l[t], 0), n - 1) * a.stride_tok + c4;
        xk[k] = xv[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (a.K_out) xk[k] = *reinterpret_cast<const float4*>(a.K + src);
        if (a.V_out) xv[k] = *reinterpret_cast<const float4*>(a.V + src);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int t = t0 + (tid >> 5) + 32 * k;
        if (t < b) {
          if (a.K_out) *reinterpret_cast<float4*>(a.K_out + (ob + t) * kD + c4) = xk[k];
          if (a.V_out) *reinterpret_cast<float4*>(a.V_out + (ob + t) * kD + c4) = xv[k];
        }
      }
    }
  }
}

bool dense_f32_supported(const Layout& lay, int b) {
  return lay.dtype == DT_F32 && lay.n <= 256 && b <= kF32MaxB;
}

hipError_t launch_select_dense_f32(const void* V, const float* s, const Layout& lay, int b, float lambda,
                                   float eps, int32_t* idx_sorted, int32_t* pick_order, float* pick_gain,
                                   hipStream_t st) {
  return launch_retain_dense_f32(nullptr, V, nullptr, 0, s, lay, b, lambda, eps, nullptr, idx_sorted, pick_order,
                                 pick_gain, nullptr, nullptr, st);
}

hipError_t launch_retain_dense_f32(const void* K, const void* V, const void* Q, int G, const float* s,
                                   const Layout& lay, int b, float lambda, float eps, float* s_out,
                                   int32_t* idx_sorted, int32_t* pick_order, float* pick_gain, void* K_out,
                                   void* V_out, hipStream_t st) {
  F32Args a;
  a.K = static_cast<const float*>(K); a.Q = static_cast<const float*>(Q); a.G = G; a.s_out = s_out;
  a.K_out = static_cast<float*>(K_out); a.V_out = static_cast<float*>(V_out);
  a.V = static_cast<const float*>(V); a.s = s;
  a.idx_sorted = idx_sorted; a.pick_order = pick_order; a.pick_gain = pick_gain;
  a.stride_head = lay.stride_head; a.stride_tok = lay.stride_tok;
  a.n = lay.n; a.b = b; a.lambda = lambda; a.eps = eps;
  auto go = [&](auto kern, int smem) -> hipError_t {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(lay.heads), dim3(kF32Threads), smem, st, a);
    return hipGetLastError();
  };
  if (lay.n <= 64) return go(&select_dense_f32_kernel<2>, f32_smem_bytes(2));
  if (lay.n <= 128) return go(&select_dense_f32_kernel<4>, f32_smem_bytes(4));
  if (lay.n <= 192) return go(&select_dense_f32_kernel<6>, f32_smem_bytes(6));
  return go(&select_dense_f32_kernel<8>, f32_smem_bytes(8));
}

}  // namespace kvr
