// lambda = 0 for heads of more than 256 tokens: Algorithm 1's explicit top-b branch
// (paper Sec. 4.1: at lambda = 0 the selector is the baseline's modular top-k, ties to
// the lower index), followed by the compaction of the kept rows.  V is never read for
// the selection, so the kernel needs a few KB of LDS and many heads share a CU, which
// is what hides the latency of its short dependent steps:
//   1. the b-th largest score key by a bitwise search (one workgroup-wide count per bit);
//   2. the selected tokens in token order (keys above the threshold, then the lowest-
//      indexed of the equal ones) -- that list is sort(S);
//   3. each selected token's rank among the selected gives the pick order and gains;
//   4. the kept K/V rows are copied (bf16 rows; other layouts are compacted by the caller).
// Token j = 256 * k + thread: score loads are coalesced.
#include "kvr_kernels.hpp"
#include "kvr_topb.hpp"

namespace kvr {

template <int S>
__global__ __launch_bounds__(kTopbThreads) void select_topb_kernel(TopbArgs a) {
  extern __shared__ __align__(16) int32_t smem_i[];
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t key[S];
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const int j = k * kTopbThreads + tid;
    key[k] = j < a.n ? ordered_key(a.s_in[static_cast<long long>(h) * a.n + j] + 0.0f) : 0u;   // -0 counts as +0
  }
  topb_finish<S>(a, smem_i, key, h, tid, lane, w);
}

bool topb_supported(const Layout& lay, int b, float lambda) {
  return lambda == 0.0f && lay.n > 256 && lay.n <= 32 * kTopbThreads && b <= kTopbMaxB;
}

hipError_t launch_select_topb(const void* K, const void* V, const float* s, const Layout& lay, int b,
                              int32_t* idx_sorted, int32_t* pick_order, float* pick_gain, void* K_out,
                              void* V_out, hipStream_t st, const int32_t* b_h) {
  TopbArgs a;
  a.b_h = b_h;
  a.K = static_cast<const char*>(K); a.V = static_cast<const char*>(V); a.s_in = s;
  a.idx_sorted = idx_sorted; a.pick_order = pick_order; a.pick_gain = pick_gain;
  a.K_out = static_cast<char*>(K_out); a.V_out = static_cast<char*>(V_out);
  a.stride_head = lay.stride_head; a.stride_tok = lay.stride_tok;
  a.n = lay.n; a.b = b;
  if ((K_out || V_out) && lay.dtype != DT_BF16) return hipErrorInvalidValue;   // rows are copied as bf16 rows
  auto go = [&](auto kern, int slots) -> hipError_t {
    const int smem = topb_smem_bytes(slots, b);
    hipLaunchKernelGGL(kern, dim3(lay.heads), dim3(kTopbThreads), smem, st, a);
    return hipGetLastError();
  };
  if (lay.n <= 4 * kTopbThreads) return go(&select_topb_kernel<4>, 4);
  if (lay.n <= 8 * kTopbThreads) return go(&select_topb_kernel<8>, 8);
  if (lay.n <= 16 * kTopbThreads) return go(&select_topb_kernel<16>, 16);
  return go(&select_topb_kernel<32>, 32);
}

}  // namespace kvr
