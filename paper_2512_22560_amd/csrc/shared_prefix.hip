// Merge of two results over disjoint token ranges (of one trajectory's context split over calls or GPUs).
#include "rollattn_internal.h"

namespace rollattn {

namespace {

constexpr int kThreads = 256;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Attention over the union of two disjoint token ranges from the results over each (one wave per row): weights
// 2^d1 and 2^d2 on the two outputs, log2(2^d1 + 2^d2) as the new denominator's logarithm.  A side that saw nothing
// (d = -inf) has weight 0; when both saw nothing the row is zero and its logarithm -inf.
template <int D, typename T>
__global__ __launch_bounds__(kThreads) void merge_states_kernel(const T* o1, const float* __restrict__ d1, const T* o2,
                                                                const float* __restrict__ d2, T* out, float* d_out, long rows) {
  constexpr int kPer = D / 64;                            // consecutive elements per lane, moved as one vector
  typedef T vec_t __attribute__((ext_vector_type(kPer)));
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const size_t off = (size_t)row * D + lane * kPer;
  const vec_t v1 = *(const vec_t*)(o1 + off), v2 = *(const vec_t*)(o2 + off);   // out may be o1 or o2: read first
  const float a = d1[row], b = d2[row];
  const float top = fmaxf(a, b);
  const float m = (top == -INFINITY) ? 0.f : top;
  const float wa = __builtin_amdgcn_exp2f(a - m), wb = __builtin_amdgcn_exp2f(b - m);   // 2^-inf = 0
  const float tot = wa + wb;
  const float inv = tot > 0.f ? 1.f / tot : 0.f;
  vec_t r;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    // an empty side may hold anything (zeros by this library's calls): its weight is an exact zero, but keep
    // non-finite leftovers of other producers out of the sum
    const float x1 = wa > 0.f ? (float)v1[e] : 0.f, x2 = wb > 0.f ? (float)v2[e] : 0.f;
    r[e] = (T)((wa * x1 + wb * x2) * inv);
  }
  *(vec_t*)(out + off) = r;
  if (d_out && lane == 0) d_out[row] = tot > 0.f ? m + __builtin_amdgcn_logf(tot) : -INFINITY;
}

}  // namespace

hipError_t launch_merge_states(const void* o1, const float* d1, const void* o2, const float* d2, void* out, float* d_out,
                               long rows, int head_dim, bool f32, hipStream_t s) {
  const int grid = (int)((rows + kThreads / 64 - 1) / (kThreads / 64));
  if (grid == 0) return hipSuccess;
  if (head_dim == 128 && !f32) {
    hipLaunchKernelGGL((merge_states_kernel<128, __bf16>), dim3(grid), dim3(kThreads), 0, s, (const __bf16*)o1, d1, (const __bf16*)o2, d2, (__bf16*)out, d_out, rows);
  } else if (head_dim == 64 && !f32) {
    hipLaunchKernelGGL((merge_states_kernel<64, __bf16>), dim3(grid), dim3(kThreads), 0, s, (const __bf16*)o1, d1, (const __bf16*)o2, d2, (__bf16*)out, d_out, rows);
  } else if (head_dim == 128) {
    hipLaunchKernelGGL((merge_states_kernel<128, float>), dim3(grid), dim3(kThreads), 0, s, (const float*)o1, d1, (const float*)o2, d2, (float*)out, d_out, rows);
  } else if (head_dim == 64) {
    hipLaunchKernelGGL((merge_states_kernel<64, float>), dim3(grid), dim3(kThreads), 0, s, (const float*)o1, d1, (const float*)o2, d2, (float*)out, d_out, rows);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rollattn
