// State rows in and out of a world: the boundary hands over one row of 13
// floats per body, the kernels keep 13 component arrays.
//
// Both directions turn a block of 256 bodies through LDS, so that the arrays
// and the rows are each read and written in whole cache lines (a row stride of
// 13 words meets every LDS bank).  The rows may lie in pinned host memory:
// the same kernel is then the transfer, bound by the host's copy into that
// memory (12 GB/s).  At 1,024 envs of 32 bodies (1.7 MB) a load from the
// binding takes 151 us and a fetch into device memory 18 us; 13 copies per
// direction and a transpose on the host took 1.4 ms for the two.
#include <type_traits>

#include "vuda_runtime.h"

namespace vuda {
namespace {

constexpr int kBlock = 256;

__global__ __launch_bounds__(kBlock) void state_gather_kernel(const float* state, int64_t cap, int64_t nb, float* rows) {
  __shared__ float t[kBlock * kStateComps];
  const int tid = threadIdx.x;
  const int64_t first = (int64_t)blockIdx.x * kBlock;
  const int n = (int)(nb - first < kBlock ? nb - first : kBlock);
  if (tid < n) {
#pragma unroll
    for (int k = 0; k < kStateComps; ++k) t[tid * kStateComps + k] = state[k * cap + first + tid];
  }
  __syncthreads();
  float* dst = rows + first * kStateComps;
  for (int i = tid; i < n * kStateComps; i += kBlock) dst[i] = t[i];
}

// PARTS: the rows come as four arrays of 3, 3, 4 and 3 floats a body, one
// after the other.
template <bool PARTS>
__global__ __launch_bounds__(kBlock) void state_scatter_kernel(const float* rows, int64_t cap, int64_t nb, float* state) {
  __shared__ float t[kBlock * kStateComps];
  const int tid = threadIdx.x;
  const int64_t first = (int64_t)blockIdx.x * kBlock;
  const int n = (int)(nb - first < kBlock ? nb - first : kBlock);
  if constexpr (PARTS) {
    const auto part = [&](auto width, int at) {
      constexpr int w = decltype(width)::value;
      const float* src = rows + at * nb + first * w;
      for (int i = tid; i < n * w; i += kBlock) t[i / w * kStateComps + at + i % w] = src[i];
    };
    part(std::integral_constant<int, 3>{}, PX);
    part(std::integral_constant<int, 3>{}, VX);
    part(std::integral_constant<int, 4>{}, QW);
    part(std::integral_constant<int, 3>{}, WX);
  } else {
    const float* src = rows + first * kStateComps;
    for (int i = tid; i < n * kStateComps; i += kBlock) t[i] = src[i];
  }
  __syncthreads();
  if (tid < n) {
#pragma unroll
    for (int k = 0; k < kStateComps; ++k) state[k * cap + first + tid] = t[tid * kStateComps + k];
  }
}

}  // namespace

hipError_t launch_state_gather(const float* state, int64_t cap, int64_t b0, int64_t nb, float* rows, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(state_gather_kernel, dim3((unsigned)((nb + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, state + b0,
                     cap, nb, rows);
  return hipGetLastError();
}

hipError_t launch_state_scatter(const float* rows, bool parts, float* state, int64_t cap, int64_t b0, int64_t nb,
                                hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  const dim3 g((unsigned)((nb + kBlock - 1) / kBlock));
  if (parts) hipLaunchKernelGGL(state_scatter_kernel<true>, g, dim3(kBlock), 0, s, rows, cap, nb, state + b0);
  else hipLaunchKernelGGL(state_scatter_kernel<false>, g, dim3(kBlock), 0, s, rows, cap, nb, state + b0);
  return hipGetLastError();
}

}  // namespace vuda
