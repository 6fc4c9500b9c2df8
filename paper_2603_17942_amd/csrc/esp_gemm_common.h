// What the GEMM sources share.
#pragma once
#include <hip/hip_ext.h>

#include "esp_internal.h"

namespace {

constexpr int KC = 64;            // k per chunk
// silu(g) * u with the hardware exponential and reciprocal (about 1 ulp each; the result is
// rounded to bf16 next)
__device__ __forceinline__ float silu_mul(float g, float u) {
  return g * u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f));
}

// launch, with a profiling scope's events attached to the kernel when there are any
template <typename Kern, typename... Args>
void launch_kernel(Kern kern, dim3 grid, dim3 block, size_t lds, hipStream_t st, Args... args) {
  if (g_launch_events.start || g_launch_events.stop) {
    hipExtLaunchKernelGGL(kern, grid, block, (uint32_t)lds, st, g_launch_events.start, g_launch_events.stop, 0, args...);
    g_launch_events = LaunchEvents{};
  } else {
    hipLaunchKernelGGL(kern, grid, block, lds, st, args...);
  }
}

}  // namespace
