// k_readback.hip -- small results from device arrays to pinned host memory, and
// small initial values the other way, by kernels: a call that reads back a few
// counters launches one kernel and waits once, where every hipMemcpyAsync to
// or from unpinned memory is staged and waited for by itself.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "clair_launch.h"

namespace clair {

namespace {

__global__ void k_collect(CollectArgs a) {
  int at = 0;
  for (int k = 0; k < kCollectMax; ++k) {
    if ((int)threadIdx.x < a.n[k]) a.dst[at + threadIdx.x] = a.src[k][threadIdx.x];
    at += a.n[k];
  }
}

__global__ void k_copy_words(const int32_t* __restrict__ src, int32_t* __restrict__ dst, int n) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) dst[t] = src[t];
}

__global__ void k_set_ints(int32_t* dst, SetArgs a) {
  if ((int)threadIdx.x < a.n) dst[threadIdx.x] = a.v[threadIdx.x];
}

__global__ void k_copy_unless(const int32_t* __restrict__ flag, const double* __restrict__ src,
                              double* __restrict__ dst, int n) {
  if (flag && *flag) return;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) dst[t] = src[t];
}

int cgrid(int n) { return n < 256 * 1024 ? (n + 255) / 256 : 1024; }

}  // namespace

hipError_t launch_collect(const CollectArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_collect, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_copy_words(const int32_t* src, int32_t* dst, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_copy_words, dim3(cgrid(n)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}
hipError_t launch_set_ints(int32_t* dst, const SetArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_set_ints, dim3(1), dim3(64), 0, s, dst, a);
  return hipGetLastError();
}
hipError_t launch_copy_unless(const int32_t* flag, const double* src, double* dst, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_copy_unless, dim3(cgrid(n)), dim3(256), 0, s, flag, src, dst, n);
  return hipGetLastError();
}

}  // namespace clair
