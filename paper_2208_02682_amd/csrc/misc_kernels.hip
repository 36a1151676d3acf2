// Small utility kernels of the C ABI.
#include <hip/hip_runtime.h>

#include "launch.hpp"

namespace lm {

// every range to zero, or to the source given for it (blockIdx.y selects one),
// and *flag to zero: one launch instead of one fill or copy per range
__global__ void __launch_bounds__(256) k_set_ranges(SetRanges R) {
  const int q = blockIdx.y;
  unsigned long long* dst = R.dst[q];
  const unsigned long long* src = R.src[q];
  const size_t n = R.words[q];
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src ? src[i] : 0ull;
  if (R.flag && q == 0 && blockIdx.x == 0 && threadIdx.x == 0) *R.flag = 0;
}

// one RK4 step done: advance the batched runs' step counters
__global__ void k_batch_tick(long long* counters, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) counters[i] += 1;
}

void launch_batch_tick(hipStream_t st, long long* counters, int n) {
  if (n > 0) hipLaunchKernelGGL(k_batch_tick, dim3((n + 255) / 256), dim3(256), 0, st, counters, n);
}

void launch_set_ranges(hipStream_t st, const SetRanges& R) {
  size_t most = 1;
  for (int q = 0; q < R.count; ++q) most = R.words[q] > most ? R.words[q] : most;
  const size_t blocks = (most + 256 * 4 - 1) / (256 * 4);  // four words a thread, up to 1024 blocks a range
  hipLaunchKernelGGL(k_set_ranges, dim3((unsigned)(blocks < 1024 ? blocks : 1024), R.count), dim3(256), 0, st, R);
}

}  // namespace lm
