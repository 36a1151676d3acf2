// Column tiles of the column pass: how many spectral columns one block
// transforms.  Shared by the kernels and by the host code that checks launch
// schedules.
#pragma once

#include "fft_core.hpp"

namespace lm {

// column tile width: 8 columns (64-byte row segments in float32).  W = -1 / +1: half /
// twice that width (the alternative launch schedules; the arithmetic of every column
// is the same whatever the width).  A transform has at least 16 lanes, so that a
// block of half the width still is whole wavefronts.
__host__ __device__ constexpr int col_tile_of(int w) { return w < 0 ? 4 : (w > 0 ? 16 : 8); }
__host__ __device__ constexpr int col_buf(int N) { return padded_len(N) | 1; }
// The widths offered as schedules: those whose block would be whole wavefronts
// (at most 1024 threads) with 16 values per lane (12 for N = 3 * 2^k), and whose
// LDS fits in a CU's 160 KiB.  The list is part of the interface, so it does not
// follow the values per lane the kernels use (never more than 16; a width is
// then whole wavefronts with those too, which the kernels assert).
__host__ __device__ constexpr bool col_tile_usable(int n, int w, int cplx_bytes) {
  const int lanes = n / ((n % 3 == 0) ? 12 : 16);
  const int base = (lanes >= 8) ? 8 : 64 / lanes;
  const int cols = w < 0 ? base / 2 : (w > 0 ? base * 2 : base);
  const int threads = cols * lanes;
  return cols >= 1 && threads >= 64 && threads % 64 == 0 && threads <= 1024 &&
         (long long)cols * col_buf(n) * cplx_bytes <= 160LL * 1024;
}

}  // namespace lm
