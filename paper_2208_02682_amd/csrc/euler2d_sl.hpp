// Semi-Lagrangian strategy 1 (appendix B, eqs. (B.2), (B.4), (B.5)) after a
// step: departure point Y = X - d, d = dt u(X, t_{n+1}); with m = (t_n - tau)/dt
//   f~_{n+1}(X) = [m f~_n(Y) + (zeta_n(Y) + zeta_{n+1}(X)) / 2] / (m + 1)
//   eta_{n+1}(X) = [m eta_n(Y) + (m + 1/2) d] / (m + 1)
// Values at Y by the periodic bilinear or cubic interpolant.
#pragma once

#include "launch.hpp"

namespace lm {

// floor(o) taken periodically into [0, N): a finite displacement of any size
// wraps around the torus; beyond 2^30 cells, or NaN, cell 0 (non-finite
// weights then reach the outputs)
template <int N>
__device__ __forceinline__ int sl_cell(double f) {
  const int i = (fabs(f) < 1073741824.0) ? int(f) : 0;
  if constexpr ((N & (N - 1)) == 0) return i & (N - 1);
  const int r = i % N;
  return r < 0 ? r + N : r;
}

__device__ __forceinline__ void sl_cubic_weights(double a, double (&w)[4]) {
  const double p = a + 1.0, q = a - 1.0, r = a - 2.0;
  w[0] = -(a * q) * (r * (1.0 / 6.0));
  w[1] = (p * q) * (r * 0.5);
  w[2] = -(p * a) * (r * 0.5);
  w[3] = (p * a) * (q * (1.0 / 6.0));
}

// one grid point; the four gathered fields share the cell and the weights
template <int N>
__device__ __forceinline__ void sl_update(const E2DSl& a, int i) {
  if (i >= N * N) return;
  const int jx = i % N, jy = i / N;
  const double dx = 6.283185307179586476925286766559 / N;
  const double d_x = a.dt * a.u[i], d_y = a.dt * a.v[i];
  const double ox = -d_x / dx, oy = -d_y / dx;  // cell and weights from the small offset
  const double fx = floor(ox), fy = floor(oy);
  const double ax = ox - fx, ay = oy - fy;
  int bx = jx + sl_cell<N>(fx), by = jy + sl_cell<N>(fy);  // in [0, 2N)
  bx = bx >= N ? bx - N : bx;
  by = by >= N ? by - N : by;
  const double* F[4] = {a.f_old, a.znow, a.ex_old, a.ey_old};
  double at[4];
  if (a.cubic) {
    double wx[4], wy[4];
    sl_cubic_weights(ax, wx);
    sl_cubic_weights(ay, wy);
    int c[4], r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      c[k] = bx + k - 1;
      c[k] = c[k] < 0 ? c[k] + N : (c[k] >= N ? c[k] - N : c[k]);
      r[k] = by + k - 1;
      r[k] = (r[k] < 0 ? r[k] + N : (r[k] >= N ? r[k] - N : r[k])) * N;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      at[q] = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        double row = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) row += wx[k] * F[q][r[j] + c[k]];
        at[q] += wy[j] * row;
      }
    }
  } else {
    const int ix1 = bx + 1 == N ? 0 : bx + 1, iy1 = by + 1 == N ? 0 : by + 1;
    const double w00 = (1.0 - ax) * (1.0 - ay), w01 = ax * (1.0 - ay), w10 = (1.0 - ax) * ay, w11 = ax * ay;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      at[q] = w00 * F[q][by * N + bx] + w01 * F[q][by * N + ix1] + w10 * F[q][iy1 * N + bx] + w11 * F[q][iy1 * N + ix1];
  }
  const double zn = a.znext[i];
  a.f_new[i] = (a.m * at[0] + 0.5 * (at[1] + zn)) / (a.m + 1.0);
  a.ex_new[i] = (a.m * at[2] + (a.m + 0.5) * d_x) / (a.m + 1.0);
  a.ey_new[i] = (a.m * at[3] + (a.m + 0.5) * d_y) / (a.m + 1.0);
  a.z_new[i] = zn;
}

// the update alone (the last step of a call, and measurement)
template <int N>
__global__ void __launch_bounds__(256) k_e2d_sl(E2DSl a) {
  sl_update<N>(a, blockIdx.x * 256 + threadIdx.x);
}

template <int N>
void launch_e2d_sl(hipStream_t st, const E2DSl& a) {
  hipLaunchKernelGGL((k_e2d_sl<N>), dim3((N * N + 255) / 256), dim3(256), 0, st, a);
}

}  // namespace lm
