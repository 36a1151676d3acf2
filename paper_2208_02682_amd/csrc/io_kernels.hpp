// Float64 transforms used off the hot loop: physical <-> truncated spectral
// state for set_state / get_state, and the end-of-interval outputs (inverse
// transforms of the accumulators with the division by T in float64).
#pragma once

#include "io_structs.hpp"
#include "step_kernels.hpp"

namespace lm {

template <int N>
__global__ void __launch_bounds__(64 * ROW_WAVES) k_io_row_forward(IoRowFwd J, Dims d, const cplx<double>* tw) {
  using G = RowGeo<N>;
  constexpr int E = G::E, NT = G::NT;
  __shared__ __align__(16) double lds[G::RPB * 2 * G::L];
  const int grp = row_group<NT>(), t = threadIdx.x % NT;
  const int y = blockIdx.x * G::RPB + grp;
  double* buf = lds + grp * 2 * G::L;
  const int q = blockIdx.y;
  cplx<double> z[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const size_t i = (size_t)y * N + t + NT * e;
    z[e] = {J.a[q][i], J.b[q] ? J.b[q][i] : 0.0};
  }
  forward_row<double, N>(z, buf, t, tw, J.oa[q], J.b[q] ? J.ob[q] : nullptr, (unsigned)y * (unsigned)d.NKXP);
}

template <int N>
__global__ void __launch_bounds__(64 * ROW_WAVES) k_io_row_inverse(IoRowInv J, Dims d, const cplx<double>* tw) {
  using G = RowGeo<N>;
  constexpr int E = G::E, NT = G::NT;
  __shared__ __align__(16) double lds[G::RPB * 2 * G::L];
  const int grp = row_group<NT>(), t = threadIdx.x % NT;
  const int y = blockIdx.x * G::RPB + grp;
  double* buf = lds + grp * 2 * G::L;
  const int q = blockIdx.y;
  const cplx<double>* A = J.a[q];
  const cplx<double>* B = J.b[q] ? J.b[q] : A;
  cplx<double> z[E];
  load_pair<double, N, false, false>(z, A, B, (unsigned)y * (unsigned)d.NKXP, t);
  inverse_row<double, N>(z, buf, t, tw);
  bool bad = false;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const size_t i = (size_t)y * N + t + NT * e;
    const double a = z[e].x * J.sa[q] + J.ca[q];
    J.oa[q][i] = a;
    bad |= (a - a != 0.0);  // NaN or infinite
    if (J.b[q]) {
      const double b = z[e].y * J.sb[q] + J.cb[q];
      J.ob[q][i] = b;
      bad |= (b - b != 0.0);
    }
  }
  if (J.flag && __any(bad) && (threadIdx.x & 63) == 0) atomicOr(J.flag, 1);
}

template <int N>
__global__ void __launch_bounds__(col_threads<N>())
    k_io_col_forward(IoColFwd J, Dims d, const cplx<double>* tw) {
  constexpr int C = col_tile<N>();
  constexpr int E = fft_E<N>(), NT = N / E;
  __shared__ __align__(16) double lds[col_lds<double, N, C, false>()];
  const ColCtx<double, N, C> cx(lds, blockIdx.x);
  const int q = blockIdx.y;
  cplx<double> out[E];
  column_forward<double, N, C>(cx, J.src[q], nullptr, tw, out);
  if (!cx.valid) return;
  const size_t col = (size_t)cx.kx * d.NKY;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int k = cx.t + NT * r;
    int ky;
    if (k <= kcut<N>()) ky = k;
    else if (k >= N - kcut<N>()) ky = k - N;
    else continue;
    const size_t j = col + (size_t)(ky + d.K);
    cplx<double> v = out[r];
    if (cx.kx == 0 && ky == 0) v.y = 0.0;
    if (J.dst_f32[q]) {
      const cplx<float> hi = {float(v.x), float(v.y)};
      reinterpret_cast<cplx<float>*>(J.dst[q])[j] = hi;
      if (J.dst_lo[q])
        reinterpret_cast<cplx<float>*>(J.dst_lo[q])[j] = {float(v.x - double(hi.x)), float(v.y - double(hi.y))};
    } else {
      reinterpret_cast<cplx<double>*>(J.dst[q])[j] = v;
    }
  }
}

template <int N>
__global__ void __launch_bounds__(col_threads<N>())
    k_io_col_inverse(IoColInv J, Dims d, const cplx<double>* tw) {
  constexpr int C = col_tile<N>();
  constexpr int E = fft_E<N>(), NT = N / E;
  __shared__ __align__(16) double lds[col_lds<double, N, C, false>()];
  const ColCtx<double, N, C> cx(lds, blockIdx.x);
  const int q = blockIdx.y;
  const size_t col = (size_t)cx.kx * d.NKY;
  cplx<double> S[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int k = cx.t + NT * r;
    int ky;
    S[r] = {0.0, 0.0};
    if (k <= kcut<N>()) ky = k;
    else if (k >= N - kcut<N>()) ky = k - N;
    else continue;
    if (!cx.valid) continue;
    const size_t j = col + (size_t)(ky + d.K);
    if (J.src_f32[q]) {
      const cplx<float> s = reinterpret_cast<const cplx<float>*>(J.src[q])[j];
      S[r] = {double(s.x), double(s.y)};
      if (J.src_lo[q]) {
        const cplx<float> l = reinterpret_cast<const cplx<float>*>(J.src_lo[q])[j];
        S[r] = {S[r].x + double(l.x), S[r].y + double(l.y)};
      }
    } else {
      S[r] = reinterpret_cast<const cplx<double>*>(J.src[q])[j];
    }
  }
  column_inverse<double, N, C, false>(cx, S, J.dst[q], nullptr, tw);
}

}  // namespace lm
