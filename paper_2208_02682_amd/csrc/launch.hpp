// Per-N launchers (explicitly instantiated in inst_<N>.hip so that the
// kernels of different grid sizes compile in parallel).
#pragma once

#include "io_structs.hpp"
#include "run_view.hpp"

namespace lm {

template <int N> void launch_steps(RunView& r, int nsteps);   // nsteps RK4 steps
template <int N> hipError_t launch_steps_profiled(RunView& r, int nsteps, double* ms);  // + kernel times
template <int N> void launch_prologue(RunView& r);            // column pass of the current state
template <int N> void launch_prologue_dyn(RunView& r);        // of u, v, h alone
// one RK4 step for nruns runs of one (N, precision, gather, momentum, averaged fields) group; desc: device array of RunDesc<T>
template <int N> void launch_batch_step(hipStream_t st, const void* desc, int nruns, bool fp32, bool cubic, bool mom,
                                        bool gen, const Sched& sc);
void launch_batch_tick(hipStream_t st, long long* counters, int n);  // counters[i] += 1
template <int N> void launch_io_row_forward(RunView& r, const IoRowFwd& J, int count);
template <int N> void launch_io_col_forward(RunView& r, const IoColFwd& J, int count);
template <int N> void launch_io_col_inverse(RunView& r, const IoColInv& J, int count);
template <int N> void launch_io_row_inverse(RunView& r, const IoRowInv& J, int count);
// device ranges of 64-bit words set in one launch: zeroed, or copied from src
struct SetRanges {
  int count = 0;
  unsigned long long* dst[5] = {};
  const unsigned long long* src[5] = {};
  size_t words[5] = {};
  int* flag = nullptr;  // zeroed as well, when given
  void add(void* d, size_t bytes, const void* s = nullptr) {
    dst[count] = (unsigned long long*)d;
    src[count] = (const unsigned long long*)s;
    words[count++] = bytes / 8;
  }
};
void launch_set_ranges(hipStream_t st, const SetRanges& R);
// two-dimensional incompressible flow (float64; euler2d_step.hpp, euler2d_sl.hpp)
constexpr int E2D_NIC = 10;  // column-pass outputs
struct E2DPtrs {
  cplx<double>* Y;   // [4][NKX][NKY] zeta, g~, P_x, P_y
  cplx<double>* Yn;  // the state after the step
  cplx<double>* K1;  // Heun's first slope, same shape
  cplx<double>* IC;  // [E2D_NIC][N][NKXP]
  cplx<double>* RS;  // [4][N][NKXP]
  double* PH;        // [3][N][N] u, v, zeta
  const cplx<double>* tw;
  double U0, V0, dt;
};
struct E2DSl {  // one semi-Lagrangian update
  const double *u, *v, *znext, *znow, *f_old, *ex_old, *ey_old;
  double *f_new, *ex_new, *ey_new, *z_new;
  double dt, m;
  int cubic;
};
// store: u, v, zeta to PH; products: the right-hand sides' row spectra
template <int N> void launch_e2d_rows(hipStream_t st, const E2DPtrs& P, double s, int store, int products);
// stage 0, 1 of Heun's method, or -1: the current state's transforms; sl: a
// semi-Lagrangian update carried along (or null)
template <int N> void launch_e2d_columns(hipStream_t st, const E2DPtrs& P, int stage, const E2DSl* sl);
template <int N> void launch_e2d_sl(hipStream_t st, const E2DSl& a);

// strategy-1 remap of the interval outputs (float64, N x N planes)
void launch_remap_s1(RunView& r, const double* fh, const double* fz, const double* ex, const double* ey,
                     double* out, unsigned* best, int max_extent, unsigned long long* resid_bits);

#define LM_DISPATCH_N_RET(n, out, FN, ...)       \
  switch (n) {                                    \
    case 64: out = FN<64>(__VA_ARGS__); break;    \
    case 128: out = FN<128>(__VA_ARGS__); break;  \
    case 192: out = FN<192>(__VA_ARGS__); break;  \
    case 256: out = FN<256>(__VA_ARGS__); break;  \
    case 384: out = FN<384>(__VA_ARGS__); break;  \
    case 512: out = FN<512>(__VA_ARGS__); break;  \
    case 1024: out = FN<1024>(__VA_ARGS__); break;\
    default: break;                               \
  }

#define LM_DISPATCH_N(n, FN, ...)            \
  switch (n) {                               \
    case 64: FN<64>(__VA_ARGS__); break;     \
    case 128: FN<128>(__VA_ARGS__); break;   \
    case 192: FN<192>(__VA_ARGS__); break;   \
    case 256: FN<256>(__VA_ARGS__); break;   \
    case 384: FN<384>(__VA_ARGS__); break;   \
    case 512: FN<512>(__VA_ARGS__); break;   \
    case 1024: FN<1024>(__VA_ARGS__); break; \
    default: break;                          \
  }

}  // namespace lm
