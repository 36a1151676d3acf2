// C ABI of the two-dimensional incompressible flow with strategy 1
// pseudospectral and semi-Lagrangian (lm_e2d_*, include/lagmean.h).  float64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "lagmean.h"
#include "launch.hpp"
#include "twiddles.hpp"

using lm::cplx;

namespace lm {
lm_status api_fail(lm_status s, const std::string& msg);
}

namespace {

lm_status fail(lm_status s, const std::string& msg) { return lm::api_fail(s, msg); }

#define HIP_TRY(expr)                                                                    \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess) return fail(LM_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

lm_status check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LM_E_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
  return LM_OK;
}

constexpr int NOUT_E2D = 7;

}  // namespace

struct lm_e2d {
  lm::RunView v;  // dims, stream, slab and twiddles for the transform launchers
  double dt, U0, V0;
  bool cubic;
  // byte offsets in v.slab
  size_t Yb[2], K1, IC, PH, RSF, SLf[2], SLx[2], SLy[2], Zn[2], OUT, total;
  int cur;   // current semi-Lagrangian fields
  int ycur;  // current spectral state
  size_t Y() const { return Yb[ycur]; }
  bool has_state, in_interval, has_out;
  bool ic_current;  // the column-pass outputs are those of the current state
  int64_t n, n_tau;
  double T;
  template <typename X>
  X* at(size_t off) { return reinterpret_cast<X*>(v.slab + off); }
};

namespace {

lm_status e2d_layout(lm_e2d* e) {
  const lm::Dims& d = e->v.d;
  const size_t sp = d.spec_elems(), rf = d.rowfield_elems(), nn = (size_t)d.N * d.N;
  const size_t cD = sizeof(cplx<double>);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t a = o;
    o += (bytes + 255) / 256 * 256;
    return a;
  };
  e->v.L = lm::Layout{};
  e->v.L.tw64 = take(d.N * cD);
  for (int k = 0; k < 2; ++k) e->Yb[k] = take(4 * sp * cD);
  e->K1 = take(4 * sp * cD);
  e->IC = take(lm::E2D_NIC * rf * cD);
  e->PH = take(3 * nn * sizeof(double));
  e->RSF = take(4 * rf * cD);
  for (int k = 0; k < 2; ++k) {
    e->SLf[k] = take(nn * sizeof(double));
    e->SLx[k] = take(nn * sizeof(double));
    e->SLy[k] = take(nn * sizeof(double));
    e->Zn[k] = take(nn * sizeof(double));
  }
  e->OUT = take(NOUT_E2D * nn * sizeof(double));
  e->total = o;
  return LM_OK;
}

lm::E2DPtrs e2d_ptrs(lm_e2d* e) {
  lm::E2DPtrs P;
  P.Y = e->at<cplx<double>>(e->Y());
  P.Yn = e->at<cplx<double>>(e->Yb[e->ycur ^ 1]);
  P.K1 = e->at<cplx<double>>(e->K1);
  P.IC = e->at<cplx<double>>(e->IC);
  P.RS = e->at<cplx<double>>(e->RSF);
  P.PH = e->at<double>(e->PH);
  P.tw = e->at<const cplx<double>>(e->v.L.tw64);
  P.U0 = e->U0;
  P.V0 = e->V0;
  P.dt = e->dt;
  return P;
}

// the column-pass outputs of the current state
void e2d_prologue(lm_e2d* e, const lm::E2DPtrs& P) {
  if (e->ic_current) return;
  LM_DISPATCH_N(e->v.d.N, lm::launch_e2d_columns, e->v.stream, P, -1, nullptr);
  e->ic_current = true;
}

void e2d_zero_means(lm_e2d* e) {
  const size_t sp = e->v.d.spec_elems(), nn = (size_t)e->v.d.N * e->v.d.N;
  lm::SetRanges R;
  R.add(e->at<char>(e->Y()) + sp * sizeof(cplx<double>), 3 * sp * sizeof(cplx<double>));
  R.add(e->at<char>(e->SLf[e->cur]), nn * sizeof(double));
  R.add(e->at<char>(e->SLx[e->cur]), nn * sizeof(double));
  R.add(e->at<char>(e->SLy[e->cur]), nn * sizeof(double));
  lm::launch_set_ranges(e->v.stream, R);
}

// the semi-Lagrangian update after step m of the interval (u, v, zeta at its end
// are in PH), from the current set of fields to the other
lm::E2DSl e2d_sl_args(lm_e2d* e, double m) {
  const size_t nn = (size_t)e->v.d.N * e->v.d.N;
  const double* PH = e->at<double>(e->PH);
  const int c = e->cur, o = c ^ 1;
  return lm::E2DSl{PH, PH + nn, PH + 2 * nn, e->at<double>(e->Zn[c]), e->at<double>(e->SLf[c]),
                   e->at<double>(e->SLx[c]), e->at<double>(e->SLy[c]), e->at<double>(e->SLf[o]),
                   e->at<double>(e->SLx[o]), e->at<double>(e->SLy[o]), e->at<double>(e->Zn[o]), e->dt, m,
                   e->cubic ? 1 : 0};
}

// nsteps Heun steps of everything with their semi-Lagrangian updates.  A step's
// update needs u, v and zeta at its end: the next step's first rows pass stores
// them, and its blocks ride in the column launch that follows; after the last
// step a rows pass stores them and the update runs alone.  With events (a pair
// per step) every update is a launch of its own between its pair.
// A step counts once its update is launched too.  Until then the state it began
// from is whole (the next step writes over it after the update only), so when a
// launch fails the handle stays at the last step that counts.
lm_status e2d_steps(lm_e2d* e, int nsteps, hipEvent_t* ev) {
  if (nsteps <= 0) return LM_OK;
  lm::RunView& v = e->v;
  const int N = v.d.N;
  lm::E2DPtrs P = e2d_ptrs(e);
  bool pending = false;  // the spectral state is a step ahead of the update
  auto counts = [&] {
    e->cur ^= 1;
    e->n += 1;
    pending = false;
  };
  auto sl_alone = [&](double m, hipEvent_t* pair) -> lm_status {
    const lm::E2DSl a = e2d_sl_args(e, m);
    if (pair) HIP_TRY(hipEventRecord(pair[0], v.stream));
    LM_DISPATCH_N(N, lm::launch_e2d_sl, v.stream, a);
    if (pair) HIP_TRY(hipEventRecord(pair[1], v.stream));
    const lm_status st = check_launch();
    if (st == LM_OK) counts();
    return st;
  };
  auto steps = [&]() -> lm_status {
    lm_status st;
    e2d_prologue(e, P);
    for (int k = 0; k < nsteps; ++k) {
      const double m = double(e->n - e->n_tau) + (pending ? 1.0 : 0.0);
      const double s0 = m * e->dt;
      LM_DISPATCH_N(N, lm::launch_e2d_rows, v.stream, P, s0, pending ? 1 : 0, 1);
      if (pending && !ev) {
        const lm::E2DSl a = e2d_sl_args(e, m - 1.0);
        LM_DISPATCH_N(N, lm::launch_e2d_columns, v.stream, P, 0, &a);
        if ((st = check_launch()) != LM_OK) return st;
        counts();
      } else {
        if (pending && (st = sl_alone(m - 1.0, ev + 2 * (k - 1))) != LM_OK) return st;
        LM_DISPATCH_N(N, lm::launch_e2d_columns, v.stream, P, 0, nullptr);
      }
      LM_DISPATCH_N(N, lm::launch_e2d_rows, v.stream, P, s0 + e->dt, 0, 1);
      LM_DISPATCH_N(N, lm::launch_e2d_columns, v.stream, P, 1, nullptr);
      if ((st = check_launch()) != LM_OK) return st;
      e->ycur ^= 1;
      std::swap(P.Y, P.Yn);
      pending = true;
    }
    LM_DISPATCH_N(N, lm::launch_e2d_rows, v.stream, P, 0.0, 1, 0);
    return sl_alone(double(e->n - e->n_tau), ev ? ev + 2 * (nsteps - 1) : nullptr);
  };
  const lm_status st = steps();
  if (st != LM_OK) {
    if (pending) e->ycur ^= 1;
    e->ic_current = false;
  }
  return st;
}

}  // namespace

extern "C" {

lm_status lm_e2d_create(const lm_e2d_config* cfg, void* hip_stream, lm_e2d** out) {
  if (!out) return fail(LM_E_ARG, "null out");
  *out = nullptr;
  if (!cfg) return fail(LM_E_ARG, "null config");
  const int n = cfg->n;
  if (!(n == 64 || n == 128 || n == 192 || n == 256 || n == 384 || n == 512 || n == 1024))
    return fail(LM_E_UNSUPPORTED, "n must be 64, 128, 192, 256, 384, 512 or 1024");
  if (!(cfg->dt > 0.0) || !std::isfinite(cfg->dt)) return fail(LM_E_ARG, "dt must be positive and finite");
  if (!std::isfinite(cfg->U0) || !std::isfinite(cfg->V0)) return fail(LM_E_ARG, "U0, V0 must be finite");
  if (cfg->interp != LM_INTERP_BILINEAR && cfg->interp != LM_INTERP_CUBIC)
    return fail(LM_E_UNSUPPORTED, "interp must be LM_INTERP_BILINEAR or LM_INTERP_CUBIC");
  lm_e2d* e = new lm_e2d();
  e->v.d = lm::Dims::make(n);
  e->v.stream = (hipStream_t)hip_stream;
  e->v.fp32 = false;
  e->v.cubic = false;
  e->dt = cfg->dt;
  e->U0 = cfg->U0;
  e->V0 = cfg->V0;
  e->cubic = cfg->interp == LM_INTERP_CUBIC;
  e->cur = e->ycur = 0;
  e->has_state = e->in_interval = e->has_out = e->ic_current = false;
  e->n = e->n_tau = 0;
  e->T = 0.0;
  e2d_layout(e);
  hipError_t err = hipMalloc((void**)&e->v.slab, e->total);
  if (err != hipSuccess) {
    delete e;
    (void)hipGetLastError();
    return fail(LM_E_OOM, std::string("hipMalloc: ") + hipGetErrorString(err));
  }
  const std::vector<cplx<double>> tw = lm::stage_twiddles<double>(n);
  err = hipMemcpy(e->v.slab + e->v.L.tw64, tw.data(), n * sizeof(cplx<double>), hipMemcpyHostToDevice);
  if (err != hipSuccess) {
    (void)hipFree(e->v.slab);
    delete e;
    return fail(LM_E_HIP, std::string("twiddles: ") + hipGetErrorString(err));
  }
  *out = e;
  return LM_OK;
}

lm_status lm_e2d_set_vorticity(lm_e2d* e, const double* zeta, int on_device) {
  if (!e || !zeta) return fail(LM_E_ARG, "null argument");
  lm::RunView& v = e->v;
  const lm::Dims& d = v.d;
  const size_t nn = (size_t)d.N * d.N;
  const lm::StreamDrain drain{v.stream};  // the caller's buffer is read before any return
  double* PH = e->at<double>(e->PH);
  HIP_TRY(hipMemcpyAsync(PH, zeta, nn * sizeof(double), on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                         v.stream));
  cplx<double>* RSF = e->at<cplx<double>>(e->RSF);
  lm::IoRowFwd F{};
  F.a[0] = PH;
  F.oa[0] = RSF;
  LM_DISPATCH_N(d.N, lm::launch_io_row_forward, v, F, 1);
  lm::IoColFwd C{};
  C.src[0] = RSF;
  C.dst[0] = e->at<cplx<double>>(e->Y());
  C.dst_f32[0] = 0;
  LM_DISPATCH_N(d.N, lm::launch_io_col_forward, v, C, 1);
  e->cur = 0;
  lm_status st;
  e2d_zero_means(e);
  // zeta_n on the grid for the first semi-Lagrangian step
  e->ic_current = false;
  const lm::E2DPtrs P = e2d_ptrs(e);
  e2d_prologue(e, P);
  LM_DISPATCH_N(d.N, lm::launch_e2d_rows, v.stream, P, 0.0, 1, 0);
  lm::SetRanges Z;
  Z.add(e->at<double>(e->Zn[e->cur]), nn * sizeof(double), PH + 2 * nn);
  lm::launch_set_ranges(v.stream, Z);
  if ((st = check_launch()) != LM_OK) {
    e->ic_current = false;
    return st;
  }
  HIP_TRY(hipStreamSynchronize(v.stream));
  e->n = e->n_tau = 0;
  e->has_state = true;
  e->in_interval = false;
  return LM_OK;
}

lm_status lm_e2d_begin_interval(lm_e2d* e) {
  if (!e) return fail(LM_E_ARG, "null handle");
  if (!e->has_state) return fail(LM_E_STATE, "no vorticity set");
  lm_status st;
  e->ic_current = false;
  e2d_zero_means(e);
  if ((st = check_launch()) != LM_OK) return st;
  e->n_tau = e->n;
  e->in_interval = true;
  return LM_OK;
}

lm_status lm_e2d_step(lm_e2d* e, int32_t nsteps) {
  if (!e) return fail(LM_E_ARG, "null handle");
  if (nsteps < 0) return fail(LM_E_ARG, "nsteps < 0");
  if (!e->has_state) return fail(LM_E_STATE, "no vorticity set");
  return e2d_steps(e, nsteps, nullptr);
}

lm_status lm_e2d_step_profiled(lm_e2d* e, int32_t nsteps, double* ms_step, double* ms_sl) {
  if (!e || !ms_step || !ms_sl) return fail(LM_E_ARG, "null argument");
  if (nsteps <= 0 || nsteps > 4096) return fail(LM_E_ARG, "nsteps must be in 1..4096");
  if (!e->has_state) return fail(LM_E_STATE, "no vorticity set");
  std::vector<hipEvent_t> ev(2 * nsteps + 2, nullptr);
  lm_status st = LM_OK;
  for (auto& x : ev)
    if (hipEventCreateWithFlags(&x, hipEventDisableSystemFence) != hipSuccess) st = fail(LM_E_HIP, "event creation");
  if (st == LM_OK && hipEventRecord(ev[2 * nsteps], e->v.stream) != hipSuccess) st = fail(LM_E_HIP, "event record");
  if (st == LM_OK) st = e2d_steps(e, nsteps, ev.data());
  if (st == LM_OK && hipEventRecord(ev[2 * nsteps + 1], e->v.stream) != hipSuccess) st = fail(LM_E_HIP, "event record");
  if (st == LM_OK && hipEventSynchronize(ev[2 * nsteps + 1]) != hipSuccess) st = fail(LM_E_HIP, "event sync");
  if (st == LM_OK) {
    double sl = 0.0;
    float t = 0.f;
    for (int k = 0; k < nsteps; ++k) {
      if (hipEventElapsedTime(&t, ev[2 * k], ev[2 * k + 1]) != hipSuccess) st = fail(LM_E_HIP, "elapsed time");
      sl += t;
    }
    if (hipEventElapsedTime(&t, ev[2 * nsteps], ev[2 * nsteps + 1]) != hipSuccess) st = fail(LM_E_HIP, "elapsed time");
    *ms_step = double(t) / nsteps;
    *ms_sl = sl / nsteps;
  }
  for (auto& x : ev)
    if (x) (void)hipEventDestroy(x);
  return st;
}

lm_status lm_e2d_end_interval(lm_e2d* e, double* T_out) {
  if (!e) return fail(LM_E_ARG, "null handle");
  if (!e->in_interval) return fail(LM_E_STATE, "no open interval");
  if (e->n == e->n_tau) return fail(LM_E_STATE, "interval holds no step");
  lm::RunView& v = e->v;
  const lm::Dims& d = v.d;
  const size_t sp = d.spec_elems(), rf = d.rowfield_elems(), nn = (size_t)d.N * d.N;
  const double T = double(e->n - e->n_tau) * e->dt;
  const lm::StreamDrain drain{v.stream};
  cplx<double>* IC = e->at<cplx<double>>(e->IC);
  e->ic_current = false;  // its buffer takes the outputs' transforms
  double* OUT = e->at<double>(e->OUT);
  lm::IoColInv J{};
  for (int q = 0; q < 4; ++q) {
    J.src[q] = e->at<cplx<double>>(e->Y()) + q * sp;
    J.src_f32[q] = 0;
    J.dst[q] = IC + q * rf;
  }
  LM_DISPATCH_N(d.N, lm::launch_io_col_inverse, v, J, 4);
  lm::IoRowInv K{};
  for (int p = 0; p < 2; ++p) {
    K.a[p] = IC + (2 * p) * rf;
    K.b[p] = IC + (2 * p + 1) * rf;
    K.oa[p] = OUT + (2 * p) * nn;
    K.ob[p] = OUT + (2 * p + 1) * nn;
    K.sa[p] = (p == 0) ? 1.0 : 1.0 / T;  // zeta itself, then g~ / T; P_x / T, P_y / T
    K.sb[p] = 1.0 / T;
  }
  LM_DISPATCH_N(d.N, lm::launch_io_row_inverse, v, K, 2);
  const size_t plane = nn * sizeof(double);
  lm::SetRanges R;
  R.add(OUT + 4 * nn, plane, e->at<double>(e->SLf[e->cur]));
  R.add(OUT + 5 * nn, plane, e->at<double>(e->SLx[e->cur]));
  R.add(OUT + 6 * nn, plane, e->at<double>(e->SLy[e->cur]));
  lm::launch_set_ranges(v.stream, R);
  lm_status st;
  if ((st = check_launch()) != LM_OK) return st;
  HIP_TRY(hipStreamSynchronize(v.stream));
  e->T = T;
  e->has_out = true;
  e->in_interval = false;
  if (T_out) *T_out = T;
  return LM_OK;
}

lm_status lm_e2d_read(lm_e2d* e, int32_t kind, double* out, int on_device) {
  if (!e || !out) return fail(LM_E_ARG, "null argument");
  if (kind < LM_E2D_ZETA || kind > LM_E2D_SL_ETA_Y) return fail(LM_E_ARG, "unknown kind");
  if (!e->has_out) return fail(LM_E_STATE, "no closed interval");
  const lm::StreamDrain drain{e->v.stream};  // the caller's buffer is written before any return
  const size_t nn = (size_t)e->v.d.N * e->v.d.N;
  HIP_TRY(hipMemcpyAsync(out, e->at<double>(e->OUT) + kind * nn, nn * sizeof(double),
                         on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, e->v.stream));
  HIP_TRY(hipStreamSynchronize(e->v.stream));
  return LM_OK;
}

lm_status lm_e2d_destroy(lm_e2d* e) {
  if (!e) return LM_OK;
  hipError_t err = hipStreamSynchronize(e->v.stream);
  (void)hipFree(e->v.slab);
  delete e;
  if (err != hipSuccess) return fail(LM_E_HIP, std::string("hipStreamSynchronize: ") + hipGetErrorString(err));
  return LM_OK;
}

}  // extern "C"
