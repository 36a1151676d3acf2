// Definitions of the per-N launchers declared in launch.hpp.
#pragma once

#include <type_traits>
#include <vector>

#include "euler2d_step.hpp"
#include "io_kernels.hpp"
#include "launch.hpp"
#include "step_kernels.hpp"

namespace lm {

// does nothing; used to separate timed launches
template <int N>
__global__ void k_drain() {}

template <int N>
dim3 row_grid(int tasks) {
  return dim3(N / RowGeo<N>::RPB, tasks);
}
// the cooperative rows passes: one block per group of WR rows
template <typename T, int N>
dim3 coop_grid() {
  return dim3(N / CoopGeo<T, N>::WR);
}
template <int N, int W = 0>
dim3 col_grid(const Dims& d, int groups) {
  constexpr int C = col_tile<N, W>();
  return dim3((d.NKX + C - 1) / C, groups);
}
template <int N, int W = 0>
dim3 col_block() {
  return dim3(col_threads<N, W>());
}

// calls go(std::integral_constant<int, W>) with the schedule's tile width W
// (the default width if that one is not usable for this N and precision)
template <typename T, int N, typename F>
void with_tile(int tile, F&& go) {
  constexpr int cb = (int)sizeof(cplx<T>);
  if constexpr (col_tile_usable(N, -1, cb)) {
    if (tile < 0) return go(std::integral_constant<int, -1>{});
  }
  if constexpr (col_tile_usable(N, 1, cb)) {
    if (tile > 0) return go(std::integral_constant<int, 1>{});
  }
  go(std::integral_constant<int, 0>{});
}

// which column groups a launch carries: slots [first, first + count) of one stage
// (stage < 0: the prologue), ys the stage-value buffer that holds their stage's
// input (the buffers are flipped by the caller once per stage)
struct ColPart {
  int stage = 0, first = 0, count = 0, ys = 0;
};

template <typename T>
ColArgs<T> col_args(RunView& r, const ColPart& c, int tiles) {
  cplx<T>* Ys[2] = {(cplx<T>*)r.at(r.L.Ys0), (cplx<T>*)r.at(r.L.Ys1)};
  const int stage = c.stage;
  ColArgs<T> a;
  a.stage = stage;
  a.slot0 = c.first;
  a.nslot = c.count > 0 ? c.count : 1;
  a.cols = (c.count * tiles + 7) / 8 * 8;
  // time of the stage input this launch prepares: the current one in the
  // prologue, else the next stage's (c = 1/2, 1/2, 1, then the next step's 0)
  a.t_next = (double(r.n) + (stage < 0 ? 0.0 : (stage <= 1 ? 0.5 : 1.0))) * r.ph.dt;
  a.Ys_in = Ys[c.ys];
  a.Ys_out = (stage < 0) ? Ys[c.ys] : Ys[c.ys ^ 1];
  return a;
}

// one merged launch (small grids): A, dynamics and strategy-1 rows, or B, strategy-2
// rows, at time s since the interval start (rows set), and column groups
template <typename T, int N, bool B>
void launch_merged(RunView& r, bool rows, double s, const ColPart& c, hipStream_t st) {
  const StepPtrs<T> P = step_ptrs<T>(r);
  with_tile<T, N>(r.sched.tile, [&](auto w) {
    constexpr int W = decltype(w)::value;
    using S = typename std::conditional<B, StageB<T, N, W>, StageA<T, N, W>>::type;
    const ColArgs<T> a = col_args<T>(r, c, S::TILES);
    const int nr = rows ? S::ROWS : 0;
    const dim3 g(a.cols + nr), b(S::THREADS);
    if constexpr (B) hipLaunchKernelGGL((k_stage_b<T, N, W>), g, b, 0, st, P, r.ph, s, a, nr, r.sched.remap);
    else hipLaunchKernelGGL((k_stage_a<T, N, W>), g, b, 0, st, P, r.ph, s, a, nr, r.sched.remap);
  });
}

// column groups alone
template <typename T, int N>
void launch_columns_part(RunView& r, int stage, int first, int count, hipStream_t st) {
  const ColPart c{stage, first, count, r.ys_cur};
  if constexpr (stage_merged<T, N>()) {
    launch_merged<T, N, true>(r, false, 0.0, c, st);
  } else {
    const StepPtrs<T> P = step_ptrs<T>(r);
    with_tile<T, N>(r.sched.tile, [&](auto w) {
      constexpr int W = decltype(w)::value;
      const dim3 g = col_grid<N, W>(r.d, count), b(col_threads<N, W>());
      hipLaunchKernelGGL((k_columns<T, N, W>), g, b, 0, st, P, r.ph, col_args<T>(r, c, g.x), r.sched.remap);
    });
  }
}

template <typename T, int N>
void launch_columns_t(RunView& r, int stage) {
  launch_columns_part<T, N>(r, stage, 0, col_groups(r.ph), r.stream);
  if (stage >= 0) r.ys_cur ^= 1;
}

// the rows pass of the dynamics and strategy 1 alone
template <typename T, int N>
void launch_rows_dyn(RunView& r, double sval, hipStream_t st) {
  const dim3 g = coop_grid<T, N>(), b(DynGeo<T, N>::THREADS);
  if (r.ph.gen) {
    hipLaunchKernelGGL((k_rows_dyn<T, N, true>), g, b, 0, st, step_ptrs<T>(r), r.ph, sval, r.sched.remap);
  } else if constexpr (stage_merged<T, N>()) {
    launch_merged<T, N, false>(r, true, sval, ColPart{}, st);
  } else {
    hipLaunchKernelGGL((k_rows_dyn<T, N, false>), g, b, 0, st, step_ptrs<T>(r), r.ph, sval, r.sched.remap);
  }
}

// the momentum rows, when requested
template <typename T, int N>
void launch_rows_mom(RunView& r, double sval) {
  if (!r.mom) return;
  const StepPtrs<T> P = step_ptrs<T>(r);
  const dim3 g = coop_grid<T, N>(), b(MomGeo<T, N>::THREADS);
  if (r.cubic) hipLaunchKernelGGL((k_rows_mom<T, N, true>), g, b, 0, r.stream, P, sval, r.sched.remap);
  else hipLaunchKernelGGL((k_rows_mom<T, N, false>), g, b, 0, r.stream, P, sval, r.sched.remap);
}

// the rows pass of strategy 2 alone
template <typename T, int N>
void launch_rows_rhs(RunView& r, double sval) {
  const dim3 g = coop_grid<T, N>(), b(r.cubic ? RhsGeo<T, N>::CUB_THREADS : RhsGeo<T, N>::THREADS);
  if (r.cubic) {
    hipLaunchKernelGGL((k_rows_rhs<T, N, true>), g, b, 0, r.stream, step_ptrs<T>(r), sval, r.sched.remap);
  } else if constexpr (stage_merged<T, N>()) {
    launch_merged<T, N, true>(r, true, sval, ColPart{}, r.stream);
  } else {
    hipLaunchKernelGGL((k_rows_rhs<T, N, false>), g, b, 0, r.stream, step_ptrs<T>(r), sval, r.sched.remap);
  }
}

// Two-stream form of the steps.  Per stage the dependencies are
//   rows_dyn(i)  <- every column group of stage i-1 but those of strategy 2 (their
//                   outputs), rows_rhs(i-1) (it reads the physical fields rows_dyn
//                   rewrites) and the mean column groups of stage i-1 (they read
//                   the row spectra rows_dyn rewrites, and the stage values that
//                   the dynamics groups of stage i overwrite),
//   rows_rhs(i)  <- rows_dyn(i) and the mean column groups of stage i-1,
//   dynamics column groups(i) <- rows_dyn(i),  mean column groups(i) <- rows_dyn(i), rows_rhs(i),
// and no pass writes what a pass it may overlap with reads.  The auxiliary
// stream carries rows_dyn and the dynamics groups, the run's stream rows_rhs
// and the mean groups, so the dynamics groups overlap rows_rhs and the mean
// groups.  Same kernels, same arguments, same results as the one-stream form.
template <typename T, int N>
hipError_t launch_steps_2s(RunView& r, int nsteps) {
  static const double c[4] = {0.0, 0.5, 0.5, 1.0};
  const int nd = col_dyn_groups(r.ph), nm = col_groups(r.ph) - nd;
  hipEvent_t fork = r.ev[0], dyn = r.ev[1], rhs = r.ev[2], join = r.ev[3];
  hipError_t e = hipEventRecord(fork, r.stream);  // aux starts after everything queued so far
  if (e == hipSuccess) e = hipStreamWaitEvent(r.aux, fork, 0);
  for (int s = 0; s < nsteps && e == hipSuccess; ++s) {
    for (int stage = 0; stage < 4 && e == hipSuccess; ++stage) {
      const double sval = (double(r.n - r.n_tau) + c[stage]) * r.ph.dt;
      // the previous stage's run-stream work: rows_rhs reads the physical
      // fields rows_dyn rewrites, and the mean groups read the stage values the
      // next dynamics groups overwrite
      if (s + stage > 0) e = hipStreamWaitEvent(r.aux, rhs, 0);
      if (e != hipSuccess) break;
      launch_rows_dyn<T, N>(r, sval, r.aux);
      e = hipEventRecord(dyn, r.aux);
      launch_columns_part<T, N>(r, stage, 0, nd, r.aux);
      if (e == hipSuccess) e = hipStreamWaitEvent(r.stream, dyn, 0);
      if (e != hipSuccess) break;
      launch_rows_rhs<T, N>(r, sval);  // on the run's stream
      launch_rows_mom<T, N>(r, sval);
      launch_columns_part<T, N>(r, stage, nd, nm, r.stream);
      e = hipEventRecord(rhs, r.stream);
      r.ys_cur ^= 1;
    }
    r.n += 1;
  }
  // the run's stream resumes after the auxiliary stream's last work
  const hipError_t e2 = hipEventRecord(join, r.aux);
  const hipError_t e3 = (e2 == hipSuccess) ? hipStreamWaitEvent(r.stream, join, 0) : e2;
  return e != hipSuccess ? e : e3;
}

// One stream.  Small grids: launches A and B of every stage (k_stage_a, k_stage_b),
// the strategy-2 column groups of the last stage at the end; the rows of other
// averaged fields than (h, zeta) and of cubic gathers are kernels of their own, and
// such runs take the passes one by one, as large grids do.  Every launch goes out
// through timed(i, f): i = 0 the dynamics' and strategy 1's rows (launch A), 1 the
// rows of strategy 2 (launch B, and the momentum rows), 2 columns alone.
template <typename T, int N, typename F>
void launch_steps_through(RunView& r, int nsteps, F&& timed) {
  static const double c[4] = {0.0, 0.5, 0.5, 1.0};
  const int n1 = col_first_groups(r.ph), n2 = col_second_groups(r.ph);
  const bool merged = stage_merged<T, N>() && !r.ph.gen && !r.cubic;
  ColPart second;  // the strategy-2 column groups still to be launched
  for (int st = 0; st < nsteps; ++st) {
    for (int stage = 0; stage < 4; ++stage) {
      // time since the interval start, from integers
      const double sval = (double(r.n - r.n_tau) + c[stage]) * r.ph.dt;
      if constexpr (stage_merged<T, N>()) {
        if (merged) {
          timed(0, [&] { launch_merged<T, N, false>(r, true, sval, second, r.stream); });
          timed(1, [&] {
            launch_merged<T, N, true>(r, true, sval, ColPart{stage, 0, n1, r.ys_cur}, r.stream);
            launch_rows_mom<T, N>(r, sval);
          });
          second = ColPart{stage, n1, n2, r.ys_cur};
          r.ys_cur ^= 1;
          continue;
        }
      }
      timed(0, [&] { launch_rows_dyn<T, N>(r, sval, r.stream); });
      timed(1, [&] {
        launch_rows_rhs<T, N>(r, sval);
        launch_rows_mom<T, N>(r, sval);
      });
      timed(2, [&] { launch_columns_t<T, N>(r, stage); });
    }
    r.n += 1;
  }
  if constexpr (stage_merged<T, N>()) {
    if (second.count) timed(2, [&] { launch_merged<T, N, true>(r, false, 0.0, second, r.stream); });
  }
}

template <typename T, int N>
void launch_steps_t(RunView& r, int nsteps) {
  if (r.sched.streams == 2 && r.aux && nsteps > 0) {
    (void)launch_steps_2s<T, N>(r, nsteps);  // launch errors surface through hipGetLastError
    return;
  }
  launch_steps_through<T, N>(r, nsteps, [](int, auto&& f) { f(); });
}

// The one-stream launches of launch_steps_t, each bracketed by a pair of events on
// the run's stream; nothing synchronises until all steps are enqueued, so the
// kernels run back to back.  The durations are accumulated into ms[0..2].
template <typename T, int N>
hipError_t launch_steps_profiled_t(RunView& r, int nsteps, double* ms) {
  const int nev = (nsteps * 4 * 3 + 1) * 2;
  std::vector<hipEvent_t> ev(nev);
  std::vector<int> kind;  // of each pair
  kind.reserve(nev / 2);
  hipError_t err = hipSuccess;
  int made = 0;
  // device-scope markers: no system-scope cache release around every launch
  for (; made < nev && err == hipSuccess; ++made) err = hipEventCreateWithFlags(&ev[made], hipEventDisableSystemFence);
  if (err != hipSuccess) {
    for (int i = 0; i < made - 1; ++i) (void)hipEventDestroy(ev[i]);
    return err;
  }
  launch_steps_through<T, N>(r, nsteps, [&](int i, auto&& f) {
    // an empty kernel between one kernel's end marker and the next one's start
    // marker absorbs the work done at kernel boundaries, so each interval covers
    // one kernel's execution only
    const int e = 2 * (int)kind.size();
    kind.push_back(i);
    (void)hipEventRecord(ev[e], r.stream);
    f();
    (void)hipEventRecord(ev[e + 1], r.stream);
    hipLaunchKernelGGL(k_drain<N>, dim3(1), dim3(64), 0, r.stream);
  });
  if (!kind.empty()) err = hipEventSynchronize(ev[2 * kind.size() - 1]);
  for (size_t i = 0; i < kind.size() && err == hipSuccess; ++i) {
    float t = 0.f;
    err = hipEventElapsedTime(&t, ev[2 * i], ev[2 * i + 1]);
    ms[kind[i]] += t;
  }
  for (auto& x : ev) (void)hipEventDestroy(x);
  return err;
}

template <int N>
hipError_t launch_steps_profiled(RunView& r, int nsteps, double* ms) {
  if (r.fp32) return launch_steps_profiled_t<float, N>(r, nsteps, ms);
  return launch_steps_profiled_t<double, N>(r, nsteps, ms);
}

// one RK4 step of every run of one (N, precision) group, all runs' blocks in each
// launch: up to batch_merged_runs() runs the launches of launch_steps_t, beyond them
// the passes one by one, each a kernel of its own
template <typename T, int N>
void launch_batch_step_t(hipStream_t st, const RunDesc<T>* desc, int nruns, bool cubic, bool mom, bool gen,
                         const Sched& sc) {
  Phys gp{};
  gp.mom = mom;
  gp.gen = gen;
  const int rm = sc.remap;
  dim3 gr = coop_grid<T, N>();  // one pass per launch: blockIdx.z selects the run
  gr.z = nruns;
  const dim3 b1(DynGeo<T, N>::THREADS), b2(cubic ? RhsGeo<T, N>::CUB_THREADS : RhsGeo<T, N>::THREADS), bm(MomGeo<T, N>::THREADS);
  auto launch_mom = [&](int stage) {
    if (!mom) return;
    if (cubic) hipLaunchKernelGGL((k_rows_mom_b<T, N, true>), gr, bm, 0, st, desc, stage, rm);
    else hipLaunchKernelGGL((k_rows_mom_b<T, N, false>), gr, bm, 0, st, desc, stage, rm);
  };
  with_tile<T, N>(batch_tile<T, N>(nruns, sc.tile), [&](auto w) {
    constexpr int W = decltype(w)::value;
    if constexpr (stage_merged<T, N>()) {
      if (nruns <= batch_merged_runs<T, N>()) {
        using A = StageA<T, N, W>;
        using B = StageB<T, N, W>;
        const int n1 = col_first_groups(gp), n2 = col_second_groups(gp);
        auto launch_ab = [&](bool b, bool rows, int stage, int cstage, int first, int count) {
          const int nc = (count * A::TILES * nruns + 7) / 8 * 8, nr = rows ? A::ROWS * nruns : 0, ns = count > 0 ? count : 1;
          if (b) hipLaunchKernelGGL((k_stage_b_b<T, N, W>), dim3(nc + nr), dim3(B::THREADS), 0, st, desc, nruns, stage,
                                    cstage, first, ns, nc, nr, rm);
          else hipLaunchKernelGGL((k_stage_a_b<T, N, W>), dim3(nc + nr), dim3(A::THREADS), 0, st, desc, nruns, stage,
                                  cstage, first, ns, nc, nr, rm);
        };
        if (!gen && !cubic) {
          for (int stage = 0; stage < 4; ++stage) {
            launch_ab(false, true, stage, stage - 1, n1, stage > 0 ? n2 : 0);
            launch_ab(true, true, stage, stage, 0, n1);
            launch_mom(stage);
          }
          launch_ab(true, false, 0, 3, n1, n2);
          return;
        }
        for (int stage = 0; stage < 4; ++stage) {
          if (gen) hipLaunchKernelGGL((k_rows_dyn_b<T, N, true>), gr, b1, 0, st, desc, stage, rm);
          else launch_ab(false, true, stage, 0, 0, 0);
          if (cubic) hipLaunchKernelGGL((k_rows_rhs_b<T, N, true>), gr, b2, 0, st, desc, stage, rm);
          else launch_ab(true, true, stage, 0, 0, 0);
          launch_mom(stage);
          launch_ab(true, false, 0, stage, 0, n1 + n2);
        }
        return;
      }
    }
    for (int stage = 0; stage < 4; ++stage) {
      if (gen) hipLaunchKernelGGL((k_rows_dyn_b<T, N, true>), gr, b1, 0, st, desc, stage, rm);
      else hipLaunchKernelGGL((k_rows_dyn_b<T, N, false>), gr, b1, 0, st, desc, stage, rm);
      if (cubic) hipLaunchKernelGGL((k_rows_rhs_b<T, N, true>), gr, b2, 0, st, desc, stage, rm);
      else hipLaunchKernelGGL((k_rows_rhs_b<T, N, false>), gr, b2, 0, st, desc, stage, rm);
      launch_mom(stage);
      dim3 g3 = col_grid<N, W>(Dims::make(N), col_groups(gp));
      g3.z = nruns;
      hipLaunchKernelGGL((k_columns_b<T, N, W>), g3, dim3(col_threads<N, W>()), 0, st, desc, stage, rm);
    }
  });
}

template <int N>
void launch_batch_step(hipStream_t st, const void* desc, int nruns, bool fp32, bool cubic, bool mom, bool gen,
                       const Sched& sc) {
  if (fp32) launch_batch_step_t<float, N>(st, (const RunDesc<float>*)desc, nruns, cubic, mom, gen, sc);
  else launch_batch_step_t<double, N>(st, (const RunDesc<double>*)desc, nruns, cubic, mom, gen, sc);
}

template <int N>
void launch_steps(RunView& r, int nsteps) {
  if (r.fp32) launch_steps_t<float, N>(r, nsteps);
  else launch_steps_t<double, N>(r, nsteps);
}

template <int N>
void launch_prologue(RunView& r) {
  if (r.fp32) launch_columns_t<float, N>(r, -1);
  else launch_columns_t<double, N>(r, -1);
}

template <int N>
void launch_prologue_dyn(RunView& r) {
  if (r.fp32) launch_columns_part<float, N>(r, -1, 0, 3, r.stream);
  else launch_columns_part<double, N>(r, -1, 0, 3, r.stream);
}

template <int N>
void launch_io_col_inverse(RunView& r, const IoColInv& J, int count) {
  hipLaunchKernelGGL((k_io_col_inverse<N>), col_grid<N>(r.d, count), col_block<N>(), 0, r.stream, J, r.d,
                     (const cplx<double>*)r.at(r.L.tw64));
}
template <int N>
void launch_io_row_inverse(RunView& r, const IoRowInv& J, int count) {
  hipLaunchKernelGGL((k_io_row_inverse<N>), row_grid<N>(count), dim3(64 * ROW_WAVES), 0, r.stream, J, r.d,
                     (const cplx<double>*)r.at(r.L.tw64));
}
template <int N>
void launch_io_row_forward(RunView& r, const IoRowFwd& J, int count) {
  hipLaunchKernelGGL((k_io_row_forward<N>), row_grid<N>(count), dim3(64 * ROW_WAVES), 0, r.stream, J, r.d,
                     (const cplx<double>*)r.at(r.L.tw64));
}
template <int N>
void launch_io_col_forward(RunView& r, const IoColFwd& J, int count) {
  hipLaunchKernelGGL((k_io_col_forward<N>), col_grid<N>(r.d, count), col_block<N>(), 0, r.stream, J, r.d,
                     (const cplx<double>*)r.at(r.L.tw64));
}

}  // namespace lm

// The per-precision step launchers (and with them every time-stepping kernel)
// are instantiated in inst_<N>_f32.hip and inst_<N>_f64.hip, the dispatchers
// and the float64 boundary launchers in inst_<N>.hip: three translation units
// per grid size compile in parallel.
#define LM_INSTANTIATE_T(T, N)                                                                           \
  namespace lm {                                                                                         \
  template void launch_steps_t<T, N>(RunView&, int);                                                     \
  template hipError_t launch_steps_profiled_t<T, N>(RunView&, int, double*);                             \
  template void launch_columns_t<T, N>(RunView&, int);                                                   \
  template void launch_columns_part<T, N>(RunView&, int, int, int, hipStream_t);                         \
  template void launch_batch_step_t<T, N>(hipStream_t, const RunDesc<T>*, int, bool, bool, bool, const Sched&); \
  }

#define LM_EXTERN_T(T, N)                                                                                       \
  namespace lm {                                                                                                \
  extern template void launch_steps_t<T, N>(RunView&, int);                                                     \
  extern template hipError_t launch_steps_profiled_t<T, N>(RunView&, int, double*);                             \
  extern template void launch_columns_t<T, N>(RunView&, int);                                                   \
  extern template void launch_columns_part<T, N>(RunView&, int, int, int, hipStream_t);                         \
  extern template void launch_batch_step_t<T, N>(hipStream_t, const RunDesc<T>*, int, bool, bool, bool, const Sched&); \
  }

#define LM_INSTANTIATE(N)                                                                             \
  LM_EXTERN_T(float, N)                                                                               \
  LM_EXTERN_T(double, N)                                                                              \
  namespace lm {                                                                                      \
  template void launch_steps<N>(RunView&, int);                                                       \
  template void launch_batch_step<N>(hipStream_t, const void*, int, bool, bool, bool, bool, const Sched&); \
  template hipError_t launch_steps_profiled<N>(RunView&, int, double*);                               \
  template void launch_prologue<N>(RunView&);                                                         \
  template void launch_prologue_dyn<N>(RunView&);                                                     \
  template void launch_io_row_forward<N>(RunView&, const IoRowFwd&, int);                             \
  template void launch_io_col_forward<N>(RunView&, const IoColFwd&, int);                             \
  template void launch_io_col_inverse<N>(RunView&, const IoColInv&, int);                             \
  template void launch_io_row_inverse<N>(RunView&, const IoRowInv&, int);                             \
  template void launch_e2d_rows<N>(hipStream_t, const E2DPtrs&, double, int, int);                    \
  template void launch_e2d_columns<N>(hipStream_t, const E2DPtrs&, int, const E2DSl*);                \
  template void launch_e2d_sl<N>(hipStream_t, const E2DSl&);                                          \
  }
