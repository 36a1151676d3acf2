// A kernel launch that fails in lm_e2d_step: one launch after another is refused
// (by the stand-in runtime's launch call, overridden here), and the handle has to
// stay at the last step whose launches all went out.  Prints, per refused launch,
// the steps the handle counts then and after two more steps.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdio>
#include <vector>

#include "lagmean.h"

namespace {
int g_seen = 0, g_refuse = -1;  // launches since armed; the one refused
hipError_t g_err = hipSuccess;

int steps_of(double T, double dt) { return (int)std::lround(T / dt); }
}  // namespace

extern "C" hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shm, hipStream_t s) {
  static auto real = (hipError_t(*)(const void*, dim3, dim3, void**, size_t, hipStream_t))dlsym(RTLD_NEXT, "hipLaunchKernel");
  if (g_seen++ == g_refuse) return g_err = hipErrorInvalidConfiguration;
  return real(f, grid, block, args, shm, s);
}
extern "C" hipError_t hipGetLastError() {
  static auto real = (hipError_t(*)())dlsym(RTLD_NEXT, "hipGetLastError");
  const hipError_t e = g_err;
  g_err = hipSuccess;
  return e != hipSuccess ? e : real();
}

int main() {
  const double dt = 0.01;
  const lm_e2d_config cfg{64, dt, 0.0, 0.0, LM_INTERP_BILINEAR};
  const std::vector<double> zeta(64 * 64, 0.5);
  for (int profiled = 0; profiled < 2; ++profiled) {
    for (int refuse = 0;; ++refuse) {
      lm_e2d* e = nullptr;
      double T = 0.0, a, b;
      if (lm_e2d_create(&cfg, nullptr, &e) != LM_OK || lm_e2d_set_vorticity(e, zeta.data(), 0) != LM_OK ||
          lm_e2d_begin_interval(e) != LM_OK)
        return 1;
      g_seen = 0;
      g_refuse = refuse;
      const lm_status st = profiled ? lm_e2d_step_profiled(e, 3, &a, &b) : lm_e2d_step(e, 3);
      g_refuse = -1;
      if (st == LM_OK) {  // past the call's last launch
        lm_e2d_destroy(e);
        break;
      }
      const lm_status end = lm_e2d_end_interval(e, &T);  // refused while no step counts
      const int first = end == LM_OK ? steps_of(T, dt) : (end == LM_E_STATE ? 0 : -1);
      if (end == LM_OK && lm_e2d_begin_interval(e) != LM_OK) return 1;
      if (lm_e2d_step(e, 2) != LM_OK || lm_e2d_end_interval(e, &T) != LM_OK) return 1;
      std::printf("%d %d %d %d %d\n", profiled, refuse, (int)st, first, steps_of(T, dt));
      lm_e2d_destroy(e);
    }
  }
  return 0;
}
