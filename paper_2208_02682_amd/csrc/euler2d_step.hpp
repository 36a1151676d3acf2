// Passes of the two-dimensional incompressible flow (section 4.1) with strategy 1
// pseudospectral (eqs. (4.1), (3.9)) and semi-Lagrangian (appendix B), float64.
//
// A Heun stage is two launches, as the shallow-water stage's passes:
//   rows     u = -psi_y, v = psi_x, zeta and the gradients of zeta, g~, P_x, P_y by
//            inverse row transforms; the products u.grad zeta, zeta - u.grad g~,
//            s u - u.grad P_x, s v - u.grad P_y; forward row transforms;
//   columns  forward column transforms, Heun's update of the four spectral fields,
//            and the inverse column transforms of the next input: psi, zeta, g~, P
//            and their y derivatives (x derivatives are taken in the row pass).
// The semi-Lagrangian update of a step needs u, v and zeta at its end, which the
// next step's first rows pass forms anyway: its blocks ride in the column launch
// after that pass, and the last step of a call gets a rows pass of its own.  Four
// launches a step (instead of twenty, one per transform direction and product:
// 128^2, us per step 68 -> 27, launch-bound before).
#pragma once

#include "euler2d_sl.hpp"
#include "launch.hpp"
#include "step_kernels.hpp"

namespace lm {

// column-pass outputs
enum E2DInter : int { EI_PSI = 0, EI_PSI_Y, EI_Z, EI_Z_Y, EI_G, EI_G_Y, EI_PX, EI_PX_Y, EI_PY, EI_PY_Y, NEI = 10 };
static_assert(NEI == E2D_NIC, "intermediates");

// ---------------------------------------------------------------------------
// rows: six waves per group of rows, one inverse transform each: (u, v), zeta and
// the four gradients; waves 2 and 4 forward-transform the pairs of products
// (zeta, g~) and (P_x, P_y), waves 3 and 5 handing them theirs.
// ---------------------------------------------------------------------------
template <int N>
struct E2DRowGeo : CoopGeo<double, N> {
  using G = CoopGeo<double, N>;
  static constexpr int WAVES = 6, THREADS = 64 * WAVES;
  static constexpr int BUFS = G::SPLIT ? 7 : 6;  // split: v gets a buffer of its own
  static constexpr int LDS = BUFS * G::WR * G::RB;
};

template <int N>
__global__ void __launch_bounds__((E2DRowGeo<N>::THREADS), 2) k_e2d_rows(E2DPtrs P, double s, int store, int products) {
  using T = double;
  using G = E2DRowGeo<N>;
  constexpr int E = G::E, NT = G::NT, WR = G::WR, RB = G::RB;
  constexpr bool SPLIT = G::SPLIT;
  __shared__ __align__(16) T lds[G::LDS];
  int rowblock, unused, zz;
  xcd_split(gridDim.x, 1, rowblock, unused, zz, 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // the wave's role
  const int lane = threadIdx.x % 64;
  const int g = lane / NT, t = lane % NT;
  const int y = rowblock * WR + g;
  auto buf = [&](int i) { return lds + (i * WR + g) * RB; };
  const SharedPair<T, SPLIT> UV{buf(0), buf(SPLIT ? 6 : 0)};
  T* mine = buf(w);
  constexpr Dims d = dims_of<N>();
  constexpr size_t rf = d.rowfield_elems();
  const unsigned row = (unsigned)y * (unsigned)d.NKXP;
  const unsigned at = (unsigned)(y * N + t);

  cplx<T> z[E];
  if (w >= 2 && !products) {
    __syncthreads();
    return;
  }
  if (w == 0) {
    // psi_y + i psi_x: (u, v) = (-re, im)
    load_pair<T, N, false, true>(z, P.IC + EI_PSI_Y * rf, P.IC + EI_PSI * rf, row, t);
  } else if (w == 1) {
    load_pair<T, N, false, false>(z, P.IC + EI_Z * rf, P.IC + EI_Z * rf, row, t);
  } else {
    const cplx<T>* A = P.IC + (EI_Z + 2 * (w - 2)) * rf;
    load_pair<T, N, true, false>(z, A, A + rf, row, t);
  }
  inverse_row<T, N, SPLIT>(z, mine, t, P.tw);
  if (w == 0) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      z[e] = {P.U0 - z[e].x, P.V0 + z[e].y};
      UV.put(t + NT * e, z[e]);
      if (store) {
        put32(P.PH + NT * e, at, z[e].x);
        put32(P.PH + (size_t)N * N + NT * e, at, z[e].y);
      }
    }
  } else if (w == 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      mine[t + NT * e] = z[e].x;
      if (store) put32(P.PH + (size_t)2 * N * N + NT * e, at, z[e].x);
    }
  }
  __syncthreads();
  if (w < 2 || !products) {
    if (products) __syncthreads();
    return;
  }
  const T* zeta = buf(1);
  T* pair = buf(w & ~1);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = t + NT * e;
    const cplx<T> uv = UV.get(x);
    const T adv = uv.x * z[e].x + uv.y * z[e].y;
    // the vorticity's product keeps its sign until the column pass
    const T f = (w == 3) ? zeta[x] : (w == 4) ? s * uv.x : s * uv.y;
    z[e].x = (w == 2) ? adv : f - adv;
    if (e % 4 == 3) sched_fence();
  }
  if (w & 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) pair[t + NT * e] = z[e].x;
  }
  __syncthreads();
  if (w & 1) return;
#pragma unroll
  for (int e = 0; e < E; ++e) z[e].y = mine[t + NT * e];
  xsync<NT>();
  cplx<T>* OA = P.RS + (w - 2) * rf;
  forward_row<T, N, SPLIT>(z, mine, t, P.tw, OA, OA + rf, row);
}

// ---------------------------------------------------------------------------
// columns: groups 0..3 = zeta, g~, P_x, P_y, group 4 = psi (from zeta's update,
// formed again: a second forward transform costs less than a block with twice the
// inverse ones).  stage 0: K1 = R, next input Y + dt K1; stage 1: Yn = Y + dt/2
// (K1 + R), the next input; stage < 0: the current state's transforms only.  The
// new state goes to a buffer of its own, so that groups 0 and 4 read the same old
// one.  Narrow tiles: five groups alone fill the chip poorly (512^2, 8 columns per
// block 26 us, 4 columns and psi apart 17).  Blocks before the column tiles carry
// the semi-Lagrangian update.
// ---------------------------------------------------------------------------
constexpr int E2D_W = -1;  // tile width
// both inverse transforms side by side up to 512^2, one more size than the columns of
// a run: with this few blocks latency bounds them (512^2, one after the other, an
// interval of 15 steps 1061 -> 1204 us)
template <typename T, int N, int C>
__host__ __device__ constexpr bool e2d_dual() {
  return fft_E<N>() <= 12 && 2 * C * col_buf(N) * sizeof(cplx<T>) <= 80 * 1024;
}
template <int N>
__global__ void __launch_bounds__((col_threads<N, E2D_W>()), 1)
    k_e2d_columns(E2DPtrs P, int stage, int sl_blocks, E2DSl sl) {
  using T = double;
  constexpr int C = col_tile<N, E2D_W>();
  constexpr int E = fft_E<N>();
  constexpr Dims d = dims_of<N>();
  constexpr size_t sp = d.spec_elems(), rf = d.rowfield_elems();
  constexpr int TILES = (d.NKX + C - 1) / C;
  __shared__ __align__(16) T lds[col_lds<T, N, C, e2d_dual<T, N, C>()>()];
  int b = blockIdx.x;
  if (b < sl_blocks) {
    sl_update<N>(sl, b * col_threads<N, E2D_W>() + (int)threadIdx.x);
    return;
  }
  b -= sl_blocks;
  const int group = b / TILES;
  const bool psi = group == 4;
  const int q = psi ? 0 : group;  // the state field
  const ColCtx<T, N, C> cx(lds, b % TILES);
  const cplx<T>* Y = P.Y + q * sp;
  cplx<T>* Yn = P.Yn + q * sp;
  cplx<T>* K1 = P.K1 + q * sp;

  cplx<T> S[E], k1[E], R[E];
  auto load = [&](int r) {
    const ColIdx<N> ix{cx.t, r};
    S[r] = k1[r] = {0.0, 0.0};
    if (ix.none()) return;
    const unsigned j = cx.ky0 + ix.lane();
    S[r] = at32(Y + ix.off(), j);
    if (stage == 1) k1[r] = at32(K1 + ix.off(), j);
  };
  // small grids: the state is in flight before the transform
  constexpr bool PRE = E <= 8;
  if constexpr (PRE) {
#pragma unroll
    for (int r = 0; r < E; ++r) load(r);
    sched_fence();
  }
  if (stage >= 0) column_forward<T, N, C>(cx, P.RS + q * rf, nullptr, P.tw, R);
  if constexpr (!PRE) {
#pragma unroll
    for (int r = 0; r < E; ++r) load(r);
  }
  const double sg = (q == 0) ? -1.0 : 1.0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const ColIdx<N> ix{cx.t, r};
    const bool keep = !ix.none() && ix.in() && cx.valid;
    if (stage >= 0 && keep) {
      const unsigned j = cx.ky0 + ix.lane();
      cplx<T> v = {sg * R[r].x, sg * R[r].y};
      if (cx.kx == 0 && ix.ky() == 0) v.y = 0.0;
      if (stage == 0) {
        if (!psi) put32(K1 + ix.off(), j, v);
        S[r] = {S[r].x + P.dt * v.x, S[r].y + P.dt * v.y};
      } else {
        S[r] = {S[r].x + 0.5 * P.dt * (k1[r].x + v.x), S[r].y + 0.5 * P.dt * (k1[r].y + v.y)};
        if (!psi) put32(Yn + ix.off(), j, S[r]);
      }
    }
    if (!keep) S[r] = {0.0, 0.0};
  }
  if (psi) {
    // psi = -zeta / |k|^2, its k = 0 mode zero
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const ColIdx<N> ix{cx.t, r};
      const double kx = cx.kx, ky = ix.none() ? 0 : ix.ky();
      const double k2 = kx * kx + ky * ky;
      const double inv = k2 > 0.0 ? 1.0 / k2 : 0.0;
      S[r] = {-S[r].x * inv, -S[r].y * inv};
    }
  }
  cplx<T>* out = P.IC + (psi ? EI_PSI : EI_Z + 2 * q) * rf;
  column_inverse<T, N, C, true, e2d_dual<T, N, C>()>(cx, S, out, out + rf, P.tw);
}

template <int N>
void launch_e2d_rows(hipStream_t st, const E2DPtrs& P, double s, int store, int products) {
  hipLaunchKernelGGL((k_e2d_rows<N>), dim3(N / E2DRowGeo<N>::WR), dim3(E2DRowGeo<N>::THREADS), 0, st, P, s, store,
                     products);
}
template <int N>
void launch_e2d_columns(hipStream_t st, const E2DPtrs& P, int stage, const E2DSl* sl) {
  constexpr int C = col_tile<N, E2D_W>(), TH = col_threads<N, E2D_W>(), TILES = (dims_of<N>().NKX + C - 1) / C;
  const int nsl = sl ? (N * N + TH - 1) / TH : 0;
  hipLaunchKernelGGL((k_e2d_columns<N>), dim3(5 * TILES + nsl), dim3(TH), 0, st, P, stage, nsl, sl ? *sl : E2DSl{});
}

}  // namespace lm
