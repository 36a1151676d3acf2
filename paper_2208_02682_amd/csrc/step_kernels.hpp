// Hot-path kernels of one RK4 stage (templated on the transform precision T and N).
//
// One stage of the coupled system is three passes (two launches on small grids,
// see stage_merged):
//
//  rows_dyn   per grid row: inverse row transforms of the column-pass outputs to
//             physical u, v, eta = h - H, zeta (zeta = dv/dx - du/dy); stores
//             them interleaved for the gathers; forms zeta v, zeta u,
//             K = (u^2+v^2)/2, eta u, eta v and strategy 1's right-hand sides
//               f - u.grad g-tilde                                   (eq. (4.1)) and
//               (t-tau) u - u.grad P  (inverse lift map, eq. (3.9) in P form)
//             and forward-transforms them along the row.
//
// The physical passes carry the depth anomaly eta = h - H instead of the total
// depth h, and the h accumulators of the three averages integrate eta; H is put
// back exactly where it enters (H u and H v in the flux divergence, H s in the
// accumulators, + H in the float64 outputs).  This is the same arithmetic as the
// total-depth form up to rounding (each average is linear in the averaged field
// and exact for constants) but keeps the full float32 precision for eta.
//  rows_rhs   per grid row: strategy 2's right-hand sides in physical space,
//               u(x+xi) - w - (w.grad) xi  for both components     (eq. (4.5a)),
//               w = xi/(t-tau), or u/2 at t = tau, and
//               f(x+xi) - w.grad g-bar, f in {h, zeta}             (eq. (4.5b)),
//             then forward row transforms.
//             u(x+xi) and f(x+xi) are periodic bilinear (or cubic) interpolants.
//  columns    per spectral column kx and prognostic field: forward column
//             transforms, masked spectral assembly of the right-hand side
//             (Coriolis, Bernoulli gradient, flux divergence, -nu8 |k|^8), the
//             classical RK4 update (FP64 for xi and P), and the inverse column
//             transforms of the next stage's input, ready for the next rows pass.
//
// Two real row fields share one complex transform (z = a + i b).
#pragma once

#include <type_traits>

#include "fft_core.hpp"
#include "col_tile.hpp"
#include "layout.hpp"
#include "step_args.hpp"

namespace lm {

constexpr int ROW_WAVES = 4;  // wavefronts per row-kernel block

// row kernels: one lane group of NT = N / E lanes per grid row
template <int N>
struct RowGeo {
  static constexpr int E = fft_E<N>(), NT = N / E;
  static constexpr int RPB = 64 * ROW_WAVES / NT;  // rows per block
  static constexpr int L = padded_len(N);           // LDS slots per row
  static_assert(RPB >= 1 && N % RPB == 0, "row geometry");
};

// group index (uniform per wavefront when a group spans whole wavefronts)
template <int NT>
__device__ __forceinline__ int row_group() {
  if constexpr (NT >= 64) return __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
  else return threadIdx.x / NT;
}

// the sizes of a compiled grid, as constants
template <int N>
__host__ __device__ constexpr Dims dims_of() { return Dims::make(N); }

template <int N, int W = 0>
__host__ __device__ constexpr int col_tile() { return col_tile_of(W); }
template <int N, int W = 0>
__host__ __device__ constexpr int col_threads() { return col_tile<N, W>() * (N / fft_E<N>()); }

// --------------------------------------------------------------------------
// row helpers
// --------------------------------------------------------------------------

// Element i of an array at a base that is uniform over the wavefront: the base
// stays in scalar registers and the lane's part is one 32-bit offset, shared by
// every array read at the same place (all arrays are far below 4 GiB).
template <typename X>
__device__ __forceinline__ X at32(const X* __restrict__ base, unsigned i) {
  return *reinterpret_cast<const X*>(reinterpret_cast<const char*>(base) + i * (unsigned)sizeof(X));
}
template <typename X>
__device__ __forceinline__ void put32(X* base, unsigned i, X v) {
  *reinterpret_cast<X*>(reinterpret_cast<char*>(base) + i * (unsigned)sizeof(X)) = v;
}

// Which coefficient |kx| = kk of a half spectrum (kx = 0..K) entry k = t + NT r of
// a full row takes, and how: entries 0..K as stored, N-K..N-1 (negative kx) the
// conjugate of N - k, none in between.  For most r one rule holds for every lane;
// then the place is a lane's offset (t, or NT - t for mirrored entries) plus a
// constant, which costs no address arithmetic.  Lanes without a coefficient read
// a clamped place and select zero, so that the unrolled loops have no branches.
template <int N>
struct HalfIdx {
  static constexpr int E = fft_E<N>(), NT = N / E, K = kcut<N>();
  int t, r;
  __device__ __forceinline__ bool all_lo() const { return NT * r + NT - 1 <= K; }
  __device__ __forceinline__ bool all_hi() const { return NT * r >= N - K; }
  __device__ __forceinline__ bool none() const { return NT * r > K && NT * r + NT - 1 < N - K; }
  __device__ __forceinline__ bool lo() const { return all_lo() || (!all_hi() && t + NT * r <= K); }
  __device__ __forceinline__ bool in() const { return all_lo() || all_hi() || t + NT * r <= K || t + NT * r >= N - K; }
  // kk = lane() + off()
  __device__ __forceinline__ int lane() const {
    if (all_lo()) return t;
    if (all_hi()) return NT - t;
    const int k = t + NT * r;
    return min(k <= K ? k : N - k, K);
  }
  __device__ __forceinline__ int off() const { return all_lo() ? NT * r : (all_hi() ? N - NT * (r + 1) : 0); }
  __device__ __forceinline__ bool zero() const { return r == 0 && t == 0; }
};

// entry k of the length-N spectrum of a' + i b' from the coefficients a, b of two
// real rows at kk (conjugated for negative kx, real at kx = 0)
template <typename T, int N>
__device__ __forceinline__ cplx<T> full_entry(const HalfIdx<N>& h, cplx<T> a, cplx<T> b) {
  if (h.r == 0) {
    const T sy = h.zero() ? T(0) : T(1);
    a.y *= sy;
    b.y *= sy;
  }
  const cplx<T> lo = {a.x - b.y, a.y + b.x}, hi = {a.x + b.y, b.x - a.y};
  if (h.all_lo()) return lo;
  if (h.all_hi()) return hi;
  const cplx<T> z = h.lo() ? lo : hi;
  return h.in() ? z : cplx<T>{T(0), T(0)};
}

// Build lane registers of the length-N spectrum Z = A' + i B' of two real rows
// from their half spectra (kx = 0..K), row .. row + K of the fields A and B.
// A' = i kx A if DXA (likewise B).  Index k = t + NT r.
template <typename T, int N, bool DXA, bool DXB>
__device__ __forceinline__ void load_pair(cplx<T> (&z)[fft_E<N>()], const cplx<T>* __restrict__ A,
                                          const cplx<T>* __restrict__ B, unsigned row, int t) {
  constexpr int E = fft_E<N>();
  sched_fence();
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const HalfIdx<N> h{t, r};
    if (h.none()) {
      z[r] = {T(0), T(0)};
      continue;
    }
    cplx<T> a = at32(A + h.off(), row + h.lane()), b = at32(B + h.off(), row + h.lane());
    const T kk = T(h.lane()) + T(h.off());
    if (DXA) a = {-kk * a.y, kk * a.x};
    if (DXB) b = {-kk * b.y, kk * b.x};
    z[r] = full_entry<T, N>(h, a, b);
  }
}

// spectrum of eta + i zeta from the column-pass outputs of h, v and i ky u: the
// zeta spectrum is i kx C_v - C_uy.  Same layout as load_pair.
template <typename T, int N>
__device__ __forceinline__ void load_depth_vorticity(cplx<T> (&z)[fft_E<N>()], const cplx<T>* __restrict__ Ch,
                                                     const cplx<T>* __restrict__ Cv,
                                                     const cplx<T>* __restrict__ Cuy, unsigned row, int t) {
  constexpr int E = fft_E<N>();
  sched_fence();
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const HalfIdx<N> h{t, r};
    if (h.none()) {
      z[r] = {T(0), T(0)};
      continue;
    }
    const unsigned i = row + h.lane();
    const cplx<T> a = at32(Ch + h.off(), i), cv = at32(Cv + h.off(), i), cu = at32(Cuy + h.off(), i);
    const T kk = T(h.lane()) + T(h.off());
    z[r] = full_entry<T, N>(h, a, cplx<T>{-kk * cv.y - cu.x, kk * cv.x - cu.y});
  }
}

// Inverse-transform a pair and leave lane values p[e] at x = t + NT e.
template <typename T, int N, bool SPLIT = false>
__device__ __forceinline__ void inverse_row(cplx<T> (&z)[fft_E<N>()], T* buf, int t,
                                            const cplx<T>* __restrict__ tw) {
  fft<T, N, fft_E<N>(), +1, true, SPLIT>(z, buf, t, tw);
  sched_fence();
}

// Forward-transform z = a + i b (lane values at x = t + NT e) and store the
// half spectra of a and b (kx = 0..K) to row .. row + K of the fields OA and OB
// (OB null: a alone).  The mirror entries Z(N - k) come through the buffer.
template <typename T, int N, bool SPLIT = false>
__device__ __forceinline__ void forward_row(cplx<T> (&z)[fft_E<N>()], T* buf, int t, const cplx<T>* __restrict__ tw,
                                            cplx<T>* __restrict__ OA, cplx<T>* __restrict__ OB, unsigned row) {
  constexpr int E = fft_E<N>(), NT = N / E, K = kcut<N>(), KR = (K + NT) / NT;
  fft<T, N, E, -1, SPLIT, SPLIT>(z, buf, t, tw);
  auto put = [&](int r, cplx<T> zk, cplx<T> zm) {
    put32(OA + NT * r, row + t, cplx<T>{T(0.5) * (zk.x + zm.x), T(0.5) * (zk.y - zm.y)});
    if (OB) put32(OB + NT * r, row + t, cplx<T>{T(0.5) * (zk.y + zm.y), T(-0.5) * (zk.x - zm.x)});
  };
  // the mirror of entry t + NT r: N - t - NT r, and 0 for entry 0
  auto mirror = [&](int r) -> LaneIdx {
    if (r == 0) return {t == 0 ? 0 : N - t, 0};
    return {NT - t, N - NT * (r + 1)};
  };
  if constexpr (!SPLIT) {
    const cplx<T>* cb = reinterpret_cast<const cplx<T>*>(buf);
#pragma unroll
    for (int r = 0; r < KR; ++r) {
      if (t + NT * r > K) break;
      put(r, cb[pidx(LaneIdx{t, NT * r})], cb[pidx(mirror(r))]);
    }
  } else {
    cplx<T> m[KR];
#pragma unroll
    for (int e = 0; e < E; ++e) buf[pidx(LaneIdx{t, NT * e})] = z[e].x;
    xsync<NT>();
#pragma unroll
    for (int r = 0; r < KR; ++r) m[r].x = buf[pidx(mirror(r))];
    xsync<NT>();
#pragma unroll
    for (int e = 0; e < E; ++e) buf[pidx(LaneIdx{t, NT * e})] = z[e].y;
    xsync<NT>();
#pragma unroll
    for (int r = 0; r < KR; ++r) m[r].y = buf[pidx(mirror(r))];
#pragma unroll
    for (int r = 0; r < KR; ++r)
      if (t + NT * r <= K) put(r, z[r], m[r]);
  }
  xsync<NT>();
  sched_fence();
}

// i in [-N, 2N) to [0, N): a mask for powers of two, two selects otherwise
template <int N>
__device__ __forceinline__ int wrap2N(int i) {
  if constexpr ((N & (N - 1)) == 0) {
    return i & (N - 1);
  } else {
    i = (i < 0) ? i + N : i;
    return (i >= N) ? i - N : i;
  }
}

// The cell offset floor(o) of a gather (o = displacement / dx) taken
// periodically into [0, N): a finite displacement of any size wraps around the
// torus.  Offsets beyond 2^30 cells and NaN land on cell 0 (their weights are
// non-finite, which the end-of-interval check reports).
template <int N, typename T>
__device__ __forceinline__ int cell_mod(T f) {
  const int i = (fabs(f) < T(1073741824.0)) ? int(f) : 0;
  if constexpr ((N & (N - 1)) == 0) {
    return i & (N - 1);
  } else {
    const int r = i % N;
    return r < 0 ? r + N : r;
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).
// Renumber the flattened block index so that every XCD receives a contiguous
// run of logical blocks, and split the logical index with the task (or field
// group) fastest: each XCD then gets an even mix of heavy and light tasks, and
// all tasks of neighbouring rows / column tiles meet in the same L2 (the
// gathers, re-read rows and shared 128-byte lines hit in L2).
constexpr int NUM_XCD = 8;
// remap = 0 keeps the hardware order (logical index = flattened block index).
__device__ __forceinline__ void xcd_split(int nslow, int nfast, int& slow, int& fast, int& z, int remap) {
  const int total = nslow * nfast * gridDim.z;
  const int b = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
  const int q = total / NUM_XCD, r = total % NUM_XCD;
  const int xcd = b % NUM_XCD;
  const int logical = remap ? xcd * q + min(xcd, r) + b / NUM_XCD : b;
  fast = logical % nfast;
  const int rest = logical / nfast;
  slow = rest % nslow;
  z = rest / nslow;
}

// periodic bilinear interpolation at x + xi of one pair of the interleaved
// physical fields: (u, v) if pair == 0, the averaged fields if pair == 1 (uniform
// over the wave; 8 bytes per corner instead of the whole 16-byte point)
template <typename T, int N>
__device__ __forceinline__ cplx<T> gather2(const P4<T>* __restrict__ F, int pair, int x, int y, T xix, T xiy) {
  const T scl = T(double(N) / 6.283185307179586476925286766559);
  T ox = xix * scl, oy = xiy * scl;
  const T fx = floor(ox), fy = floor(oy);
  const T ax = ox - fx, ay = oy - fy;
  // x + (fx mod N) and y + (fy mod N) lie in [0, 2N)
  const int ix0 = wrap2N<N>(x + cell_mod<N>(fx)), iy0 = wrap2N<N>(y + cell_mod<N>(fy));
  const int ix1 = (ix0 + 1 == N) ? 0 : ix0 + 1, iy1 = (iy0 + 1 == N) ? 0 : iy0 + 1;
  // uniform base plus 32-bit byte offsets (the field is far below 4 GiB)
  const char* F2 = reinterpret_cast<const char*>(F) + pair * sizeof(cplx<T>);
  constexpr unsigned PT = sizeof(P4<T>), ROW = N * sizeof(P4<T>);
  const unsigned r0 = unsigned(iy0) * ROW, r1 = unsigned(iy1) * ROW;
  const unsigned c0 = unsigned(ix0) * PT, c1 = unsigned(ix1) * PT;
  const cplx<T> f00 = *reinterpret_cast<const cplx<T>*>(F2 + (r0 + c0));
  const cplx<T> f01 = *reinterpret_cast<const cplx<T>*>(F2 + (r0 + c1));
  const cplx<T> f10 = *reinterpret_cast<const cplx<T>*>(F2 + (r1 + c0));
  const cplx<T> f11 = *reinterpret_cast<const cplx<T>*>(F2 + (r1 + c1));
  const T w00 = (T(1) - ax) * (T(1) - ay), w01 = ax * (T(1) - ay);
  const T w10 = (T(1) - ax) * ay, w11 = ax * ay;
  return {w00 * f00.x + w01 * f01.x + w10 * f10.x + w11 * f11.x,
          w00 * f00.y + w01 * f01.y + w10 * f10.y + w11 * f11.y};
}

// periodic tensor-product cubic (4-point Lagrange) interpolation at x + xi of
// one pair of the interleaved physical fields, as gather2: with
// o = xi / dx, i0 = floor(o), a = o - i0, the nodes i0-1 .. i0+2 carry
// -a(a-1)(a-2)/6, (a+1)(a-1)(a-2)/2, -(a+1)a(a-2)/2, (a+1)a(a-1)/6
template <typename T>
__device__ __forceinline__ void cubic_weights(T a, T (&w)[4]) {
  const T p = a + T(1), q = a - T(1), r = a - T(2), sixth = T(1.0 / 6.0);  // no divisions
  w[0] = -(a * q) * (r * sixth);
  w[1] = (p * q) * (r * T(0.5));
  w[2] = -(p * a) * (r * T(0.5));
  w[3] = (p * a) * (q * sixth);
}
template <typename T, int N>
__device__ __forceinline__ cplx<T> gather2_cubic(const P4<T>* __restrict__ F, int pair, int x, int y, T xix, T xiy) {
  const T scl = T(double(N) / 6.283185307179586476925286766559);
  T ox = xix * scl, oy = xiy * scl;
  const T fx = floor(ox), fy = floor(oy);
  const T ax = ox - fx, ay = oy - fy;
  T wx[4], wy[4];
  cubic_weights(ax, wx);
  cubic_weights(ay, wy);
  const int bx = wrap2N<N>(x + cell_mod<N>(fx)), by = wrap2N<N>(y + cell_mod<N>(fy));
  const char* F2 = reinterpret_cast<const char*>(F) + pair * sizeof(cplx<T>);
  constexpr unsigned PT = sizeof(P4<T>), ROW = N * sizeof(P4<T>);
  unsigned col[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int c = bx + i - 1;
    c = c < 0 ? c + N : (c >= N ? c - N : c);
    col[i] = unsigned(c) * PT;
  }
  cplx<T> out = {T(0), T(0)};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int r = by + j - 1;
    r = r < 0 ? r + N : (r >= N ? r - N : r);
    const unsigned ro = unsigned(r) * ROW;
    cplx<T> row = {T(0), T(0)};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const cplx<T> f = *reinterpret_cast<const cplx<T>*>(F2 + (ro + col[i]));
      row.x += wx[i] * f.x;
      row.y += wx[i] * f.y;
    }
    out.x += wy[j] * row.x;
    out.y += wy[j] * row.y;
  }
  return out;
}

// points of a lane whose corners are loaded together (n points to gather): four,
// but two of the cubic gathers' sixteen corners at 1024, where a third wave per
// SIMD is worth more than the registers
template <int N, bool CUB>
__host__ __device__ constexpr int gather_points(int n) {
  const int g = CUB && N >= 1024 ? 2 : 4;
  return n % g == 0 ? g : (n % 2 == 0 ? 2 : 1);
}

// the pair of fields at x + xi, by either interpolant
template <typename T, int N, bool CUB>
__device__ __forceinline__ cplx<T> gather_pair(const P4<T>* __restrict__ F, int pair, int x, int y, T xix, T xiy) {
  if constexpr (CUB) return gather2_cubic<T, N>(F, pair, x, y, xix, xiy);
  else return gather2<T, N>(F, pair, x, y, xix, xiy);
}

// --------------------------------------------------------------------------
// the rows passes: blocks of cooperating waves
// --------------------------------------------------------------------------
// A block holds one group of rows (WR = 64 / NT rows, one per lane group of each
// wave); its waves share the row's transforms.  They load and inverse-transform
// pairs of fields side by side, exchange physical values through LDS, form the
// products and forward-transform them: a row is two or three transforms deep,
// however many fields it carries, instead of a chain of all of them on one wave
// (four to seven transforms deep), and strategy 1 shares the physical fields the
// dynamics form instead of reading them back.  Both passes together, us per stage,
// chains -> cooperating: 64^2 float64 23.4 -> 12.9, 256^2 float32 19.2 -> 13.8,
// 512^2 float64 47 -> 28, 1024^2 float32 49.9 -> 44.7, 1024^2 float64 143 -> 81.
// What bounds them: latency below 512^2 (a block's loads, two or three transforms
// and a gather in sequence), instruction issue and memory about equally at 1024^2.
template <typename T, int N>
struct CoopGeo {
  static constexpr int E = fft_E<N>(), NT = N / E;
  static_assert(NT <= 64 && 64 % NT == 0, "row groups within a wave");
  static constexpr int WR = 64 / NT;  // rows per block
  // large rows exchange real and imaginary parts in turn: half the LDS per
  // transform, so that more blocks fit a CU
  static constexpr bool SPLIT = N >= 1024 || (sizeof(T) == 8 && N >= 512);
  // a row's buffer, in values of T (an even number: pairs are kept there too)
  static constexpr int RB = SPLIT ? (padded_len(N) + 1) / 2 * 2 : 2 * padded_len(N);
  static_assert(N % WR == 0, "row geometry");
};

// values of a row shared between the waves: pairs in one buffer, or, split, the
// second component in a buffer of its own
template <typename T, bool SPLIT>
struct SharedPair {
  T *a, *b;
  __device__ __forceinline__ void put(int x, cplx<T> v) const {
    if constexpr (SPLIT) {
      a[x] = v.x;
      b[x] = v.y;
    } else {
      reinterpret_cast<cplx<T>*>(a)[x] = v;
    }
  }
  __device__ __forceinline__ cplx<T> get(int x) const {
    if constexpr (SPLIT) return {a[x], b[x]};
    else return reinterpret_cast<const cplx<T>*>(a)[x];
  }
};

// value of an averaging slot's field at a point (FieldSel); selects, no branches,
// so that the unrolled loops stay one block
template <typename T>
__device__ __forceinline__ T field_value(int fs, const cplx<T>& uv, const cplx<T>& hz, const Phys& ph) {
  const T q = (T(ph.f) + hz.y) / (T(ph.H) + hz.x);  // potential vorticity (f + zeta) / h
  T r = (fs == FS_ETA) ? hz.x : hz.y;
  r = (fs == FS_U) ? uv.x : r;
  r = (fs == FS_V) ? uv.y : r;
  return (fs == FS_Q) ? q : r;
}

// --------------------------------------------------------------------------
// rows_dyn: dynamics and strategy 1
// --------------------------------------------------------------------------
// Inverse transforms of (u, v), (eta, zeta) and the gradients of g-tilde_0,
// g-tilde_1, P_x, P_y; from the physical u, v, eta, zeta the products zeta v and
// zeta u, K = (u^2 + v^2) / 2 and eta u, eta v, -u . grad g-tilde (both fields one
// pair) and s u - u . grad P (another), forward-transformed.  u, v and the averaged
// fields are stored for the gathers.  For the default averaged fields (eta, zeta)
// the source f of eq. (4.1) is added in the column pass from the stage spectra
// (as the Eulerian accumulators take it), so that only the advection term goes
// through physical space and float32 rounding; other averaged fields (GEN) take f
// here, and their own spectra for the Eulerian means.
//
// Two shares of this work:
//   SIX (N < 1024), one inverse transform per wave, two deep:
//     wave 0 (u, v), then zeta v, zeta u     wave 1 (eta, zeta), then K, eta u
//     wave 2 grad g~_0, then the g~ pair     wave 3 grad g~_1, then eta v
//     wave 4 grad P_x, then the P pair       wave 5 grad P_y, then (GEN) f_0, f_1
//   four waves (N = 1024), three transforms each, one barrier:
//     wave 0 (u, v), zeta v, zeta u, (GEN) f_0, f_1    wave 1 (eta, zeta), K, eta u, eta v
//     wave 2 grad g~_0, grad g~_1, the g~ pair         wave 3 grad P_x, grad P_y, the P pair
template <typename T, int N>
struct DynGeo : CoopGeo<T, N> {
  using G = CoopGeo<T, N>;
  static constexpr bool SIX = N < 1024;
  static constexpr int WAVES = SIX ? 6 : 4, THREADS = 64 * WAVES;
  // six: shared pairs overlay their waves' buffers (split: second components apart);
  // four: shared pairs apart from the transform buffers (split always)
  static constexpr int BUFS = G::SPLIT ? 8 : 6;
  static_assert(SIX || G::SPLIT, "four waves: split exchanges");
  static constexpr int LDS = BUFS * G::WR * G::RB;
  // registers for this many resident waves per SIMD; the averaged fields' formulas
  // (gen) take more of them
  static constexpr int min_waves(bool gen) {
    const bool f32 = sizeof(T) == 4;
    return gen ? (f32 ? 2 : 1) : (SIX ? 3 : (f32 ? 4 : 2));
  }
};

template <typename T, int N, bool GEN>
__device__ __forceinline__ void rows_dyn_four(const StepPtrs<T>& P, const Phys& ph, double s,
                                              int rowblock, T* lds) {
  using G = DynGeo<T, N>;
  constexpr int E = G::E, NT = G::NT, WR = G::WR, RB = G::RB;
  constexpr bool SPLIT = true;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // the wave's role
  const int lane = threadIdx.x % 64;
  const int g = lane / NT, t = lane % NT;
  const int y = rowblock * WR + g;
  auto buf = [&](int i) { return lds + (i * WR + g) * RB; };
  const SharedPair<T, SPLIT> UV{buf(4), buf(5)}, HZ{buf(6), buf(7)};
  T* mine = buf(w);
  constexpr Dims d = dims_of<N>();
  constexpr size_t rf = d.rowfield_elems();
  const unsigned row = (unsigned)y * (unsigned)d.NKXP;
  const cplx<T>* A = P.IC + (w == 2 ? IC_GTH : IC_PX) * rf;  // waves 2, 3: their first field

  cplx<T> z[E];
  if (w == 0) {
    load_pair<T, N, false, false>(z, P.IC + IC_U * rf, P.IC + IC_V * rf, row, t);
  } else if (w == 1) {
    load_depth_vorticity<T, N>(z, P.IC + IC_H * rf, P.IC + IC_V * rf, P.IC + IC_UY * rf, row, t);
  } else {
    load_pair<T, N, true, false>(z, A, A + rf, row, t);
  }
  inverse_row<T, N, SPLIT>(z, mine, t, P.tw);
  if (w < 2) {
    const SharedPair<T, SPLIT> S{w == 0 ? UV.a : HZ.a, w == 0 ? UV.b : HZ.b};
#pragma unroll
    for (int e = 0; e < E; ++e) S.put(t + NT * e, z[e]);
  }
  __syncthreads();
  if (w < 2) {
    const unsigned at = (unsigned)(y * N + t);
    if (w == 0) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const cplx<T> uv = z[e], hz = HZ.get(t + NT * e);
        if constexpr (!GEN) put32(P.uvhz + NT * e, at, P4<T>{uv.x, uv.y, hz.x, hz.y});
        else put32(P.uvhz + NT * e, at, P4<T>{uv.x, uv.y, field_value<T>(ph.fs0, uv, hz, ph), field_value<T>(ph.fs1, uv, hz, ph)});
        z[e] = {hz.y * uv.y, hz.y * uv.x};
        if (e % 4 == 3) sched_fence();
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const cplx<T> uv = UV.get(t + NT * e), hz = z[e];
        z[e] = {T(0.5) * (uv.x * uv.x + uv.y * uv.y), hz.x * uv.x};
        if (e % 4 == 3) sched_fence();
      }
    }
    if (!ph.kin) {
      cplx<T>* OA = P.RS + (w == 0 ? RS_ZV : RS_K) * rf;
      cplx<T>* OB = P.RS + (w == 0 ? RS_ZU : RS_HU) * rf;
      forward_row<T, N, SPLIT>(z, mine, t, P.tw, OA, OB, row);
    }
    if (w == 0) {
      if constexpr (GEN) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const cplx<T> uv = UV.get(t + NT * e), hz = HZ.get(t + NT * e);
          z[e] = {field_value<T>(ph.fs0, uv, hz, ph), field_value<T>(ph.fs1, uv, hz, ph)};
          if (e % 4 == 3) sched_fence();
        }
        forward_row<T, N, SPLIT>(z, mine, t, P.tw, P.RS + RS_F0 * rf, P.RS + RS_F1 * rf, row);
      }
    } else if (!ph.kin) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int x = t + NT * e;
        z[e] = {HZ.get(x).x * UV.get(x).y, T(0)};
        if (e % 4 == 3) sched_fence();
      }
      forward_row<T, N, SPLIT>(z, mine, t, P.tw, P.RS + RS_HV * rf, nullptr, row);
    }
    return;
  }
  // f - u . grad of the wave's two fields: f = s u, s v for P, 0 or the averaged
  // fields for g-tilde
  const bool isP = w == 3;
  const T sT = T(s);
  cplx<T> a[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = t + NT * e;
    const cplx<T> uv = UV.get(x);
    T f = isP ? sT * uv.x : T(0);
    if constexpr (GEN) f = isP ? f : field_value<T>(ph.fs0, uv, HZ.get(x), ph);
    a[e].x = f - (uv.x * z[e].x + uv.y * z[e].y);
    if (e % 4 == 3) sched_fence();
  }
  load_pair<T, N, true, false>(z, A + 2 * rf, A + 3 * rf, row, t);
  inverse_row<T, N, SPLIT>(z, mine, t, P.tw);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = t + NT * e;
    const cplx<T> uv = UV.get(x);
    T f = isP ? sT * uv.y : T(0);
    if constexpr (GEN) f = isP ? f : field_value<T>(ph.fs1, uv, HZ.get(x), ph);
    a[e].y = f - (uv.x * z[e].x + uv.y * z[e].y);
    if (e % 4 == 3) sched_fence();
  }
  cplx<T>* OA = P.RS + (isP ? RS_PX : RS_GTH) * rf;
  forward_row<T, N, SPLIT>(a, mine, t, P.tw, OA, OA + rf, row);
}

template <typename T, int N, bool GEN>
__device__ __forceinline__ void rows_dyn_six(const StepPtrs<T>& P, const Phys& ph, double s,
                                              int rowblock, T* lds) {
  using G = DynGeo<T, N>;
  constexpr int E = G::E, NT = G::NT, WR = G::WR, RB = G::RB;
  constexpr bool SPLIT = G::SPLIT;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // the wave's role
  const int lane = threadIdx.x % 64;
  const int g = lane / NT, t = lane % NT;
  const int y = rowblock * WR + g;
  auto buf = [&](int i) { return lds + (i * WR + g) * RB; };
  const SharedPair<T, SPLIT> UV{buf(0), buf(SPLIT ? 6 : 0)}, HZ{buf(1), buf(SPLIT ? 7 : 1)};
  T* mine = buf(w);
  constexpr Dims d = dims_of<N>();
  constexpr size_t rf = d.rowfield_elems();
  const unsigned row = (unsigned)y * (unsigned)d.NKXP;

  cplx<T> z[E];
  if (w == 0) {
    load_pair<T, N, false, false>(z, P.IC + IC_U * rf, P.IC + IC_V * rf, row, t);
  } else if (w == 1) {
    load_depth_vorticity<T, N>(z, P.IC + IC_H * rf, P.IC + IC_V * rf, P.IC + IC_UY * rf, row, t);
  } else {
    const cplx<T>* A = P.IC + (IC_GTH + 2 * (w - 2)) * rf;  // g-tilde_0, g-tilde_1, P_x, P_y
    load_pair<T, N, true, false>(z, A, A + rf, row, t);
  }
  inverse_row<T, N, SPLIT>(z, mine, t, P.tw);
  if (w < 2) {
    const SharedPair<T, SPLIT> S{w == 0 ? UV.a : HZ.a, w == 0 ? UV.b : HZ.b};
#pragma unroll
    for (int e = 0; e < E; ++e) S.put(t + NT * e, z[e]);
  }
  __syncthreads();
  cplx<T>*OA = nullptr, *OB = nullptr;
  if (w == 0) {
    const unsigned at = (unsigned)(y * N + t);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const cplx<T> uv = z[e], hz = HZ.get(t + NT * e);
      if constexpr (!GEN) put32(P.uvhz + NT * e, at, P4<T>{uv.x, uv.y, hz.x, hz.y});
      else put32(P.uvhz + NT * e, at, P4<T>{uv.x, uv.y, field_value<T>(ph.fs0, uv, hz, ph), field_value<T>(ph.fs1, uv, hz, ph)});
      z[e] = {hz.y * uv.y, hz.y * uv.x};
      if (e % 4 == 3) sched_fence();
    }
    if (!ph.kin) OA = P.RS + RS_ZV * rf, OB = P.RS + RS_ZU * rf;
  } else if (w == 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const cplx<T> uv = UV.get(t + NT * e), hz = z[e];
      z[e] = {T(0.5) * (uv.x * uv.x + uv.y * uv.y), hz.x * uv.x};
      if (e % 4 == 3) sched_fence();
    }
    if (!ph.kin) OA = P.RS + RS_K * rf, OB = P.RS + RS_HU * rf;
  } else {
    // f - u . grad (one field per wave): f = s u or s v for P, 0 or the averaged
    // field for g-tilde
    const bool isP = w >= 4;
    const T sT = T(s);
    T* pair = buf(w & ~1);  // the even wave's buffer takes the odd wave's values
    const int fs = (w == 2) ? ph.fs0 : ph.fs1;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int x = t + NT * e;
      const cplx<T> uv = UV.get(x);
      T f = isP ? sT * ((w & 1) ? uv.y : uv.x) : T(0);
      if constexpr (GEN) f = isP ? f : field_value<T>(fs, uv, HZ.get(x), ph);
      z[e].x = f - (uv.x * z[e].x + uv.y * z[e].y);
      if (e % 4 == 3) sched_fence();
    }
    if (w & 1) {
#pragma unroll
      for (int e = 0; e < E; ++e) pair[t + NT * e] = z[e].x;
      if (w == 3) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int x = t + NT * e;
          z[e] = {HZ.get(x).x * UV.get(x).y, T(0)};
          if (e % 4 == 3) sched_fence();
        }
        if (!ph.kin) OA = P.RS + RS_HV * rf;
      } else if constexpr (GEN) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const cplx<T> uv = UV.get(t + NT * e), hz = HZ.get(t + NT * e);
          z[e] = {field_value<T>(ph.fs0, uv, hz, ph), field_value<T>(ph.fs1, uv, hz, ph)};
          if (e % 4 == 3) sched_fence();
        }
        OA = P.RS + RS_F0 * rf, OB = P.RS + RS_F1 * rf;
      }
    } else {
      OA = P.RS + (w == 2 ? RS_GTH : RS_PX) * rf, OB = OA + rf;
    }
  }
  __syncthreads();
  if (!OA) return;
  if (w == 2 || w == 4) {
#pragma unroll
    for (int e = 0; e < E; ++e) z[e].y = mine[t + NT * e];
    xsync<NT>();
  }
  forward_row<T, N, SPLIT>(z, mine, t, P.tw, OA, OB, row);
}

template <typename T, int N, bool GEN>
__device__ __forceinline__ void rows_dyn_body(const StepPtrs<T>& P, const Phys& ph, double s,
                                              int rowblock, T* lds) {
  if constexpr (DynGeo<T, N>::SIX) rows_dyn_six<T, N, GEN>(P, ph, s, rowblock, lds);
  else rows_dyn_four<T, N, GEN>(P, ph, s, rowblock, lds);
}

// GEN: averaged fields other than (eta, zeta)
template <typename T, int N, bool GEN>
__global__ void __launch_bounds__((DynGeo<T, N>::THREADS), (DynGeo<T, N>::min_waves(GEN)))
    k_rows_dyn(StepPtrs<T> P, Phys ph, double s, int remap) {
  __shared__ __align__(16) T lds[DynGeo<T, N>::LDS];
  int rowblock, unused, z;
  xcd_split(gridDim.x, 1, rowblock, unused, z, remap);
  rows_dyn_body<T, N, GEN>(P, ph, s, rowblock, lds);
}

// --------------------------------------------------------------------------
// rows_rhs: strategy 2
// --------------------------------------------------------------------------
// Four waves, the pairs (xi_x, xi_y) and (g-bar_0, g-bar_1) of two waves each.
// Wave 0 inverse-transforms xi and shares it, waves 1, 2 and 3 the gradients of
// xi_x, xi_y and g-bar_0, wave 0 then that of g-bar_1.  Of the pair's
//   u(x+xi) - w - (w . grad) xi   (both components, eq. (4.5a)),
//   f(x+xi) - w . grad g-bar      (eq. (4.5b))
// each wave forms its own component's gradient terms; waves 1 and 3 gather their
// pair; waves 2 and 0 hand theirs to waves 1 and 3, which forward-transform the pair.
// The sixteen corners of the cubic gathers have waves of their own (GATHER_WAVES),
// an even share of a pair's points each, beside the second transform and the products;
// rows exchanged in parts have no LDS to spare for that, there waves 2 and 0 take
// half of their pair's points.  With the momentum rows' shared gathers, both passes
// per stage: 384^2 float32 40.7 -> 22.3 us, 192^2 float64 40.8 -> 25.3, 64^2 float64
// 12.4 -> 11.7 (bilinear gathers stay whole: 128^2 float32 62.6 us per
// step whole, 64.4 in halves).
// w = xi / (t - tau) is the partial-mean velocity (u / 2 at t = tau).
template <typename T, int N>
struct RhsGeo : CoopGeo<T, N> {
  using G = CoopGeo<T, N>;
  // of cubic gathers; with twelve values per lane eight (4 -> 8 waves, a step with
  // momentum: 384^2 float32 186.6 -> 183.3 us, 192^2 float32 143.3 -> 139.0; bilinear
  // gathers on four waves of their own: 192^2 float32 68.8 -> 65.4, but 384^2 float64
  // 145.6 -> 155.7)
  static constexpr int GATHER_WAVES = G::SPLIT ? 0 : (G::E == 12 ? 8 : 4);
  static constexpr int WAVES = 4, THREADS = 64 * WAVES, CUB_THREADS = 64 * (WAVES + GATHER_WAVES);
  static constexpr int BUFS = G::SPLIT ? 6 : 5;  // four transform buffers, then xi
  static constexpr int LDS = BUFS * G::WR * G::RB;
  // registers for this many resident waves per SIMD
  static constexpr int min_waves(bool cub) {
    return sizeof(T) == 4 ? (cub ? (N < 1024 ? 2 : 3) : 4) : (cub ? 1 : 2);
  }
};

template <typename T, int N, bool CUB, bool SPOS>
__device__ __forceinline__ void rhs_products(const P4<T>* __restrict__ F, double s, int y, int t, int w,
                                             const SharedPair<T, CoopGeo<T, N>::SPLIT>& XI,
                                             cplx<T> (&z)[fft_E<N>()], T* pair, cplx<T>* half) {
  // points that waves 1 and 3 gather
  constexpr int E = fft_E<N>(), NT = N / E, H = !CUB ? E : (RhsGeo<T, N>::GATHER_WAVES ? 0 : E / 2);
  constexpr int GG = gather_points<N, CUB>(H);
  const T inv_s = SPOS ? T(1.0 / s) : T(0);
  const unsigned at = (unsigned)(y * N);
  // w and the wave's own component: -w_i - w . grad
  const bool subx = (w == 1), suby = (w == 2);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = t + NT * e;
    cplx<T> v;
    if constexpr (SPOS) {
      const cplx<T> xi = XI.get(x);
      v = {xi.x * inv_s, xi.y * inv_s};
    } else {
      const P4<T> q = at32(F + NT * e, at + t);
      v = {T(0.5) * q.u, T(0.5) * q.v};
    }
    const T own = subx ? v.x : (suby ? v.y : T(0));
    z[e].x = -own - (v.x * z[e].x + v.y * z[e].y);
    if (e % 4 == 3) sched_fence();
  }
  if (w & 1) {
#pragma unroll
    for (int e0 = 0; e0 < H; e0 += GG) {
#pragma unroll
      for (int e = e0; e < e0 + GG; ++e) {
        const cplx<T> xi = XI.get(t + NT * e);
        const cplx<T> g = gather_pair<T, N, CUB>(F, w >> 1, t + NT * e, y, xi.x, xi.y);
        z[e] = {g.x + z[e].x, g.y};
      }
      sched_fence();
    }
#pragma unroll
    for (int e = H; e < E; ++e) z[e].y = T(0);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) pair[t + NT * e] = z[e].x;
    if constexpr (H == E || H == 0) return;
#pragma unroll
    for (int e0 = H; e0 < E; e0 += GG) {
#pragma unroll
      for (int e = e0; e < e0 + GG; ++e) {
        const cplx<T> xi = XI.get(t + NT * e);
        half[t + NT * (e - H)] = gather_pair<T, N, CUB>(F, w == 0 ? 1 : 0, t + NT * e, y, xi.x, xi.y);
      }
      sched_fence();
    }
  }
}

template <typename T, int N, bool CUB>
__device__ __forceinline__ void rows_rhs_body(const StepPtrs<T>& P, double s, int rowblock, T* lds) {
  using G = RhsGeo<T, N>;
  constexpr int E = G::E, NT = G::NT, WR = G::WR, RB = G::RB;
  constexpr bool SPLIT = G::SPLIT;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // the wave's role
  const int lane = threadIdx.x % 64;
  const int g = lane / NT, t = lane % NT;
  const int y = rowblock * WR + g;
  auto buf = [&](int i) { return lds + (i * WR + g) * RB; };
  const SharedPair<T, SPLIT> XI{buf(4), buf(SPLIT ? 5 : 4)};
  T* mine = buf(w);
  constexpr Dims d = dims_of<N>();
  constexpr size_t rf = d.rowfield_elems();
  const unsigned row = (unsigned)y * (unsigned)d.NKXP;

  // The gather waves leave a pair for wave q = 1 or 3: first components behind the N
  // values that waves 2 and 0 hand over in q's buffer, second ones in wave 2's (which
  // transforms nothing more, so neither q overwrites what the other still reads).
  constexpr bool GW = CUB && G::GATHER_WAVES > 0;
  auto gathered = [&](int q) { return SharedPair<T, true>{buf(q) + N, buf(2) + (q == 3 ? N : 0)}; };
  if constexpr (GW) {
    if (w >= G::WAVES) {
      __syncthreads();  // xi is there, and waves 1 to 3 are done with their buffers
      constexpr int PARTS = G::GATHER_WAVES / 2, H = E / PARTS, GG = gather_points<N, CUB>(H);
      const int i = w - G::WAVES, pair = i % 2, e1 = i / 2 * H;
      const SharedPair<T, true> to = gathered(2 * pair + 1);
#pragma unroll
      for (int e0 = 0; e0 < H; e0 += GG) {
#pragma unroll
        for (int e = e0; e < e0 + GG; ++e) {
          const int x = t + NT * (e1 + e);
          const cplx<T> xi = XI.get(x);
          to.put(x, gather_pair<T, N, CUB>(P.uvhz, pair, x, y, xi.x, xi.y));
        }
        sched_fence();
      }
      __syncthreads();
      return;
    }
  }

  cplx<T> z[E];
  if (w == 0) {
    load_pair<T, N, false, false>(z, P.IC + IC_XIX * rf, P.IC + IC_XIY * rf, row, t);
  } else {
    const cplx<T>* A = P.IC + (IC_XIX + 2 * (w - 1)) * rf;  // xi_x, xi_y, g-bar_0
    load_pair<T, N, true, false>(z, A, A + rf, row, t);
  }
  inverse_row<T, N, SPLIT>(z, mine, t, P.tw);
  if (w == 0) {
#pragma unroll
    for (int e = 0; e < E; ++e) XI.put(t + NT * e, z[e]);
  }
  __syncthreads();
  if (w == 0) {
    load_pair<T, N, true, false>(z, P.IC + IC_GBZ * rf, P.IC + (IC_GBZ + 1) * rf, row, t);
    inverse_row<T, N, SPLIT>(z, mine, t, P.tw);
  }
  // the even waves' component goes to their partner's transform buffer, their half
  // of the gathered points (N / 2 pairs) to their own
  T* pair = buf(w == 0 ? 3 : 1);
  if (s > 0.0) rhs_products<T, N, CUB, true>(P.uvhz, s, y, t, w, XI, z, pair, reinterpret_cast<cplx<T>*>(mine));
  else rhs_products<T, N, CUB, false>(P.uvhz, s, y, t, w, XI, z, pair, reinterpret_cast<cplx<T>*>(mine));
  __syncthreads();
  if (!(w & 1)) return;
  const cplx<T>* half = reinterpret_cast<const cplx<T>*>(buf(w == 1 ? 2 : 0));
#pragma unroll
  for (int e = 0; e < E; ++e) {
    z[e].y = z[e].y + mine[t + NT * e];
    if constexpr (GW) {
      const cplx<T> g = gathered(w).get(t + NT * e);
      z[e] = {z[e].x + g.x, z[e].y + g.y};
    } else if (CUB && e >= E / 2) {
      const cplx<T> g = half[t + NT * (e - E / 2)];
      z[e] = {z[e].x + g.x, z[e].y + g.y};
    }
  }
  xsync<NT>();
  cplx<T>* OA = P.RS + (w == 1 ? RS_XIX : RS_GBH) * rf;
  forward_row<T, N, SPLIT>(z, mine, t, P.tw, OA, OA + rf, row);
}

// CUB: cubic instead of bilinear strategy-2 gathers
template <typename T, int N, bool CUB>
__global__ void __launch_bounds__((CUB ? RhsGeo<T, N>::CUB_THREADS : RhsGeo<T, N>::THREADS), (RhsGeo<T, N>::min_waves(CUB)))
    k_rows_rhs(StepPtrs<T> P, double s, int remap) {
  __shared__ __align__(16) T lds[RhsGeo<T, N>::LDS];
  int rowblock, unused, z;
  xcd_split(gridDim.x, 1, rowblock, unused, z, remap);
  rows_rhs_body<T, N, CUB>(P, s, rowblock, lds);
}

// --------------------------------------------------------------------------
// rows_mom: the strategy-2 mean of the momentum 1-form (appendix C, eq. (C.4)
// in the g-bar form of eq. (4.5b)), launched after rows_rhs when requested:
//   R_i = u_j(x + xi)(delta_ij + d_i xi_j) - w_j d_j g_i - g_j d_i xi_j / s
// (w = xi / s, or u / 2 at s = 0, where g = 0 and the last term is not formed).
// --------------------------------------------------------------------------
// Six waves: wave 0 inverse-transforms xi and wave 1 g (both shared), waves 2 and
// 3 d_x (xi_x, xi_y) and d_y (xi_x, xi_y), waves 4 and 5 grad g_x and grad g_y.
// Waves 0 to 3 gather u at a quarter of the points x + xi each and share it, while
// waves 4 and 5 form -w . grad g_i; then waves 2 and 3 form
//   u_i + sum_j (u_j - g_j / s) d_i xi_j,
// and wave 2 adds the halves of both components and forward-transforms the pair.
// (Gathered on waves 2 and 3, every point twice: both strategy-2 passes of a cubic
// run, us per stage, 1024^2 float32 79 -> 67, float64 259 -> 202.)
template <typename T, int N>
struct MomGeo : CoopGeo<T, N> {
  using G = CoopGeo<T, N>;
  static constexpr int WAVES = 6, THREADS = 64 * WAVES;
  static constexpr int BUFS = G::SPLIT ? 8 : 6;  // split: xi_y and g_y get buffers of their own
  static constexpr int LDS = BUFS * G::WR * G::RB;
  static constexpr int min_waves(bool cub) { return sizeof(T) == 4 ? (cub && N < 1024 ? 2 : 3) : (cub ? 1 : 2); }
};

template <typename T, int N, bool CUB>
__device__ __forceinline__ void rows_mom_body(const StepPtrs<T>& P, double s, int rowblock, T* lds) {
  using G = MomGeo<T, N>;
  constexpr int E = G::E, NT = G::NT, WR = G::WR, RB = G::RB;
  constexpr bool SPLIT = G::SPLIT;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // the wave's role
  const int lane = threadIdx.x % 64;
  const int g = lane / NT, t = lane % NT;
  const int y = rowblock * WR + g;
  auto buf = [&](int i) { return lds + (i * WR + g) * RB; };
  const SharedPair<T, SPLIT> XI{buf(0), buf(SPLIT ? 6 : 0)}, GM{buf(1), buf(SPLIT ? 7 : 1)};
  const SharedPair<T, SPLIT> U{buf(2), buf(SPLIT ? 3 : 2)};  // their own transforms are done by then
  T* mine = buf(w);
  constexpr Dims d = dims_of<N>();
  constexpr size_t rf = d.rowfield_elems();
  const unsigned row = (unsigned)y * (unsigned)d.NKXP;
  const P4<T>* F = P.uvhz;

  cplx<T> z[E];
  if (w == 2) {
    load_pair<T, N, true, true>(z, P.IC + IC_XIX * rf, P.IC + IC_XIY * rf, row, t);
  } else if (w >= 4) {
    const cplx<T>* A = P.IC + (w == 4 ? IC_GMX : IC_GMY) * rf;
    load_pair<T, N, true, false>(z, A, A + rf, row, t);
  } else {
    // xi, g, and the column pass's i ky versions of xi
    const cplx<T>* A = P.IC + (w == 0 ? IC_XIX : w == 1 ? IC_GMX : IC_XIX_Y) * rf;
    load_pair<T, N, false, false>(z, A, A + 2 * rf, row, t);
  }
  inverse_row<T, N, SPLIT>(z, mine, t, P.tw);
  if (w < 2) {
    const SharedPair<T, SPLIT> S{w == 0 ? XI.a : GM.a, w == 0 ? XI.b : GM.b};
#pragma unroll
    for (int e = 0; e < E; ++e) S.put(t + NT * e, z[e]);
  }
  __syncthreads();
  const bool spos = s > 0.0;
  const T inv_s = spos ? T(1.0 / s) : T(0);
  if (w < 4) {
    constexpr int Q = E / 4, GG = gather_points<N, CUB>(Q);
    static_assert(E % 4 == 0, "four waves gather");
#pragma unroll
    for (int e0 = 0; e0 < Q; e0 += GG) {
#pragma unroll
      for (int e = e0; e < e0 + GG; ++e) {
        const int x = t + NT * (w * Q + e);
        const cplx<T> xi = XI.get(x);
        U.put(x, gather_pair<T, N, CUB>(F, 0, x, y, xi.x, xi.y));
      }
      sched_fence();
    }
  } else {
    const unsigned at = (unsigned)(y * N);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int x = t + NT * e;
      const cplx<T> xi = XI.get(x);
      cplx<T> v = {xi.x * inv_s, xi.y * inv_s};
      if (!spos) {
        const P4<T> q = at32(F, at + x);
        v = {T(0.5) * q.u, T(0.5) * q.v};
      }
      mine[x] = -(v.x * z[e].x + v.y * z[e].y);
      if (e % 4 == 3) sched_fence();
    }
  }
  __syncthreads();
  T* r3 = buf(0);  // wave 3's half: xi has been read
  if (w == 2 || w == 3) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int x = t + NT * e;
      const cplx<T> u = U.get(x), gm = GM.get(x);
      const T gx = spos ? gm.x * inv_s : T(0), gy = spos ? gm.y * inv_s : T(0);
      const T ui = (w == 2) ? u.x : u.y;
      z[e].x = ui + ((u.x - gx) * z[e].x + (u.y - gy) * z[e].y);
      if (w == 3) r3[x] = z[e].x;
      if (e % 4 == 3) sched_fence();
    }
  }
  __syncthreads();
  if (w != 2) return;
  const T *r4 = buf(4), *r5 = buf(5);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = t + NT * e;
    z[e] = {z[e].x + r4[x], r3[x] + r5[x]};
  }
  forward_row<T, N, SPLIT>(z, mine, t, P.tw, P.RS + RS_GMX * rf, P.RS + RS_GMY * rf, row);
}

template <typename T, int N, bool CUB>
__global__ void __launch_bounds__((MomGeo<T, N>::THREADS), (MomGeo<T, N>::min_waves(CUB)))
    k_rows_mom(StepPtrs<T> P, double s, int remap) {
  __shared__ __align__(16) T lds[MomGeo<T, N>::LDS];
  int rowblock, unused, z;
  xcd_split(gridDim.x, 1, rowblock, unused, z, remap);
  rows_mom_body<T, N, CUB>(P, s, rowblock, lds);
}

// --------------------------------------------------------------------------
// columns
// --------------------------------------------------------------------------

// (hi, lo) + d for a float value carried as two words: Knuth's two-sum of hi
// and d gives the sum and its exact rounding error, which is folded into lo
// before the pair is renormalised (|lo| <= half an ulp of hi).  Contraction to
// fused multiply-adds is off here: the error terms need the plain roundings.
__device__ __forceinline__ void comp_add(float& hi, float& lo, float d) {
#pragma clang fp contract(off)
  const float s = hi + d;
  const float bp = s - hi;
  const float err = (hi - (s - bp)) + (d - bp);
  const float t = lo + err;
  const float h2 = s + t;
  lo = t - (h2 - s);
  hi = h2;
}

// Classical RK4 on one coefficient, in registers: y the state, lo its trailing
// word (compensated float state), a the accumulator of k1 + 2 k2 + 2 k3; k the
// stage's right-hand side.  Returns the next stage input (the new state after
// stage 3) and updates a (stages 0-2) or y and lo (stage 3), which the caller
// stores.  Float state is compensated: y holds the leading word and lo the
// trailing one, so the state itself carries about 48 significant bits and the
// rounding of the state at every step no longer accumulates over a long run.
// Stage inputs, right-hand sides and the accumulator stay float (their rounding
// enters once per step, scaled by dt).  Float64 state ignores lo.
// K: the stage's kind, fixed at compile time (a uniform branch around whole
// batches instead of one per coefficient): 0 the first stage, 1 the two middle
// ones, whose coefficient cn is dt/2 or dt, 3 the last.
template <int K, typename TS>
__device__ __forceinline__ cplx<TS> rk4v(cplx<TS>& y, cplx<TS>& lo, cplx<TS>& a, cplx<TS> k, double dt, double cn) {
  if constexpr (K == 0) {
    a = k;
    const TS c = TS(0.5 * dt);
    return {y.x + c * k.x, y.y + c * k.y};
  } else if constexpr (K == 1) {
    a = {a.x + TS(2) * k.x, a.y + TS(2) * k.y};
    const TS c = TS(cn);
    return {y.x + c * k.x, y.y + c * k.y};
  } else {
    const TS c = TS(dt / 6.0);
    if constexpr (std::is_same<TS, float>::value) {
      comp_add(y.x, lo.x, c * (a.x + k.x));
      comp_add(y.y, lo.y, c * (a.y + k.y));
    } else {
      y = {y.x + c * (a.x + k.x), y.y + c * (a.y + k.y)};
    }
    return y;
  }
}

// the words rk4v writes back: a at stages 0-2, y and lo at stage 3 (it reads y
// always, a from stage 1, lo at stage 3 for float)
template <int K, typename TS>
__device__ __forceinline__ void rk4_store(cplx<TS>* Yp, cplx<TS>* Lp, cplx<TS>* Ap, unsigned j, const cplx<TS>& y,
                                          const cplx<TS>& lo, const cplx<TS>& a) {
  if constexpr (K < 3) {
    put32(Ap, j, a);
  } else {
    put32(Yp, j, y);
    if constexpr (std::is_same<TS, float>::value) put32(Lp, j, lo);
  }
}

template <typename T, int N, int C>
struct ColCtx {
  static constexpr int E = fft_E<N>(), NT = N / E;
  static constexpr int CS = 2 * col_buf(N);  // a column's buffer, in values of T
  T* lds;           // C buffers
  T* buf;           // this lane group's buffer
  int c, t, kx0, kx;
  bool valid;       // kx <= K
  unsigned ky0;     // index of ky = 0 in the column's state (columns past K: of column K)
  __device__ __forceinline__ ColCtx(T* l, int tile) : lds(l) {
    constexpr Dims d = dims_of<N>();
    c = threadIdx.x / NT;
    t = threadIdx.x % NT;
    buf = lds + c * CS;
    kx0 = tile * C;
    kx = kx0 + c;
    valid = kx <= kcut<N>();
    ky0 = (unsigned)(min(kx, kcut<N>()) * d.NKY + d.K);
  }
};

// Coefficient ky that entry k = t + NT r of a column transform stands for:
// k <= K: ky = k, k >= N - K: ky = k - N, none in between.  Most r are the same
// for every lane; their place in the state is then the lane's offset plus a
// constant.  Lanes without a coefficient read a valid place (ky = 0) and are
// dropped at the store.
template <int N>
struct ColIdx {
  static constexpr int E = fft_E<N>(), NT = N / E, K = kcut<N>();
  int t, r;
  __device__ __forceinline__ bool all_lo() const { return NT * r + NT - 1 <= K; }
  __device__ __forceinline__ bool all_hi() const { return NT * r >= N - K; }
  __device__ __forceinline__ bool none() const { return NT * r > K && NT * r + NT - 1 < N - K; }
  __device__ __forceinline__ bool in() const { return all_lo() || all_hi() || t + NT * r <= K || t + NT * r >= N - K; }
  // ky = lane() + off()
  __device__ __forceinline__ int lane() const {
    if (all_lo() || all_hi()) return t;
    const int k = t + NT * r;
    return k <= K ? k : (k >= N - K ? k - N : 0);
  }
  __device__ __forceinline__ int off() const { return all_lo() ? NT * r : (all_hi() ? NT * r - N : 0); }
  __device__ __forceinline__ int ky() const { return lane() + off(); }
};

// one complex value of a buffer-resource load (8 or 16 bytes)
template <typename T>
__device__ __forceinline__ cplx<T> buffer_cplx(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
  if constexpr (sizeof(cplx<T>) == 8) return __builtin_bit_cast(cplx<T>, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0));
  else return __builtin_bit_cast(cplx<T>, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0));
}

// block-wide: columns kx0..kx0+C-1 of a [N][NKXP] field A, or of A - i kx B, into
// lane registers, v[r] = row t + NT r of the lane group's column.  A thread loads
// one column c at rows y = threadIdx.x / C + NT k; the tile is transposed in LDS.
// A field is read as one buffer resource: the thread's offset sits in one vector
// register and the row step of each of its E loads in a scalar register, so all E
// loads are in flight at once for the price of their data registers.  (A column's
// kx is fixed, so the x derivative of B joins A before the one transform.)
// Columns past K read the row's padding and are replaced by zeros.
template <typename T, int N, int C, bool DX>
__device__ __forceinline__ void tile_load(const ColCtx<T, N, C>& cx, const cplx<T>* __restrict__ A,
                                          const cplx<T>* __restrict__ B, cplx<T> (&v)[fft_E<N>()]) {
  using X = ColCtx<T, N, C>;
  constexpr int E = X::E, NT = X::NT;
  constexpr Dims d = dims_of<N>();
  constexpr int bytes = (int)(d.rowfield_elems() * sizeof(cplx<T>));
  const int c = threadIdx.x % C, y0 = threadIdx.x / C;
  const bool in = cx.kx0 + c <= kcut<N>();
  const __amdgpu_buffer_rsrc_t ra =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<cplx<T>*>(A), (short)0, bytes, 0x00020000);
  const unsigned voff = ((unsigned)y0 * (unsigned)d.NKXP + (unsigned)(cx.kx0 + c)) * (unsigned)sizeof(cplx<T>);
  constexpr unsigned dy = (unsigned)NT * (unsigned)d.NKXP * (unsigned)sizeof(cplx<T>);
  cplx<T> val[E];
#pragma unroll
  for (int k = 0; k < E; ++k) val[k] = buffer_cplx<T>(ra, voff, (unsigned)k * dy);
  if constexpr (DX) {
    const __amdgpu_buffer_rsrc_t rb =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<cplx<T>*>(B), (short)0, bytes, 0x00020000);
    const T kx = T(cx.kx0 + c);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const cplx<T> b = buffer_cplx<T>(rb, voff, (unsigned)k * dy);
      val[k] = {val[k].x + kx * b.y, val[k].y - kx * b.x};
    }
  }
#pragma unroll
  for (int k = 0; k < E; ++k) val[k] = in ? val[k] : cplx<T>{T(0), T(0)};
  T* col = cx.lds + c * X::CS;
  __syncthreads();  // the buffers' earlier contents have been read
#pragma unroll
  for (int k = 0; k < E; ++k) reinterpret_cast<cplx<T>*>(col)[pidx(LaneIdx{y0, NT * k})] = val[k];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < E; ++r) v[r] = reinterpret_cast<const cplx<T>*>(cx.buf)[pidx(LaneIdx{cx.t, NT * r})];
  xsync<NT>();
}

// block-wide: the C buffers at lds (entries in natural order) to columns
// kx0.. of a [N][NKXP] field, after a barrier of the caller.  The block is C * N /
// E threads, a compile-time count, so the loop unrolls and all of a thread's LDS
// reads are issued before its stores.
template <typename T, int N, int C>
__device__ __forceinline__ void tile_store(const ColCtx<T, N, C>& cx, const T* lds, cplx<T>* __restrict__ dst) {
  using X = ColCtx<T, N, C>;
  constexpr Dims d = dims_of<N>();
  const int c = (int)threadIdx.x % C, y0 = (int)threadIdx.x / C;
  const unsigned at = (unsigned)(y0 * d.NKXP + cx.kx0 + c);
  if (cx.kx0 + c <= kcut<N>()) {
    const cplx<T>* col = reinterpret_cast<const cplx<T>*>(lds + c * X::CS);
#pragma unroll
    for (int k = 0; k < X::E; ++k)
      put32(dst + (size_t)X::NT * k * d.NKXP, at, col[pidx(LaneIdx{y0, X::NT * k})]);
  }
}

// forward column transform of one row-spectrum field A, or of A - i kx B (DX):
// the masked, 1/N^2-normalised right-hand-side values at k = t + NT r
template <typename T, int N, int C, bool DX = false>
__device__ __forceinline__ void column_forward(const ColCtx<T, N, C>& cx, const cplx<T>* A, const cplx<T>* B,
                                               const cplx<T>* __restrict__ tw, cplx<T> (&out)[fft_E<N>()]) {
  using X = ColCtx<T, N, C>;
  tile_load<T, N, C, DX>(cx, A, B, out);
  // with 16 values per lane they come back through the buffer: kept in registers
  // across the last stage, the kernels spill
  fft<T, N, X::E, -1, (X::E < 16)>(out, cx.buf, cx.t, tw);
  if constexpr (X::E >= 16) {
#pragma unroll
    for (int r = 0; r < X::E; ++r) out[r] = reinterpret_cast<const cplx<T>*>(cx.buf)[pidx(LaneIdx{cx.t, X::NT * r})];
  }
  const T inv = T(1.0 / (double(N) * double(N)));
#pragma unroll
  for (int r = 0; r < X::E; ++r) out[r] = {out[r].x * inv, out[r].y * inv};
}

// whether a block's two inverse transforms (a field and its i ky version) run side
// by side in two sets of buffers: on the grids whose columns are bound by latency,
// where a second set leaves room for two blocks per CU.  (Not at 512^2, whose blocks
// fill the chip: one set and four waves per SIMD instead of two sets and three, with
// the state's loads after the transforms, float32 130.7 -> 127.9 us per step, float64
// 182.6 -> 173.0.)
template <typename T, int N, int C>
__host__ __device__ constexpr bool col_dual() {
  return (fft_E<N>() == 4 || fft_E<N>() == 12) && 2 * C * col_buf(N) * sizeof(cplx<T>) <= 80 * 1024;
}
// a column block's LDS, in values of T
template <typename T, int N, int C, bool DUAL = col_dual<T, N, C>()>
__host__ __device__ constexpr int col_lds() {
  return (DUAL ? 2 : 1) * C * ColCtx<T, N, C>::CS;
}

// inverse column transforms of values S at k = t + NT r (already zero outside
// the mask) to the intermediate field dst and, with WITH_DY, of i ky S to dst_dy
template <typename T, int N, int C, bool WITH_DY, bool DUAL = col_dual<T, N, C>()>
__device__ __forceinline__ void column_inverse(const ColCtx<T, N, C>& cx, const cplx<T> (&S)[fft_E<N>()],
                                               cplx<T>* dst, cplx<T>* dst_dy, const cplx<T>* __restrict__ tw) {
  using X = ColCtx<T, N, C>;
  constexpr int E = X::E, NT = X::NT;
  auto value = [&](int r, bool dy) -> cplx<T> {
    const cplx<T> q = S[r];
    if (!dy) return q;
    const int k = cx.t + NT * r;
    const int ky = (k <= N / 2) ? k : k - N;
    return {-T(ky) * q.y, T(ky) * q.x};
  };
  // no barrier: since the last block-wide tile access (whose last barrier every
  // wave has passed) only this lane group has touched its buffer
  if constexpr (WITH_DY && DUAL) {
    cplx<T> v[2][E];
#pragma unroll
    for (int r = 0; r < E; ++r) v[0][r] = value(r, false), v[1][r] = value(r, true);
    constexpr int SECOND = C * X::CS;
    T* const b[2] = {cx.buf, cx.buf + SECOND};
    fft_side_by_side<T, N, E, +1, false, false, 2>(v, b, cx.t, tw);
    __syncthreads();
    tile_store<T, N, C>(cx, cx.lds, dst);
    tile_store<T, N, C>(cx, cx.lds + SECOND, dst_dy);
  } else {
#pragma unroll
    for (int pass = 0; pass < (WITH_DY ? 2 : 1); ++pass) {
      if (pass) __syncthreads();  // the tile before has been read
      cplx<T> v[E];
#pragma unroll
      for (int r = 0; r < E; ++r) v[r] = value(r, pass);
      cplx<T>* out = pass ? dst_dy : dst;
      fft<T, N, E, +1>(v, cx.buf, cx.t, tw);
      __syncthreads();
      tile_store<T, N, C>(cx, cx.lds, out);
    }
  }
}

// Fourier coefficient (the stored kx >= 0 half, 1/N^2-normalised) of u, v or h
// (G = CG_U, CG_V, CG_H) of the prescribed flow at time t: a linear Poincare
// plane wave h' = A cos(theta), theta = k.x - omega t + phase, with the linear
// shallow-water polarisation of section 4.2.1, eq. (4.8), in any direction,
//   u' = A (omega kx cos(theta) - f ky sin(theta)) / (H |k|^2),
//   v' = A (omega ky cos(theta) + f kx sin(theta)) / (H |k|^2),
// plus the uniform flow (U0, V0), and the depth H at k = 0.  With
// cos(theta) = (e^{i theta} + e^{-i theta}) / 2 the +k mode's coefficient is
// (A / 2) C e^{i (phase - omega t)}, C = 1, (omega kx + i f ky) / (H |k|^2) or
// (omega ky - i f kx) / (H |k|^2); a stored entry at -k holds its conjugate.
template <int G>
__device__ cplx<double> kin_coef(int kx, int ky, double t, const Phys& ph) {
  cplx<double> c = {0.0, 0.0};
  if (kx == 0 && ky == 0) c.x = (G == CG_U) ? ph.U0 : (G == CG_V) ? ph.V0 : ph.H;
  const int wx = int(ph.kx), wy = int(ph.ky);
  const bool plus = (kx == wx && ky == wy), minus = (kx == -wx && ky == -wy);
  if ((wx == 0 && wy == 0) || !(plus || minus)) return c;
  const double k2 = ph.kx * ph.kx + ph.ky * ph.ky;
  double cr = 1.0, ci = 0.0;
  if (G == CG_U) {
    cr = ph.omega * ph.kx / (ph.H * k2);
    ci = ph.f * ph.ky / (ph.H * k2);
  } else if (G == CG_V) {
    cr = ph.omega * ph.ky / (ph.H * k2);
    ci = -ph.f * ph.kx / (ph.H * k2);
  }
  double sn, cs;
  sincos(ph.phase - ph.omega * t, &sn, &cs);
  const double a = 0.5 * ph.A;
  cplx<double> m = {a * (cr * cs - ci * sn), a * (cr * sn + ci * cs)};
  if (minus) m.y = -m.y;
  c.x += m.x;
  c.y += m.y;
  return c;
}

// stage >= 0: the RK4 stage; stage < 0: the prologue (the current state's
// column-pass outputs only).  t_next: time of the stage input this launch
// prepares (the prescribed flow of a kinematic run is evaluated there).
// G: the group's kind, g the group itself; groups that differ only in their
// fields' places (xi and P: CG_XIX, the momentum 1-form: CG_GMX, the Eulerian
// means of other fields: CG_EF0) share a kind.
template <typename T, int N, int C, int G>
__device__ __forceinline__ void column_group(const ColCtx<T, N, C>& cx, const StepPtrs<T>& P, const Phys& ph, int g,
                                             int stage, double t_next, const cplx<T>* __restrict__ Ys_in,
                                             cplx<T>* __restrict__ Ys_out) {
  constexpr int E = fft_E<N>(), NT = N / E;
  constexpr bool DBL = G == CG_XIX;
  constexpr bool DYN = (G == CG_U || G == CG_V || G == CG_H);
  constexpr bool EUL = G == CG_EF0;  // Eulerian accumulators of the averaged fields
  using TS = typename std::conditional<DBL, double, T>::type;
  constexpr Dims d = dims_of<N>();
  constexpr size_t sp = d.spec_elems(), rf = d.rowfield_elems();
  if constexpr (EUL) {
    if (stage < 0) return;  // not an input of the rows passes
  }

  // right-hand-side inputs of this group: F0, and for the dynamics F1
  static_assert(RS_PY - RS_XIX == CG_PY - CG_XIX && IC_PY - IC_XIX == 2 * (CG_PY - CG_XIX), "mean groups in field order");
  const int F0 = (G == CG_U) ? RS_ZV : (G == CG_V) ? RS_ZU : (G == CG_H) ? RS_HU : (G == CG_GMX) ? RS_GMX + (g - CG_GMX)
               : EUL ? RS_F0 + (g - CG_EF0) : RS_XIX + (g - CG_XIX);
  constexpr int F1 = (G == CG_U || G == CG_V) ? RS_K : RS_HV;

  // state of this group
  cplx<TS>* Y;
  cplx<TS>* YL = nullptr;  // trailing words of compensated float state
  cplx<TS>* A;
  if constexpr (DBL) {
    const int sd = (g < CG_PX) ? SD_XIX + (g - CG_XIX) : SD_PX + (g - CG_PX);
    Y = P.Yd + sd * sp;
    A = P.Ad + sd * sp;
  } else {
    const int sr = (G == CG_U) ? SF_U : (G == CG_V) ? SF_V : (G == CG_H) ? SF_H : (G == CG_GBH) ? SF_GBH
                 : (G == CG_GBZ) ? SF_GBZ : (G == CG_GTH) ? SF_GTH : (G == CG_GTZ) ? SF_GTZ
                 : (G == CG_GMX) ? SF_GMX + (g - CG_GMX) : SF_EH + (g - CG_EF0);
    Y = reinterpret_cast<cplx<TS>*>(P.Yr) + sr * sp;
    if constexpr (std::is_same<TS, float>::value) YL = reinterpret_cast<cplx<TS>*>(P.Yl) + sr * sp;
    A = reinterpret_cast<cplx<TS>*>(P.Ar) + sr * sp;
  }
  const T fT = T(ph.f), gT = T(ph.g), HT = T(ph.H);

  // the next stage input, in the transforms' precision
  cplx<T> S[E];
  if (stage < 0 || (DYN && ph.kin)) {
    // prologue (the current state's transforms) or a prescribed flow (a kinematic
    // run has no dynamics right-hand sides)
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const ColIdx<N> ix{cx.t, r};
      S[r] = {T(0), T(0)};
      if (ix.none() || !(ix.in() && cx.valid)) continue;
      const unsigned j = cx.ky0 + ix.lane();
      if constexpr (DYN) {
        if (ph.kin) {
          // the next stage input is the prescribed flow at t_next
          const cplx<double> c = kin_coef<G>(cx.kx, ix.ky(), t_next, ph);
          S[r] = {T(c.x), T(c.y)};
          put32(Ys_out + (G - CG_U) * sp + ix.off(), j, S[r]);
          continue;
        }
      }
      const cplx<TS> now = at32(Y + ix.off(), j);
      S[r] = {T(now.x), T(now.y)};
      if constexpr (DYN) put32(Ys_out + (G - CG_U) * sp + ix.off(), j, S[r]);
    }
  } else {
    // RK4 stage.  The coefficients are taken in batches of RB: every load of a
    // batch (stage values, state, accumulator) is issued before its first
    // store, so the batch's loads are in flight together (stores to the state
    // could alias later loads as far as the compiler knows, which would
    // otherwise serialise the coefficients).  With four values per lane (64^2,
    // 128^2, 256^2) one batch takes all of a lane's coefficients, and its loads are
    // issued before the forward transforms (PRE): they wait for memory once, not twice.
    // For the default averaged fields (eta, zeta) the g-tilde groups take their
    // source f from the stage spectra, f = eta (h less H at k = 0) for g-tilde_h
    // and f = i kx v - i ky u for g-tilde_zeta (eq. (4.1): the rows pass formed
    // only - u . grad g-tilde).  The Eulerian accumulators, dE_f/dt = f, the same
    // spectrum with no transform, ride along with the g-tilde groups (even batch
    // positions r, where f is at hand) and the g-bar groups (odd ones), which
    // balances the blocks.  (Other averaged fields: sources in the rows pass,
    // Eulerian means in groups CG_EF0/EF1.)
    constexpr bool EULA = (G == CG_GTH || G == CG_GBH), EULB = (G == CG_GTZ || G == CG_GBZ);
    constexpr bool SRCG = (G == CG_GTH || G == CG_GTZ);
    constexpr int EPAR = SRCG ? 0 : 1;
    const double cn = (stage == 1) ? 0.5 * ph.dt : ph.dt;
    constexpr bool PRE = E == 4;
    constexpr int RB0 = (DBL || DYN || EULA || EULB) ? 2 : 4;  // (4 and 8: spills at 16 values per lane)
    constexpr int RB = PRE ? E : ((E % RB0 == 0) ? RB0 : 4);
    static_assert(E % RB == 0, "coefficient batches");
    cplx<T> su[RB], sv[RB], sh[RB];
    cplx<TS> y[RB], lo[RB], a[RB];
    cplx<T> ey[RB], el[RB], ea[RB];  // Eulerian accumulator
    // acc1, acc3: the accumulator and the trailing words are wanted (stages 1 to 3,
    // and 3); eul: the group carries an Eulerian accumulator.  One line of code for
    // all stages: written once per stage kind, the arrays end up in scratch memory
    // (64^2 float64 44.4 us per step, so 41.2)
    auto load = [&](bool eul, bool acc1, bool acc3, int r0i) {
      auto each = [&](auto f) {
#pragma unroll
        for (int q = 0; q < RB; ++q) {
          const ColIdx<N> ix{cx.t, r0i + q};
          if (!ix.none()) f(q, ix.off(), cx.ky0 + ix.lane(), (r0i + q) % 2 == EPAR);
        }
      };
      constexpr int se = EULA ? SF_EH : SF_EZ;
      each([&](int q, int o, unsigned j, bool) {
        if constexpr (DYN) {
          su[q] = at32(Ys_in + 0 * sp + o, j);
          sv[q] = at32(Ys_in + 1 * sp + o, j);
          sh[q] = at32(Ys_in + 2 * sp + o, j);
        }
        y[q] = at32(Y + o, j);
      });
      if (acc1) each([&](int q, int o, unsigned j, bool) { a[q] = at32(A + o, j); });
      if constexpr (std::is_same<TS, float>::value) {
        if (acc3) each([&](int q, int o, unsigned j, bool) { lo[q] = at32(YL + o, j); });
      }
      if constexpr (EULA || EULB) {
        if (eul) {
          each([&](int q, int o, unsigned j, bool acc) {
            if (SRCG || acc) {
              if constexpr (EULA) {
                sh[q] = at32(Ys_in + 2 * sp + o, j);
              } else {
                su[q] = at32(Ys_in + 0 * sp + o, j);
                sv[q] = at32(Ys_in + 1 * sp + o, j);
              }
            }
            if (acc) ey[q] = at32(P.Yr + se * sp + o, j);
          });
          if (acc1) each([&](int q, int o, unsigned j, bool acc) { if (acc) ea[q] = at32(P.Ar + se * sp + o, j); });
          if constexpr (std::is_same<T, float>::value) {
            if (acc3) each([&](int q, int o, unsigned j, bool acc) { if (acc) el[q] = at32(P.Yl + se * sp + o, j); });
          }
        }
      }
    };
    cplx<T> r0[E];  // the transformed right-hand side
    // kind: the stage's (rk4v)
    auto update = [&](auto kind, auto eulc, int r0i) {
      constexpr int KS = decltype(kind)::value;
      constexpr bool eul = decltype(eulc)::value;
      // a fresh view of the lane's index for every batch: what is computed from it
      // (wavenumbers, the hyperviscosity) stays inside the batch, instead of being
      // formed for all coefficients ahead of the stage kinds' common code
      int t = cx.t;
      if constexpr (!PRE) asm volatile("" : "+v"(t));
#pragma unroll
      for (int q = 0; q < RB; ++q) {
        const int r = r0i + q;
        const ColIdx<N> ix{t, r};
        S[r] = {T(0), T(0)};
        if (ix.none() || !(ix.in() && cx.valid)) continue;
        const int ky = ix.ky(), o = ix.off();
        const unsigned j = cx.ky0 + ix.lane();
        const T kxT = T(cx.kx), kyT = T(ky);
        cplx<T> fsrc = {T(0), T(0)};  // f = eta or zeta from the stage spectra
        if constexpr (EULA || EULB) {
          // dE_eta/dt = eta (h less H at k = 0), dE_zeta/dt = i kx v - i ky u
          const bool acc = r % 2 == EPAR;
          if (eul && (SRCG || acc)) {
            if constexpr (EULA) {
              fsrc = sh[q];
              if (cx.kx == 0 && ky == 0) fsrc.x -= HT;
            } else {
              fsrc = {-kxT * sv[q].y + kyT * su[q].y, kxT * sv[q].x - kyT * su[q].x};
            }
          }
          if (eul && acc) {
            constexpr int se = EULA ? SF_EH : SF_EZ;
            rk4v<KS, T>(ey[q], el[q], ea[q], fsrc, ph.dt, cn);
            rk4_store<KS, T>(P.Yr + se * sp + o, P.Yl + se * sp + o, P.Ar + se * sp + o, j, ey[q], el[q], ea[q]);
          }
        }
        const double k2 = double(cx.kx) * cx.kx + double(ky) * ky;
        const T hv = T(ph.nu8 * (k2 * k2) * (k2 * k2));
        cplx<T> R;
        if constexpr (G == CG_U) {
          // (zeta v - i kx K) + f v - i kx g h - nu8 |k|^8 u
          const cplx<T> u = su[q], v = sv[q], h = sh[q];
          R = {r0[r].x + fT * v.x + kxT * (gT * h.y) - hv * u.x, r0[r].y + fT * v.y - kxT * (gT * h.x) - hv * u.y};
        } else if constexpr (G == CG_V) {
          // (-zeta u - i ky K) - f u - i ky g h - nu8 |k|^8 v
          const cplx<T> u = su[q], v = sv[q], h = sh[q];
          R = {r0[r].x - fT * u.x + kyT * (gT * h.y) - hv * v.x, r0[r].y - fT * u.y - kyT * (gT * h.x) - hv * v.y};
        } else if constexpr (G == CG_H) {
          // (-i kx F(eta u) - i ky F(eta v)) - i kx H u - i ky H v - nu8 |k|^8 h
          const cplx<T> u = su[q], v = sv[q], h = sh[q];
          R = {r0[r].x + kxT * (HT * u.y) + kyT * (HT * v.y) - hv * h.x,
               r0[r].y - kxT * (HT * u.x) - kyT * (HT * v.x) - hv * h.y};
        } else {
          R = r0[r];
          if constexpr (SRCG) R = {R.x + fsrc.x, R.y + fsrc.y};
          (void)hv;
        }
        const cplx<TS> Rk = {TS(R.x), TS(R.y)};
        const cplx<TS> next = rk4v<KS, TS>(y[q], lo[q], a[q], Rk, ph.dt, cn);
        S[r] = {T(next.x), T(next.y)};
        rk4_store<KS, TS>(Y + o, YL + o, A + o, j, y[q], lo[q], a[q]);
        if constexpr (DYN) put32(Ys_out + (G - CG_U) * sp + o, j, S[r]);
      }
    };
    // f(kind, eul) for this launch's stage and run
    auto with_kind = [&](auto&& f) {
      auto by_stage = [&](auto eulc) {
        if (stage == 0) f(std::integral_constant<int, 0>{}, eulc);
        else if (stage < 3) f(std::integral_constant<int, 1>{}, eulc);
        else f(std::integral_constant<int, 3>{}, eulc);
      };
      if constexpr (EULA || EULB) {
        if (!ph.gen) by_stage(std::true_type{});
        else by_stage(std::false_type{});
      } else {
        by_stage(std::false_type{});
      }
    };
    if constexpr (PRE) {
      load(!ph.gen, stage >= 1, stage == 3, 0);
      sched_fence();
    }
    // the transformed products; the dynamics groups' two inputs as one spectrum:
    //   u: zeta v - i kx K   v: -zeta u - i ky K   h: -i kx (eta u) - i ky (eta v)
    // (an i kx joins before the transform, where kx is a column's constant; an i ky
    // after it, its input first, so that one spectrum at a time is in registers)
    if constexpr (G == CG_U) {
      column_forward<T, N, C, true>(cx, P.RS + F0 * rf, P.RS + F1 * rf, P.tw, r0);
    } else if constexpr (G == CG_V || G == CG_H) {
      column_forward<T, N, C>(cx, P.RS + F1 * rf, nullptr, P.tw, r0);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int k = cx.t + NT * r;
        const T ky = T((k <= N / 2) ? k : k - N);
        r0[r] = {ky * r0[r].y, -ky * r0[r].x};
      }
      cplx<T> f[E];
      column_forward<T, N, C>(cx, P.RS + F0 * rf, nullptr, P.tw, f);
      const T kx = T(cx.kx);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        if constexpr (G == CG_V) r0[r] = {r0[r].x - f[r].x, r0[r].y - f[r].y};
        else r0[r] = {r0[r].x + kx * f[r].y, r0[r].y - kx * f[r].x};
      }
    } else {
      column_forward<T, N, C>(cx, P.RS + F0 * rf, nullptr, P.tw, r0);
    }
    with_kind([&](auto kind, auto eulc) {
#pragma unroll
      for (int r0i = 0; r0i < E; r0i += RB) {
        if constexpr (!PRE) {
          constexpr int KS = decltype(kind)::value;
          load(decltype(eulc)::value, KS >= 1, KS == 3, r0i);
          sched_fence();  // the batch's loads together, and none of the next one's with them
        }
        update(kind, eulc, r0i);
        if constexpr (!PRE) sched_fence();
      }
    });
  }

  // inverse column transforms of the next stage input
  if constexpr (G == CG_U) {
    column_inverse<T, N, C, true>(cx, S, P.IC + IC_U * rf, P.IC + IC_UY * rf, P.tw);
  } else if constexpr (G == CG_V) {
    column_inverse<T, N, C, false>(cx, S, P.IC + IC_V * rf, nullptr, P.tw);
  } else if constexpr (G == CG_H) {
    // the rows passes work with eta = h - H: drop H from the mean (k = 0, lane 0)
    if (cx.kx == 0 && cx.t == 0) S[0].x -= T(ph.H);
    column_inverse<T, N, C, false>(cx, S, P.IC + IC_H * rf, nullptr, P.tw);
  } else if constexpr (!EUL) {
    const int o = (G == CG_GMX) ? IC_GMX + 2 * (g - CG_GMX) : IC_XIX + 2 * (g - CG_XIX);
    column_inverse<T, N, C, true>(cx, S, P.IC + o * rf, P.IC + (o + 1) * rf, P.tw);
  }
}

// stage >= 0: RK4 stage; stage < 0: only transform the current state (prologue)
template <typename T, int N, int C>
__device__ __forceinline__ void columns_body(const StepPtrs<T>& P, const Phys& ph, int stage, double t_next,
                                             const cplx<T>* Ys_in, cplx<T>* Ys_out, int tile, int slot, T* lds) {
  const ColCtx<T, N, C> cx(lds, tile);
  const int g = col_group_of(ph, slot);
#define LM_CG(k) column_group<T, N, C, k>(cx, P, ph, g, stage, t_next, Ys_in, Ys_out)
  switch (g) {
    case CG_U: LM_CG(CG_U); break;
    case CG_V: LM_CG(CG_V); break;
    case CG_H: LM_CG(CG_H); break;
    case CG_GBH: LM_CG(CG_GBH); break;
    case CG_GBZ: LM_CG(CG_GBZ); break;
    case CG_GTH: LM_CG(CG_GTH); break;
    case CG_GTZ: LM_CG(CG_GTZ); break;
    case CG_GMX: case CG_GMY: LM_CG(CG_GMX); break;
    case CG_EF0: case CG_EF1: LM_CG(CG_EF0); break;
    default: LM_CG(CG_XIX); break;  // xi_x, xi_y, P_x, P_y
  }
#undef LM_CG
}

// --------------------------------------------------------------------------
// the launches of a stage
// --------------------------------------------------------------------------
// Large grids: three passes in order, rows of the dynamics and strategy 1, rows of
// strategy 2, all column groups.
//
// Small grids (stage_merged): blocks of a rows pass and of the column groups that
// do not depend on it share a launch; stage i is
//   A(i)  dynamics and strategy-1 rows of stage i, with the strategy-2 (and
//         momentum) column groups of stage i - 1
//   B(i)  strategy-2 rows of stage i, with the dynamics and strategy-1 column
//         groups of stage i (their inputs came with A(i))
// so a stage has two launch boundaries instead of three, and two chains side by
// side.  Every block does what it would in a launch of its own.  Neither part of a
// launch writes what the other reads: A's columns write the strategy-2 state and
// inputs, which only B's rows read; its rows write the physical fields and the
// dynamics' and strategy-1 row spectra; B's columns write those groups' state,
// inputs and the other stage-value buffer.  A launch of one kind alone is the same
// kernel with no blocks of the other.  Measured per step, three passes -> two
// launches: 64^2 float64 59.1 -> 44.4 us, 128^2 float32 62.2 -> 53.9, 192^2 float32
// 99.6 -> 67.8, 256^2 float64 100.4 -> 96.7, 384^2 float32 141 -> 116 (41.2, 49.4,
// 68.7, 87.8 and 105 with the state's loads in one straight line and the tiles
// tuned).  512^2 and 1024^2 keep the passes apart: their passes fill the chip, and with
// the columns as they were then the larger of the two parts' registers and LDS cost
// both (512^2 float32 130.6 -> 139.3).  That no longer holds: with one set of buffers
// and four waves per SIMD in the columns, merged launches would be the faster at the
// best tile of each form (apart / merged, from one state: 512^2 float32 123.8 / 114.3,
// float64 162.7 / 156.3, 1024^2 float32 316.6 / 308.2, float64 664.6 / 634.3, all but
// the first with the half-width tile); the line has not been moved yet.
template <typename T, int N>
__host__ __device__ constexpr bool stage_merged() { return N < 512; }

// Runs of a batched group up to which its launches are merged.  Merging pays while a
// pass leaves the chip idle; once the row blocks fill it, they only lose by the column
// groups' registers (rows of 64^2 to 256^2 take about 50 VGPRs in float32 and 75 in
// float64 in kernels of their own, 118 and 175 here).  Those registers leave 4096
// (float32) or 2048 (float64) waves resident, 640 or 320 blocks of launch A's six row
// waves, and there both sides measure the same.  With twelve values per lane the
// passes apart are less efficient: 8 and 14 runs.  A step, merged / apart, us: 64^2
// float64 12 runs 73 / 80, 64 runs 237 / 190; 128^2 float32 8 runs 90 / 94, 12 runs
// 127 / 123, 64 runs 470 / 419; 128^2 float64 5 runs 112 / 120, 64 runs 921 / 742;
// 192^2 float64 12 runs 311 / 336, 64 runs 1630 / 1481; 256^2 float32 2 runs 103 / 105,
// 12 runs 352 / 306, 64 runs 2190 / 1870; 256^2 float64 1 run 111 / 113, 16 runs
// 991 / 726, 64 runs 3945 / 2865; 384^2 float32 7 runs 382 / 399, 16 runs 1063 / 980.
template <typename T, int N>
__host__ __device__ constexpr int batch_merged_runs() {
  constexpr bool f32 = sizeof(T) == 4;
  if (!stage_merged<T, N>()) return 0;
  if (fft_E<N>() == 12) return f32 ? 8 : 14;
  return (f32 ? 640 : 320) / (N / CoopGeo<T, N>::WR);
}

// Tile width of a batched group's columns for the schedule's: half-width tiles are for
// few blocks, so a group of eight runs or more in passes apart takes at least the
// default (half / default, us a step: 256^2 float32 5 runs 171 / 170, 8 runs 230 / 228,
// 12 runs 312 / 306, 64 runs 1965 / 1870; 192^2 float32 12 runs 207 / 202, 64 runs
// 967 / 920; 384^2 float32 16 runs 1016 / 980; but one run of 256^2, merged, 77 / 88).
template <typename T, int N>
__host__ __device__ constexpr int batch_tile(int nruns, int tile) {
  return stage_merged<T, N>() && nruns >= 8 && nruns > batch_merged_runs<T, N>() && tile < 0 ? 0 : tile;
}

template <typename T, int N, int W, int ROW_THREADS, int ROW_LDS>
struct StageGeo {
  static constexpr int C = col_tile<N, W>(), COL_THREADS = col_threads<N, W>();
  static constexpr int THREADS = COL_THREADS > ROW_THREADS ? COL_THREADS : ROW_THREADS;
  static constexpr int LDS = col_lds<T, N, C>() > ROW_LDS ? col_lds<T, N, C>() : ROW_LDS;  // values of T
  static constexpr int TILES = (dims_of<N>().NKX + C - 1) / C;
  static constexpr int ROWS = N / CoopGeo<T, N>::WR;  // row blocks of a run
  static_assert(COL_THREADS % 64 == 0 && THREADS <= 1024 && ROWS % 8 == 0, "stage blocks");
};
template <typename T, int N, int W>
using StageA = StageGeo<T, N, W, DynGeo<T, N>::THREADS, DynGeo<T, N>::LDS>;
template <typename T, int N, int W>
using StageB = StageGeo<T, N, W, RhsGeo<T, N>::THREADS, RhsGeo<T, N>::LDS>;

// Resident waves per SIMD the column groups' registers leave room for: from 512
// on in float32 4 (at most 128 registers), in float64 2; smaller grids, which do not
// fill the chip, are not held to that (with four values per lane a lane's whole state
// is in registers).
template <typename T, int N>
__host__ __device__ constexpr int col_waves() {
  return N >= 512 ? (sizeof(T) == 4 ? 4 : 2) : (sizeof(T) == 4 ? 2 : 1);
}

// the column pass (grid = (column tiles, group slots)), slots from slot0 on
template <typename T>
struct ColArgs {
  int stage, slot0, nslot, cols;  // stage < 0: the prologue; cols: column blocks (merged launches)
  double t_next;
  const cplx<T>* Ys_in;
  cplx<T>* Ys_out;
};

// W: column tile width (col_tile<N, W>)
template <typename T, int N, int W>
__global__ void __launch_bounds__((col_threads<N, W>()), (col_waves<T, N>()))
    k_columns(StepPtrs<T> P, Phys ph, ColArgs<T> ca, int remap) {
  constexpr int C = col_tile<N, W>();
  static_assert(col_threads<N, W>() % 64 == 0 && col_threads<N, W>() <= 1024, "column block");
  __shared__ __align__(16) T lds[col_lds<T, N, C>()];
  int tile, slot, z;
  xcd_split(gridDim.x, gridDim.y, tile, slot, z, remap);
  columns_body<T, N, C>(P, ph, ca.stage, ca.t_next, ca.Ys_in, ca.Ys_out, tile, ca.slot0 + slot, lds);
}

// what a block of a stage launch is: column blocks come first (cols of them, a
// multiple of 8, of which nslot * TILES * runs do work), then row blocks.
// Workgroups go round-robin to the 8 XCDs (each with its own L2): with remap every
// XCD gets a contiguous run of column tiles (all groups of a tile next to each
// other) and of rows, as xcd_split.
struct StageRole {
  bool col, idle;
  int tile, slot, row, run;
};
template <typename S>
__device__ __forceinline__ StageRole stage_role(unsigned cols, unsigned nslot, unsigned runs, unsigned rows, int remap) {
  StageRole r{};
  const unsigned b = blockIdx.x, x = b % NUM_XCD;
  r.col = b < cols;
  if (r.col) {
    const unsigned i = remap ? x * (cols / NUM_XCD) + b / NUM_XCD : b;
    r.idle = i >= nslot * S::TILES * runs;
    r.slot = (int)(i % nslot);
    const unsigned rest = i / nslot;
    r.tile = (int)(rest % S::TILES);
    r.run = (int)(rest / S::TILES);
  } else {
    const unsigned bb = b - cols;
    const unsigned i = remap ? x * (rows / NUM_XCD) + bb / NUM_XCD : bb;
    r.row = (int)(i % S::ROWS);
    r.run = (int)(i / S::ROWS);
  }
  return r;
}

template <typename T, int N, int W>
__global__ void __launch_bounds__((StageA<T, N, W>::THREADS), (col_waves<T, N>()))
    k_stage_a(StepPtrs<T> P, Phys ph, double s, ColArgs<T> ca, int rows, int remap) {
  using S = StageA<T, N, W>;
  __shared__ __align__(16) T lds[S::LDS];
  const StageRole r = stage_role<S>(ca.cols, ca.nslot, 1, rows, remap);
  if (r.col) {
    if (r.idle || threadIdx.x >= S::COL_THREADS) return;
    columns_body<T, N, S::C>(P, ph, ca.stage, ca.t_next, ca.Ys_in, ca.Ys_out, r.tile, ca.slot0 + r.slot, lds);
  } else {
    if (threadIdx.x >= DynGeo<T, N>::THREADS) return;
    rows_dyn_body<T, N, false>(P, ph, s, r.row, lds);
  }
}

template <typename T, int N, int W>
__global__ void __launch_bounds__((StageB<T, N, W>::THREADS), (col_waves<T, N>()))
    k_stage_b(StepPtrs<T> P, Phys ph, double s, ColArgs<T> ca, int rows, int remap) {
  using S = StageB<T, N, W>;
  __shared__ __align__(16) T lds[S::LDS];
  const StageRole r = stage_role<S>(ca.cols, ca.nslot, 1, rows, remap);
  if (r.col) {
    if (r.idle || threadIdx.x >= S::COL_THREADS) return;
    columns_body<T, N, S::C>(P, ph, ca.stage, ca.t_next, ca.Ys_in, ca.Ys_out, r.tile, ca.slot0 + r.slot, lds);
  } else {
    if (threadIdx.x >= RhsGeo<T, N>::THREADS) return;
    rows_rhs_body<T, N, false>(P, s, r.row, lds);
  }
}

// --------------------------------------------------------------------------
// batched entry points: the launches of many runs of one (N, precision) group
// --------------------------------------------------------------------------

// time since the interval start at a stage, from integers (as the single-run path)
template <typename T>
__device__ __forceinline__ double batch_s(const RunDesc<T>& R, int stage) {
  const double c = (stage == 0) ? 0.0 : ((stage == 3) ? 1.0 : 0.5);
  return (double(*R.counter) + c) * R.ph.dt;
}

template <typename T, int N, bool GEN>
__global__ void __launch_bounds__((DynGeo<T, N>::THREADS), (DynGeo<T, N>::min_waves(GEN)))
    k_rows_dyn_b(const RunDesc<T>* __restrict__ runs, int stage, int remap) {
  __shared__ __align__(16) T lds[DynGeo<T, N>::LDS];
  int rowblock, unused, z;
  xcd_split(gridDim.x, 1, rowblock, unused, z, remap);
  const RunDesc<T>& R = runs[z];
  rows_dyn_body<T, N, GEN>(R.P, R.ph, batch_s(R, stage), rowblock, lds);
}

template <typename T, int N, bool CUB>
__global__ void __launch_bounds__((CUB ? RhsGeo<T, N>::CUB_THREADS : RhsGeo<T, N>::THREADS), (RhsGeo<T, N>::min_waves(CUB)))
    k_rows_rhs_b(const RunDesc<T>* __restrict__ runs, int stage, int remap) {
  __shared__ __align__(16) T lds[RhsGeo<T, N>::LDS];
  int rowblock, unused, z;
  xcd_split(gridDim.x, 1, rowblock, unused, z, remap);
  const RunDesc<T>& R = runs[z];
  rows_rhs_body<T, N, CUB>(R.P, batch_s(R, stage), rowblock, lds);
}

template <typename T, int N, bool CUB>
__global__ void __launch_bounds__((MomGeo<T, N>::THREADS), (MomGeo<T, N>::min_waves(CUB)))
    k_rows_mom_b(const RunDesc<T>* __restrict__ runs, int stage, int remap) {
  __shared__ __align__(16) T lds[MomGeo<T, N>::LDS];
  int rowblock, unused, z;
  xcd_split(gridDim.x, 1, rowblock, unused, z, remap);
  const RunDesc<T>& R = runs[z];
  rows_mom_body<T, N, CUB>(R.P, batch_s(R, stage), rowblock, lds);
}

// the column part of a batched launch; stage parity selects the stage-value
// buffers: between steps the current stage input is always Ys0 (four swaps per step)
template <typename T, int N, int C>
__device__ __forceinline__ void columns_run(const RunDesc<T>& R, int stage, int tile, int slot, T* lds) {
  const cplx<T>* Ys_in = (stage & 1) ? R.Ys1 : R.Ys0;
  cplx<T>* Ys_out = (stage & 1) ? R.Ys0 : R.Ys1;
  // time of the next stage input, from integers (as the single-run path)
  const double cn = (stage <= 1) ? 0.5 : 1.0;
  const double t_next = (double(R.n_tau + *R.counter) + cn) * R.ph.dt;
  columns_body<T, N, C>(R.P, R.ph, stage, t_next, Ys_in, Ys_out, tile, slot, lds);
}

template <typename T, int N, int W>
__global__ void __launch_bounds__((col_threads<N, W>()), (col_waves<T, N>()))
    k_columns_b(const RunDesc<T>* __restrict__ runs, int stage, int remap) {
  constexpr int C = col_tile<N, W>();
  __shared__ __align__(16) T lds[col_lds<T, N, C>()];
  int tile, slot, z;
  xcd_split(gridDim.x, gridDim.y, tile, slot, z, remap);
  columns_run<T, N, C>(runs[z], stage, tile, slot, lds);
}

// stage: of the rows; the columns are those of cstage
template <typename T, int N, int W>
__global__ void __launch_bounds__((StageA<T, N, W>::THREADS), (col_waves<T, N>()))
    k_stage_a_b(const RunDesc<T>* __restrict__ runs, int nruns, int stage, int cstage, int slot0, int nslot, int cols,
                int rows, int remap) {
  using S = StageA<T, N, W>;
  __shared__ __align__(16) T lds[S::LDS];
  const StageRole r = stage_role<S>(cols, nslot, nruns, rows, remap);
  if (r.col) {
    if (r.idle || threadIdx.x >= S::COL_THREADS) return;
    columns_run<T, N, S::C>(runs[r.run], cstage, r.tile, slot0 + r.slot, lds);
  } else {
    if (threadIdx.x >= DynGeo<T, N>::THREADS) return;
    const RunDesc<T>& R = runs[r.run];
    rows_dyn_body<T, N, false>(R.P, R.ph, batch_s(R, stage), r.row, lds);
  }
}

template <typename T, int N, int W>
__global__ void __launch_bounds__((StageB<T, N, W>::THREADS), (col_waves<T, N>()))
    k_stage_b_b(const RunDesc<T>* __restrict__ runs, int nruns, int stage, int cstage, int slot0, int nslot, int cols,
                int rows, int remap) {
  using S = StageB<T, N, W>;
  __shared__ __align__(16) T lds[S::LDS];
  const StageRole r = stage_role<S>(cols, nslot, nruns, rows, remap);
  if (r.col) {
    if (r.idle || threadIdx.x >= S::COL_THREADS) return;
    columns_run<T, N, S::C>(runs[r.run], cstage, r.tile, slot0 + r.slot, lds);
  } else {
    if (threadIdx.x >= RhsGeo<T, N>::THREADS) return;
    const RunDesc<T>& R = runs[r.run];
    rows_rhs_body<T, N, false>(R.P, batch_s(R, stage), r.row, lds);
  }
}

}  // namespace lm
