// Batched 1-D complex FFTs held by groups of lanes (gfx950, 64-wide wavefronts).
//
// An N-point transform is owned by NT = N / E consecutive lanes; lane t of the
// group holds E complex values.  On entry lane t holds x[t + NT * e] in v[e]
// (e = 0..E-1).  The first Stockham stage is a radix-E DFT done in registers;
// later stages (radices R dividing E, each lane doing E/R butterflies) exchange
// data through the group's private LDS buffer.  On exit the spectrum is in the
// lanes' registers (lane t: entries t + NT e) or, if asked for, in the LDS
// buffer in natural order (padded indexing).  A group lies in one wavefront
// (NT <= 64), so the exchanges only need wavefront-scope ordering.
//
// Stockham autosort formulation (decimation in time): at a stage with radix R
// applied after sub-transforms of length Ns, butterfly j (0 <= j < N/R) reads
// in[j + r N/R], multiplies by w_{Ns R}^{r (j mod Ns)}, does an R-point DFT and
// writes out[(j / Ns) Ns R + (j mod Ns) + r Ns], with twiddle w_N^m,
// m = r (j mod Ns) N / (Ns R).  The twiddles (host-computed in long double) are
// stored stage by stage: the block of a stage holds entry (r - 1) Ns + k =
// exp(-2 pi i r k / (Ns R)) for r = 1..R-1, k < Ns, so the lanes of a wavefront
// (consecutive j) read consecutive entries of one block, a few cache lines per
// load instead of one line per lane.
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>

namespace lm {

template <typename T>
struct cplx {
  T x, y;
};

template <typename T>
__device__ __forceinline__ cplx<T> operator+(cplx<T> a, cplx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ cplx<T> operator-(cplx<T> a, cplx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ cplx<T> cmul(cplx<T> a, cplx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
// a * conj(b)
template <typename T>
__device__ __forceinline__ cplx<T> cmulc(cplx<T> a, cplx<T> b) {
  return {a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y};
}
// multiply by -i (DIR = -1, forward) or +i (DIR = +1, inverse)
template <int DIR, typename T>
__device__ __forceinline__ cplx<T> rot90(cplx<T> a) {
  if constexpr (DIR < 0) return {a.y, -a.x};
  else return {-a.y, a.x};
}

// wavefront-scope ordering of LDS traffic between lanes of one wave
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// keeps the instruction scheduler from moving work (in particular global loads)
// across phase boundaries, which would keep many loads in flight in registers
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// padded LDS index: one spare complex slot every 16 spreads strided accesses
// over the banks
__device__ __forceinline__ constexpr int pidx(int i) { return i + (i >> 4); }
__host__ __device__ constexpr int padded_len(int n) { return n + (n >> 4) + 1; }

// an index made of a lane's part and a constant of the unrolled loops: their
// padded index is split the same way where the constant is a multiple of the
// padding period, so that one address register and immediate offsets serve a
// whole unrolled access
struct LaneIdx {
  int v, c;
};
__device__ __forceinline__ int pidx(LaneIdx i) {
  return (i.c % 16 == 0) ? pidx(i.v) + i.c + (i.c >> 4) : pidx(i.v + i.c);
}

// ---------------------------------------------------------------------------
// small DFTs, y_q = sum_r v_r exp(DIR * 2 pi i r q / R)
// ---------------------------------------------------------------------------
template <int DIR, typename T>
__device__ __forceinline__ void dft2(cplx<T>& a, cplx<T>& b) {
  cplx<T> t = a - b;
  a = a + b;
  b = t;
}

template <int DIR, typename T>
__device__ __forceinline__ void dft4(cplx<T>& v0, cplx<T>& v1, cplx<T>& v2, cplx<T>& v3) {
  cplx<T> t0 = v0 + v2, t1 = v0 - v2, t2 = v1 + v3, t3 = rot90<DIR>(v1 - v3);
  v0 = t0 + t2;
  v2 = t0 - t2;
  v1 = t1 + t3;
  v3 = t1 - t3;
}

template <int DIR, typename T>
__device__ __forceinline__ void dft8(cplx<T>* v) {
  constexpr T s = T(0.70710678118654752440084436210484903928);
  // even / odd halves
  cplx<T> e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
  cplx<T> o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
  dft4<DIR>(e0, e1, e2, e3);
  dft4<DIR>(o0, o1, o2, o3);
  // o_q *= w8^q, w8 = exp(DIR i pi / 4)
  cplx<T> w1 = {s, T(DIR) * s};
  cplx<T> w3 = {-s, T(DIR) * s};
  o1 = cmul(o1, w1);
  o2 = rot90<DIR>(o2) ;
  // rot90 gives multiplication by DIR*i which is w8^2 = exp(DIR i pi/2)
  o3 = cmul(o3, w3);
  v[0] = e0 + o0; v[4] = e0 - o0;
  v[1] = e1 + o1; v[5] = e1 - o1;
  v[2] = e2 + o2; v[6] = e2 - o2;
  v[3] = e3 + o3; v[7] = e3 - o3;
}

template <int DIR, typename T>
__device__ __forceinline__ void dft16(cplx<T>* v) {
  constexpr T c1 = T(0.92387953251128675612818318939678828682);  // cos(pi/8)
  constexpr T s1 = T(0.38268343236508977172845998403039886676);  // sin(pi/8)
  constexpr T h = T(0.70710678118654752440084436210484903928);
  // inner radix-4 DFTs over r1 for each r2: X_{r2}[q1] = sum_r1 v[4 r1 + r2] w4^{r1 q1}
  cplx<T> X[16];
#pragma unroll
  for (int r2 = 0; r2 < 4; ++r2) {
    cplx<T> a = v[r2], b = v[4 + r2], c = v[8 + r2], d = v[12 + r2];
    dft4<DIR>(a, b, c, d);
    X[r2 * 4 + 0] = a;
    X[r2 * 4 + 1] = b;
    X[r2 * 4 + 2] = c;
    X[r2 * 4 + 3] = d;
  }
  // twiddle w16^{r2 q1}, w16 = exp(DIR 2 pi i / 16)
  const T sg = T(DIR);
  const cplx<T> w1 = {c1, sg * s1}, w2 = {h, sg * h}, w3 = {s1, sg * c1};
  const cplx<T> w6 = {-h, sg * h}, w9 = {-c1, -sg * s1};
  // r2 = 1: q1 = 1,2,3 -> w1, w2, w3
  X[5] = cmul(X[5], w1);
  X[6] = cmul(X[6], w2);
  X[7] = cmul(X[7], w3);
  // r2 = 2: w2, w4 (= DIR i), w6
  X[9] = cmul(X[9], w2);
  X[10] = rot90<DIR>(X[10]);
  X[11] = cmul(X[11], w6);
  // r2 = 3: w3, w6, w9
  X[13] = cmul(X[13], w3);
  X[14] = cmul(X[14], w6);
  X[15] = cmul(X[15], w9);
  // outer radix-4 over r2: y[q1 + 4 q2] = sum_r2 X_{r2}[q1] w4^{r2 q2}
#pragma unroll
  for (int q1 = 0; q1 < 4; ++q1) {
    cplx<T> a = X[q1], b = X[4 + q1], c = X[8 + q1], d = X[12 + q1];
    dft4<DIR>(a, b, c, d);
    v[q1] = a;
    v[q1 + 4] = b;
    v[q1 + 8] = c;
    v[q1 + 12] = d;
  }
}

template <int DIR, typename T>
__device__ __forceinline__ void dft3(cplx<T>& a, cplx<T>& b, cplx<T>& c) {
  constexpr T h = T(0.86602540378443864676372317075293618347);  // sqrt(3)/2
  const cplx<T> t1 = b + c;
  const cplx<T> t2 = {a.x - T(0.5) * t1.x, a.y - T(0.5) * t1.y};
  const cplx<T> d = b - c;
  // t3 = DIR i (sqrt 3 / 2) (b - c)
  const cplx<T> t3 = (DIR < 0) ? cplx<T>{h * d.y, -h * d.x} : cplx<T>{-h * d.y, h * d.x};
  a = a + t1;
  b = t2 + t3;
  c = t2 - t3;
}

// 12 = 3 x 4: inner radix-3 DFTs over r1 (r = 4 r1 + r2), twiddles w12^{r2 q1},
// outer radix-4 DFTs over r2, output index q = q1 + 3 q2
template <int DIR, typename T>
__device__ __forceinline__ void dft12(cplx<T>* v) {
  constexpr T c6 = T(0.86602540378443864676372317075293618347);  // cos(pi/6)
  cplx<T> X[12];
#pragma unroll
  for (int r2 = 0; r2 < 4; ++r2) {
    cplx<T> a = v[r2], b = v[4 + r2], c = v[8 + r2];
    dft3<DIR>(a, b, c);
    X[r2 * 3 + 0] = a;
    X[r2 * 3 + 1] = b;
    X[r2 * 3 + 2] = c;
  }
  const T sg = T(DIR);
  const cplx<T> w1 = {c6, sg * T(0.5)}, w2 = {T(0.5), sg * c6}, w4 = {T(-0.5), sg * c6};
  // r2 = 1: q1 = 1, 2 -> w1, w2; r2 = 2: w2, w4; r2 = 3: w3 = DIR i, w6 = -1
  X[4] = cmul(X[4], w1);
  X[5] = cmul(X[5], w2);
  X[7] = cmul(X[7], w2);
  X[8] = cmul(X[8], w4);
  X[10] = rot90<DIR>(X[10]);
  X[11] = {-X[11].x, -X[11].y};
#pragma unroll
  for (int q1 = 0; q1 < 3; ++q1) {
    cplx<T> a = X[q1], b = X[3 + q1], c = X[6 + q1], d = X[9 + q1];
    dft4<DIR>(a, b, c, d);
    v[q1] = a;
    v[q1 + 3] = b;
    v[q1 + 6] = c;
    v[q1 + 9] = d;
  }
}

template <int R, int DIR, typename T>
__device__ __forceinline__ void dft(cplx<T>* v) {
  if constexpr (R == 2) {
    dft2<DIR>(v[0], v[1]);
  } else if constexpr (R == 4) {
    dft4<DIR>(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 8) {
    dft8<DIR>(v);
  } else if constexpr (R == 16) {
    dft16<DIR>(v);
  } else if constexpr (R == 3) {
    dft3<DIR>(v[0], v[1], v[2]);
  } else if constexpr (R == 12) {
    dft12<DIR>(v);
  } else {
    static_assert(R == 2 || R == 3 || R == 4 || R == 8 || R == 12 || R == 16, "unsupported radix");
  }
}

// ---------------------------------------------------------------------------
// plans: N = E * R2 * R3 * R4 with E values per lane; the first stage is a
// radix-E DFT in registers, the later radices divide E
// ---------------------------------------------------------------------------
struct Radices {
  int R2, R3, R4;
};
__host__ __device__ constexpr Radices plan_of(int n, int e) {
  if (e == 16) {
    if (n == 1024) return {16, 4, 1};
  } else if (e == 8) {
    if (n == 512) return {8, 8, 1};
  } else if (e == 4) {
    switch (n) {
      case 64: return {4, 4, 1};
      case 128: return {4, 4, 2};
      case 256: return {4, 4, 4};
      default: break;
    }
  } else if (e == 12) {
    if (n == 192) return {4, 4, 1};
    if (n == 384) return {4, 4, 2};
  }
  return {0, 0, 0};
}
template <int N, int E>
struct Plan {
  static constexpr Radices p = plan_of(N, E);
  static_assert(p.R2 > 0 && E * p.R2 * p.R3 * p.R4 == N, "no FFT plan for this length");
  static constexpr int R2 = p.R2, R3 = p.R3, R4 = p.R4;
};

// offset of stage s (0, 1, 2: the stages of radix R2, R3, R4) in the stage-by-
// stage twiddle table, and the table's length (at most n for every plan)
__host__ __device__ constexpr int tw_offset(int n, int e, int s) {
  const Radices p = plan_of(n, e);
  const int R[3] = {p.R2, p.R3, p.R4};
  int off = 0, ns = e;
  for (int i = 0; i < s; ++i) {
    if (R[i] > 1) off += (R[i] - 1) * ns;
    ns *= R[i];
  }
  return off;
}
__host__ __device__ constexpr int tw_len(int n, int e) { return tw_offset(n, e, 3); }

// values per lane of the column and row passes.  A step of a small grid is bound
// by the latency of its dependent chains, not by the chip's rates: fewer values
// shorten a lane's work per butterfly stage and give more waves, at the price of
// one more exchange.  N <= 256: 4 (measured per step, 8 -> 4 values: 64^2 float64
// 67.8 -> 58.8 us, float32 68.2 -> 53.6, 128^2 float32 72.5 -> 62.2, 256^2 float64
// 114.9 -> 100.5).  N = 512: 8 (16 -> 8: float32 155 -> 131, float64 198 -> 183).
// N = 1024: 16, so that a transform stays inside one wavefront.  N = 3 * 2^k: 12
// (first stage radix 12 = 3 x 4; the lanes of a transform have to divide a wave).
__host__ __device__ constexpr int fft_E_of(int n) {
  return (n % 3 == 0) ? 12 : (n <= 256 ? 4 : n <= 512 ? 8 : 16);
}
template <int N>
__host__ __device__ constexpr int fft_E() { return fft_E_of(N); }

// exchanges of a transform owned by NT lanes: wavefront-scope ordering
template <int NT>
__device__ __forceinline__ void xsync() {
  static_assert(NT <= 64, "a transform lives in one wavefront");
  wave_sync();
}

// the twiddle table lives in global memory: loads through this pointer type
// are global (not generic) loads, which do not hold up the LDS counter
template <typename T>
using gptr = const __attribute__((address_space(1))) cplx<T>*;

// Registers -> the group's buffer -> registers: value i of a lane goes to entry
// wi(i), and entry ri(i) comes back, for M transforms side by side (a buffer
// each).  SPLIT: real and imaginary parts one after the other through a buffer of
// reals, half the LDS for twice the instructions (the bytes are the same).
template <typename T, int E, int NT, bool SPLIT, int M, typename WI, typename RI>
__device__ __forceinline__ void exchange(cplx<T> (&v)[M][E], T* const (&buf)[M], WI wi, RI ri) {
  if constexpr (!SPLIT) {
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int i = 0; i < E; ++i) reinterpret_cast<cplx<T>*>(buf[m])[pidx(wi(i))] = v[m][i];
    xsync<NT>();
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int i = 0; i < E; ++i) v[m][i] = reinterpret_cast<const cplx<T>*>(buf[m])[pidx(ri(i))];
    xsync<NT>();
  } else {
    static_assert(M == 1, "split exchanges are made one transform at a time");
#pragma unroll
    for (int i = 0; i < E; ++i) buf[0][pidx(wi(i))] = v[0][i].x;
    xsync<NT>();
#pragma unroll
    for (int i = 0; i < E; ++i) v[0][i].x = buf[0][pidx(ri(i))];
    xsync<NT>();
#pragma unroll
    for (int i = 0; i < E; ++i) buf[0][pidx(wi(i))] = v[0][i].y;
    xsync<NT>();
#pragma unroll
    for (int i = 0; i < E; ++i) v[0][i].y = buf[0][pidx(ri(i))];
    xsync<NT>();
  }
}

// one Stockham stage of radix R after sub-transforms of length Ns (Ns > 1) on
// values in registers, v[b R + r] = entry t + NT b + r N / R, of M transforms
// side by side; tw: the stage's twiddle block
template <typename T, int N, int E, int DIR, int Ns, int R, int M>
__device__ __forceinline__ void stockham_stage(cplx<T> (&v)[M][E], int t, gptr<T> tw) {
  constexpr int NT = N / E, NB = E / R;
  static_assert(E % R == 0, "radix must divide E");
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int k = (t + b * NT) % Ns;
#pragma unroll
    for (int r = 1; r < R; ++r) {
      const cplx<T> w = {tw[(r - 1) * Ns + k].x, tw[(r - 1) * Ns + k].y};
#pragma unroll
      for (int m = 0; m < M; ++m) v[m][b * R + r] = (DIR < 0) ? cmul(v[m][b * R + r], w) : cmulc(v[m][b * R + r], w);
      if (R == 16 && r % 5 == 0) sched_fence();  // five twiddles in flight
    }
#pragma unroll
    for (int m = 0; m < M; ++m) dft<R, DIR>(&v[m][b * R]);
  }
}

// entry that stage output i = b R + r of lane t belongs to
template <int N, int E, int Ns, int R>
__device__ __forceinline__ LaneIdx stage_out(int i, int t) {
  constexpr int NT = N / E;
  const int b = i / R, r = i % R;
  if constexpr (NT % Ns == 0) return {(t / Ns) * Ns * R + t % Ns, b * NT * R + r * Ns};
  else if constexpr (Ns % NT == 0) return {t, (b * NT / Ns) * Ns * R + (b * NT) % Ns + r * Ns};
  const int j = t + b * NT;
  return {(j / Ns) * Ns * R + j % Ns, r * Ns};
}
// entry that a stage of radix R takes as its input i
template <int N, int E, int R>
__device__ __forceinline__ LaneIdx stage_in(int i, int t) {
  return {t, (i / R) * (N / E) + (i % R) * (N / R)};
}

// swap of 32-bit words between lane rows (16 lanes) of two registers:
// ROWS = 16: odd rows of a with even rows of b; ROWS = 32: rows 2, 3 of a with
// rows 0, 1 of b (v_permlane16_swap / v_permlane32_swap)
template <int ROWS, typename V>
__device__ __forceinline__ void lane_swap(V& a, V& b) {
  static_assert(sizeof(V) % 4 == 0, "32-bit words");
  constexpr int W = sizeof(V) / 4;
  unsigned wa[W], wb[W];
  __builtin_memcpy(wa, &a, sizeof(V));
  __builtin_memcpy(wb, &b, sizeof(V));
#pragma unroll
  for (int i = 0; i < W; ++i) {
    if constexpr (ROWS == 16) {
      const auto r = __builtin_amdgcn_permlane16_swap(wa[i], wb[i], false, false);
      wa[i] = r[0];
      wb[i] = r[1];
    } else {
      const auto r = __builtin_amdgcn_permlane32_swap(wa[i], wb[i], false, false);
      wa[i] = r[0];
      wb[i] = r[1];
    }
  }
  __builtin_memcpy(&a, wa, sizeof(V));
  __builtin_memcpy(&b, wb, sizeof(V));
}

// The last two stages of N = 1024 = 256 G, G = 4 (16 values per lane, NT = 16 G
// lanes, radix 16 then radix G) with the exchange between them done across
// lanes instead of through LDS.  After the radix-16 stage, lane t = c + 16 q
// (c < 16) holds entry 256 q + c + 16 r in x[r]; with r = G a + s that entry is
// element A q + a (A = 16 / G) of lane c + 16 s in the last stage's layout
// (entry t' + NT m in element m of lane t').  So the exchange is a G x G
// transpose over q and s among the lanes c + 16 q, done with row swaps, after
// which x[G a + k] holds element A k + a, which is exactly the last stage's
// input b G + r for b = a, r = k.
template <typename T, int N, int E, int DIR, int M>
__device__ __forceinline__ void stages_16_then_G(cplx<T> (&v)[M][E], int t, gptr<T> tw) {
  constexpr int NT = N / E, G = N / 256, A = 16 / G;
  static_assert(E == 16 && G == 4 && NT == 16 * G, "plan 16 x 16 x 4");
  stockham_stage<T, N, E, DIR, 16, 16, M>(v, t, tw);
  // G x G transpose across the lanes c + 16 q
#pragma unroll
  for (int m = 0; m < M; ++m) {
    cplx<T>(&x)[E] = v[m];
#pragma unroll
    for (int a = 0; a < A; ++a) {
      lane_swap<32>(x[4 * a + 0], x[4 * a + 2]);
      lane_swap<32>(x[4 * a + 1], x[4 * a + 3]);
      lane_swap<16>(x[4 * a + 0], x[4 * a + 1]);
      lane_swap<16>(x[4 * a + 2], x[4 * a + 3]);
    }
  }
  stockham_stage<T, N, E, DIR, 256, G, M>(v, t, tw + 15 * 16);
}

// Full transform of N points held by NT = N / E lanes.  v: lane t holds
// x[t + NT e]; buf: the group's LDS buffer (padded_len(N) complex slots, or as
// many real ones with SPLIT).  On exit the spectrum is in v, lane t holding entry
// t + NT e: butterfly b of the last stage (radix R, NB = E / R butterflies per
// lane) leaves entries t + NT (b + NB r), so the natural order needs no exchange.
// Without KEEP it is put into buf (in natural order; not with SPLIT).
// DIR = -1: forward (exp(-i...)), DIR = +1: inverse (unnormalised).
// M transforms side by side (a buffer each) share the twiddles and the waits.
template <typename T, int N, int E, int DIR, bool KEEP, bool SPLIT, int M>
__device__ __forceinline__ void fft_side_by_side(cplx<T> (&v)[M][E], T* const (&buf)[M], int t,
                                                 const cplx<T>* __restrict__ tw) {
  using PL = Plan<N, E>;
  constexpr int NT = N / E, R2 = PL::R2, R3 = PL::R3, R4 = PL::R4;
  static_assert(R2 > 1, "a transform of one stage");
  constexpr int RL = R4 > 1 ? R4 : (R3 > 1 ? R3 : R2);  // radix of the last stage
  // a fresh view of the twiddle table for every transform: stops the compiler
  // from keeping twiddles of one transform live until the next one
  asm volatile("" : "+s"(tw));
  const gptr<T> ptw = (gptr<T>)tw;
#pragma unroll
  for (int m = 0; m < M; ++m) dft<E, DIR>(v[m]);
  exchange<T, E, NT, SPLIT, M>(v, buf, [&](int i) { return LaneIdx{t * E + i, 0}; },
                               [&](int i) { return stage_in<N, E, R2>(i, t); });
  if constexpr (E == 16) {
    stages_16_then_G<T, N, E, DIR, M>(v, t, ptw);
  } else {
    stockham_stage<T, N, E, DIR, E, R2, M>(v, t, ptw + tw_offset(N, E, 0));
    if constexpr (R3 > 1) {
      exchange<T, E, NT, SPLIT, M>(v, buf, [&](int i) { return stage_out<N, E, E, R2>(i, t); },
                                   [&](int i) { return stage_in<N, E, R3>(i, t); });
      stockham_stage<T, N, E, DIR, E * R2, R3, M>(v, t, ptw + tw_offset(N, E, 1));
    }
    if constexpr (R4 > 1) {
      exchange<T, E, NT, SPLIT, M>(v, buf, [&](int i) { return stage_out<N, E, E * R2, R3>(i, t); },
                                   [&](int i) { return stage_in<N, E, R4>(i, t); });
      stockham_stage<T, N, E, DIR, E * R2 * R3, R4, M>(v, t, ptw + tw_offset(N, E, 2));
    }
  }
  constexpr int NB = E / RL;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    if constexpr (KEEP) {
      cplx<T> o[E];
#pragma unroll
      for (int i = 0; i < E; ++i) o[i / RL + NB * (i % RL)] = v[m][i];
#pragma unroll
      for (int i = 0; i < E; ++i) v[m][i] = o[i];
    } else {
      static_assert(!SPLIT, "a split buffer holds no whole spectrum");
      cplx<T>* cb = reinterpret_cast<cplx<T>*>(buf[m]);
#pragma unroll
      for (int i = 0; i < E; ++i) cb[pidx(LaneIdx{t, NT * (i / RL + NB * (i % RL))})] = v[m][i];
    }
  }
  if constexpr (!KEEP) xsync<NT>();
}

template <typename T, int N, int E, int DIR, bool KEEP = false, bool SPLIT = false>
__device__ __forceinline__ void fft(cplx<T> (&v)[E], T* buf, int t, const cplx<T>* __restrict__ tw) {
  T* const b[1] = {buf};
  fft_side_by_side<T, N, E, DIR, KEEP, SPLIT, 1>(reinterpret_cast<cplx<T>(&)[1][E]>(v), b, t, tw);
}

}  // namespace lm
