// bq_kernels.hpp -- gfx950 kernels of one adaptive-AB3 extended-Boussinesq
// time step (arXiv 1909.04153, Sec. 2-3).
//
// Data layout (per domain, all in the caller's workspace):
//   * state fields with two ghost layers (Sec. 3.3), row-major, row pitch a
//     multiple of 256 B and interior column 0 256-B aligned:
//       w[2] (double-buffered), P[3], Q[3] (rings: slot n % 3 = level n);
//   * interior-only fields: E, F, G rings (slot n % 3), local solutions
//     xhP, xhQ of the chunked line solves, cell still-water depth;
//   * corner still-water depth Dc with two mirrored ghost corner layers;
//   * per-chunk boundary/interface values of the line solves, [chunk][line];
//   * one FP64 DevState: time, Delta t history, weights, status.
//
// Per step (one launch each, over all domains of a batch):
//   k_dt      Delta t from the CFL maximum (Eq. 22) and Eq. (47), AB3 weights
//             (Eq. 42) and F*/G* weights (Eq. 43-46) in FP64, wavemaker
//             ghost values at t_{n+1};
//   k_rhs     LDS tile (64 x TY + halo 2): KP07 fluxes, bed source,
//             dispersion, friction, F*/G* of the weighted P/Q history, AB3
//             update of w and of U*, V* (as increments); then the chunk-local
//             tridiagonal solves of Eq. (19)-(20) for the P, Q increments;
//   k_reduced the chunk-interface recurrences that couple the chunk-local
//             solutions of every line into the exact line solution;
//   k_final   P, Q = local solution + the chunk systems' response to the
//             neighbour-chunk values, sponge, ghost cells of the new state,
//             CFL maximum of the new state.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bq_fp64.hpp"
#include "bq_layout.hpp"

namespace bqk {

enum { WALL = 0, SINE = 1, SPONGE = 2, IRREGULAR = 3, TIMESERIES = 4 };
// west sides whose ghost cells are prescribed (wavemakers, time series)
__host__ __device__ inline bool west_driven(int bc) { return bc == SINE || bc == IRREGULAR || bc == TIMESERIES; }
enum { ST_OK = 0, ST_ENONFINITE = -4, ST_EDTMIN = -5, ST_EDONE = -7 };

constexpr int NDIAG = 256;  // blocks of the diagnostic sums

struct alignas(64) DevState {
  // committed state
  double t;                 // time of the current state
  double dt1, dt2, dt3;     // Delta t of the last three steps (dt1 most recent)
  long long n;              // steps taken
  int status;
  int pending;              // a step was scheduled by k_dt and is not yet committed
  // the step being taken
  double dt;
  double alpha[3];
  double beta[3];
  double gamma[4];          // corrector weights of X^{n+1*}, X^n, X^{n-1}, X^{n-2}
  double t_next;
  double gw[2], gP[2];      // wavemaker ghost values (cells -1, -2) at t_next
  double smax_used;         // CFL maximum the step's Delta t was taken from
  int halt;                 // 1 = kernels of this step leave the domain untouched
  int slot;                 // n % 3 of the step being taken
  unsigned long long smax_bits;  // running max of the speeds of the new state
  double mass, energy;      // diagnostics (filled on demand)
  double pad[2];
};

template <typename T>
struct DomDev {
  int nx, ny;
  int pitch, xoff;          // ghosted fields: (i, j) at (j + 2) * pitch + xoff + i
  int ipitch;               // interior fields: (i, j) at j * ipitch + i
  int cpitch;               // corners: (ic, jc) at (jc + 2) * cpitch + ic + 2
  int cx, cy;               // chunks per x-line / y-line
  int mx, my;               // chunk lengths
  int tiles_x, tiles_y;
  int bc[4];
  int fstar_order, fixed_dt, n_waves, any_sponge;
  int ts_n;                 // time-series samples (BC TIMESERIES on the west side)
  int runup;                // 1 = keep the run-up record wmax
  int corrector;            // 1 = AB3 predictor + Adams-Moulton corrector
  T dx, dy, g, B, Bc, gn2, cf, theta, eps;
  T runup_delta;
  // reciprocals of the grid spacing combinations used by the stencils
  T idx, idy, i2dx, i2dy, idx2, idy2, i4dxdy, i2dx3, i2dy3, i2dxdy2, i2dx2dy;
  // constants of the Eq. (21) coefficients per direction: 1/(2h), (B+1/3)/h^2, 1/(6h)
  T tcx[3], tcy[3];
  T sponge_w[4];
  T sponge_sigma;
  double dx_d, dy_d, g_d, cfl, ema_alpha, dt_init, dt_max, dt_min, wave_ramp, t_end, ts_dt;
  T* w[3];                  // surface double buffer; w[2] holds the predicted surface
                            // of a predictor-corrector step
  T* P[3];
  T* Q[3];
  T* E[3];
  T* F[3];
  T* G[3];
  T* Dc;
  T* Dbar;
  T* xhP;
  T* xhQ;
  T* chx;                   // [2][cx][ny]: local solution at chunk first / last
  T* chy;                   // [2][cy][nx]
  T* rsx;                   // [6][cx][ny]: static interface-recurrence coefficients
  T* rsy;                   // [6][cy][nx]
  T* ifx;                   // [2][cx][ny]: neighbour values left / right of a chunk
  T* ify;                   // [2][cy][nx]
  double* smax_tile;        // per tile: CFL maximum of the new state (written by the finalize kernel)
  double* diag_part;        // [2][NDIAG]: per-block mass / energy partial sums
  double* wave;             // [4][n_waves]: amplitude, omega, phase, wave number;
                            // time series: [2][ts_n]: eta, P samples
  T* wmax;                  // run-up record (interior layout), if kept
  double* io;               // nx * ny doubles of staging for host transfers
  DevState* st;
};

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

// Field pointers live in the per-domain descriptor in device memory, so the
// compiler cannot tell they address global memory and would emit flat
// accesses (which also wait on the LDS counter); name the address space.
template <typename T>
using gp = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gp<T> gbl(T* p) {
  return (gp<T>)p;
}

// A pointer read from device memory that is the same in every lane: pin it
// to scalar registers, so that loads through it take the scalar-base form.
template <typename P>
__device__ __forceinline__ P* uni(P* p) {
  const unsigned long long v = (unsigned long long)p;
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
  return (P*)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uni(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// materialise a value in a register at this point (the compiler may not sink
// its computation to a later use)
template <typename T>
__device__ __forceinline__ void pin(T& v) {
  __asm__ volatile("" : "+v"(v));
}

// Element `off` of a field whose base address is the same for the whole
// block: a scalar base plus a 32-bit per-lane byte offset (below 4 GiB: the
// tile kernels have a form for larger fields, and the line solves' arrays are
// below by the limit on a domain's padded fields).
template <typename T>
__device__ __forceinline__ T ldu(const T* base, unsigned off) {
  const gp<const char> b = (gp<const char>)(const char*)base;
  return *(gp<const T>)(b + (unsigned)(off * (unsigned)sizeof(T)));
}
template <typename T>
__device__ __forceinline__ void stu(T* base, unsigned off, T v) {
  const gp<char> b = (gp<char>)(char*)base;
  *(gp<T>)(b + (unsigned)(off * (unsigned)sizeof(T))) = v;
}
// N consecutive elements of a field at a block-uniform base, as one vector
// access (off is a multiple of N and the bases are 256-byte aligned)
template <typename T, int N>
struct alignas(sizeof(T) * N) Vec {
  T v[N];
};
template <typename T, int N>
struct VecRaw;
template <>
struct VecRaw<float, 1> {
  typedef float t;
};
template <>
struct VecRaw<float, 2> {
  typedef float t __attribute__((ext_vector_type(2)));
};
template <>
struct VecRaw<float, 4> {
  typedef float t __attribute__((ext_vector_type(4)));
};
template <>
struct VecRaw<double, 1> {
  typedef double t;
};
template <>
struct VecRaw<double, 2> {
  typedef double t __attribute__((ext_vector_type(2)));
};
template <int N, typename T>
__device__ __forceinline__ Vec<T, N> ldv(const T* base, unsigned off) {
  using R = typename VecRaw<T, N>::t;
  const gp<const char> b = (gp<const char>)(const char*)base;
  const R x = *(gp<const R>)(b + (unsigned)(off * (unsigned)sizeof(T)));
  Vec<T, N> r;
  __builtin_memcpy(&r, &x, sizeof r);
  return r;
}
template <int N, typename T>
__device__ __forceinline__ void stv(T* base, unsigned off, const Vec<T, N>& v) {
  using R = typename VecRaw<T, N>::t;
  R x;
  __builtin_memcpy(&x, &v, sizeof x);
  const gp<char> b = (gp<char>)(char*)base;
  *(gp<R>)(b + (unsigned)(off * (unsigned)sizeof(T))) = x;
}

// The same with the non-temporal hint, for fields that a step reads or
// writes once and that are not re-read before much other traffic (the
// history rings, the local solutions, the new state): their lines are
// evicted first, which keeps the halo rows that neighbouring tiles re-read
// in L2.  Measured on the 64-domain batch: 0.547 -> 0.517 ms per step.
template <int N, typename T>
__device__ __forceinline__ Vec<T, N> ldv_nt(const T* base, unsigned off) {
  using R = typename VecRaw<T, N>::t;
  const gp<const char> b = (gp<const char>)(const char*)base;
  const R x = __builtin_nontemporal_load((gp<const R>)(b + (unsigned)(off * (unsigned)sizeof(T))));
  Vec<T, N> r;
  __builtin_memcpy(&r, &x, sizeof r);
  return r;
}
template <int N, typename T>
__device__ __forceinline__ void stv_nt(T* base, unsigned off, const Vec<T, N>& v) {
  using R = typename VecRaw<T, N>::t;
  R x;
  __builtin_memcpy(&x, &v, sizeof x);
  const gp<char> b = (gp<char>)(char*)base;
  __builtin_nontemporal_store(x, (gp<R>)(b + (unsigned)(off * (unsigned)sizeof(T))));
}

// Square root, reciprocal and x^(-1/3) for any argument.  FP64: the library's
// correctly rounded root and division, and an inverse cube root good to 1.43 x
// 2^-53; FP32: the hardware's transcendental instructions (about 1 ulp), whose
// error is far below the FP32 path's own rounding of the state.
template <typename T> __device__ __forceinline__ T fsqrt(T x);
template <typename T> __device__ __forceinline__ T frcp(T x);
template <typename T> __device__ __forceinline__ T frcbrt(T x);   // x^(-1/3), x > 0
template <> __device__ __forceinline__ double fsqrt<double>(double x) { return sqrt(x); }
template <> __device__ __forceinline__ double frcp<double>(double x) { return 1.0 / x; }
// FP64: from the FP32 value (4e-6); outside the FP32 range by the library's
// cube root
template <> __device__ __forceinline__ double frcbrt<double>(double x) {
  if (!(x > 1e-30 && x < 1e30)) return 1.0 / cbrt(x);
  return rcbrt_from(x, (double)__builtin_amdgcn_exp2f(-0.33333333f * __builtin_amdgcn_logf((float)x)));
}
template <> __device__ __forceinline__ float fsqrt<float>(float x) { return __builtin_amdgcn_sqrtf(x); }
template <> __device__ __forceinline__ float frcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
// Reciprocal, division by a number of known reciprocal, square root and (FP64)
// inverse square root, of a positive number in ordinary range
__device__ __forceinline__ float rcp_n(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float div_n(float t, float, float id) { return t * id; }
__device__ __forceinline__ float sqrt_n(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double rcp_n(double x) { return rcp_from(x, __builtin_amdgcn_rcp(x)); }
__device__ __forceinline__ double div_n(double t, double d, double id) { return div_from(t, d, id); }
__device__ __forceinline__ double sqrt_n(double x) { return sqrt_from(x, __builtin_amdgcn_rsq(x)); }
__device__ __forceinline__ double rsq_n(double x) { return rsq_from(x, __builtin_amdgcn_rsq(x)); }
// The hardware log takes a subnormal input as 0 (giving +inf here, and a
// NaN once multiplied by the zero velocity of a film that thin): depths are
// raised to the smallest normal value first, which leaves h^(-1/3) finite
// (< 5e12) for every h > 0.
template <> __device__ __forceinline__ float frcbrt<float>(float x) {
  return __builtin_amdgcn_exp2f(-0.33333333f * __builtin_amdgcn_logf(__builtin_fmaxf(x, 1.17549435e-38f)));
}

// generalised minmod of three values: the one nearest zero when all three
// share a sign, else zero
template <typename T>
__device__ __forceinline__ T gmm(T a, T b, T c) {
  const T lo = fmin(a, fmin(b, c));
  const T hi = fmax(a, fmax(b, c));
  return lo > T(0) ? lo : (hi < T(0) ? hi : T(0));
}
// FP32: med3(a, c, 0) is minmod(a, c), and minmod(minmod(a, c), b) is the
// same value as above, in two median-of-three instructions
template <>
__device__ __forceinline__ float gmm<float>(float a, float b, float c) {
  return __builtin_amdgcn_fmed3f(__builtin_amdgcn_fmed3f(a, c, 0.0f), b, 0.0f);
}

// half the limited slope (times the cell size) of q at a cell from its two
// neighbours, ht = theta / 2: minmod(ht (q0 - qm), (qp - qm) / 4, ht (qp - q0));
// theta = 0 (LIM false; the caller takes that choice once per tile) selects
// the unlimited central slope.  Halving is exact, so the face values
// q0 -/+ hslope equal q0 -/+ slope / 2.
template <bool LIM, typename T>
__device__ __forceinline__ T hslope(T qm, T q0, T qp, T ht) {
  const T c = T(0.25) * (qp - qm);
  return LIM ? gmm(ht * (q0 - qm), c, ht * (qp - q0)) : c;
}

// Velocity factor of the KP07 desingularisation, u = q * vfac(h):
//   sqrt(2) h / sqrt(h^4 + max(h^4, eps)),
// which is exactly 1/h when h^4 >= eps (taken directly there).
template <typename T>
__device__ __forceinline__ T vfac(T h, T eps) {
  const T h2 = h * h;
  const T h4 = h2 * h2;
  if (h4 >= eps) return rcp_n(h);
  return T(1.4142135623730951) * h * frcp(fsqrt(h4 + eps));
}

template <typename T>
__device__ __forceinline__ T desing(T q, T h, T eps) {
  return q * vfac(h, eps);
}

// cell-average still-water depth from its four corners
template <typename T>
__device__ __forceinline__ T dbar4(T a, T b, T c, T d) {
  return T(0.25) * (a + b + c + d);
}

// max(D, 0) and min(D, 0) of a still-water depth (always finite).  FP32 takes
// one median-of-three: a plain fmax of a value read from memory costs a
// second instruction that quiets a possible signalling NaN first.
template <typename T>
__device__ __forceinline__ T dpos(T D) {
  return fmax(D, T(0));
}
template <>
__device__ __forceinline__ float dpos<float>(float D) {
  return __builtin_amdgcn_fmed3f(D, 0.0f, 3.402823466e38f);
}
template <typename T>
__device__ __forceinline__ T dneg(T D) {
  return fmin(D, T(0));
}
template <>
__device__ __forceinline__ float dneg<float>(float D) {
  return __builtin_amdgcn_fmed3f(D, 0.0f, -3.402823466e38f);
}

// max(a, b) of finite values; FP32 again without the quieting instruction
template <typename T>
__device__ __forceinline__ T dmax_nq(T a, T b) {
  return fmax(a, b);
}
template <>
__device__ __forceinline__ float dmax_nq<float>(float a, float b) {
  return __builtin_amdgcn_fmed3f(a, b, 3.402823466e38f);
}

// KP07 positivity correction of the surface w0 -/+ slope at a cell's low/high
// faces; Dlo/Dhi are the still-water depths there (bed = -D)
template <typename T>
__device__ __forceinline__ void positive(T w0, T Dlo, T Dhi, T& wlo, T& whi) {
  if (whi + Dhi < T(0)) {
    whi = -Dhi;
    wlo = T(2) * w0 + Dhi;
  } else if (wlo + Dlo < T(0)) {
    wlo = -Dlo;
    whi = T(2) * w0 + Dlo;
  }
}

template <typename T>
__device__ __forceinline__ T fma_(T a, T b, T c);
template <>
__device__ __forceinline__ float fma_<float>(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}
template <>
__device__ __forceinline__ double fma_<double>(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}

// One side of a face.  The hydrostatic pressure g h^2 / 2 is carried as its
// departure from the still-water value g D+^2 / 2 at the face, D+ = max(D, 0):
//   pp = g (h - D+)(h + D+) / 2,
//   h - D+ = w (wet face below the still-water line), -D (dry there), h (land).
// The still-water parts of the flux differences and of the well-balanced bed
// source cancel exactly except in cells whose two faces straddle the
// still-water line (see add_shore); keeping them would leave FP32 with a
// difference of large numbers in deep water.
//
// The face pass below takes a straight form where a wave's sides are all
// deep and this general one elsewhere, and a cell's result must not depend on
// which of them its wave took (rows of one wave front would differ, and the
// quadratic F* extrapolation amplifies that).  So both forms write their fused
// multiply-adds out, with contraction off, and compute a deep side (h^4 >=
// eps) by the same expressions.
template <typename T>
struct Side {
  T w, h, un, ut, qn, qt, dev, pa, pb, c;      // pp = pa * pb, c = sqrt(g h)
};

// velocities, recomputed discharges h u and wave speed of a side, DEEP: known
// to have h^4 >= eps.  u = sqrt(2) h q / sqrt(h^4 + max(h^4, eps)).
__device__ __forceinline__ void side_speeds(Side<float>& s, float qn, float qt, float eps, float g) {
#pragma clang fp contract(off)
  const float h2 = s.h * s.h;
  const float h4 = h2 * h2;
  if (h4 >= eps) {
    // u = q / h, and h u is q itself (exact identities)
    const float vf = rcp_n(s.h);
    s.un = qn * vf;
    s.ut = qt * vf;
    s.qn = qn;
    s.qt = qt;
  } else {
    const float r = __builtin_amdgcn_rsqf(h4 + fmax(h4, eps));
    const float sh = 1.4142135623730951f * s.h;
    s.un = sh * qn * r;
    s.ut = sh * qt * r;
    s.qn = s.h * s.un;
    s.qt = s.h * s.ut;
  }
  s.c = sqrt_n(g * s.h);
}
// FP64 keeps the one expression everywhere, u = q h / sqrt(z) with one root for
// both velocities: four roundings after h^4 where the definition's own order,
// sqrt(2) h q / sqrt(h^4 + max(h^4, eps)), has five
template <bool DEEP = false>
__device__ __forceinline__ void side_speeds(Side<double>& s, double qn, double qt, double eps, double g) {
#pragma clang fp contract(off)
  const double h2 = s.h * s.h;
  const double h4 = h2 * h2;
  const double vf = s.h * rsq_n(DEEP ? h4 : desing_sq(h4, eps));
  s.un = qn * vf;
  s.ut = qt * vf;
  s.qn = s.h * s.un;
  s.qt = s.h * s.ut;
  const double gh = g * s.h, c = sqrt_n(gh);
  s.c = DEEP || gh > 0.0 ? c : 0.0;
}

template <typename T>
__device__ __forceinline__ Side<T> make_side(T w, T qn, T qt, T Dface, T eps, T g) {
#pragma clang fp contract(off)
  Side<T> s;
  s.w = w;
  s.h = fmax(w + Dface, T(0));
  side_speeds(s, qn, qt, eps, g);
  const T Dp = dpos(Dface);
  // (h > 0 exactly when w > -D, so below the still-water line dev is max(w, -D))
  s.dev = Dface > T(0) ? dmax_nq(w, -Dface) : s.h;
  s.pa = T(0.5) * g * s.dev;
  s.pb = s.h + Dp;
  return s;
}

// central-upwind flux normal to a face, components (mass, normal momentum,
// tangential momentum); the normal momentum flux excludes g D^2 / 2.  DEEP:
// both sides are deep, so at least one of the speeds is not zero.
template <bool DEEP, typename T>
__device__ __forceinline__ void cu_flux(const Side<T>& L, const Side<T>& R, T g, T Dface, T& f0, T& fn, T& ft) {
#pragma clang fp contract(off)
  const T ap = fmax(fmax(L.un + L.c, R.un + R.c), T(0));
  const T am = fmin(fmin(L.un - L.c, R.un - R.c), T(0));
  const T den = ap - am;
  if (!DEEP && den == T(0)) {
    // both sides dry and at rest: the full flux is zero
    const T Dp = dpos(Dface);
    f0 = ft = T(0);
    fn = -T(0.5) * g * Dp * Dp;
    return;
  }
  const T inv = rcp_n(den);
  const T dis = ap * am * inv;
  const T pL = fma_(L.pa, L.pb, L.qn * L.un);
  const T pR = fma_(R.pa, R.pb, R.qn * R.un);
  const T aq = ap * L.qn, mq = am * R.qn;
  f0 = fma_(fma_(ap, L.qn, -mq), inv, dis * (R.w - L.w));
  fn = fma_(fma_(ap, pL, -(am * pR)), inv, dis * (R.qn - L.qn));
  ft = fma_(fma_(aq, L.ut, -(mq * R.ut)), inv, dis * (R.qt - L.qt));
}

// still-water remainder of (bed source - pressure flux difference) in a cell
// whose low/high faces have still-water depths Dl, Dh: zero unless exactly
// one of them is below the still-water line
template <typename T>
__device__ __forceinline__ void add_shore(T& bed, T Dl, T Dh, T g) {
  // a branch, not a select: shore faces are rare, so most waves skip it
  if (__builtin_expect((Dl > T(0)) != (Dh > T(0)), 0)) {
    const T pl = dpos(Dl), ph = dpos(Dh);
    bed += T(0.5) * g * ((Dh - Dl) * (ph + pl) - (ph * ph - pl * pl));
  }
}

// Faces of N consecutive cells of a line (stride st in the tile; w, qn, qt at
// the second cell before the first): cells -1 .. N are reconstructed once,
// the N + 1 faces between them taken once, and each cell gets its flux
// differences (low face less high) plus the well-balanced bed source
// -g h b_x with h the mean of its own face depths (with the still-water parts
// of the pressure fluxes taken out only the face-depth departures remain),
// all times dx: e (mass), n (normal momentum), t (tangential).  Df[k] is the
// still-water depth of face k - 1.
//
// What bounds it is issue, and in small domains (one wave per SIMD) latency:
// dry and thin sides, the positivity correction and shore faces each take a
// branch, about eleven a cell, between short dependent runs.  In FP64, whose
// roots and divisions are those runs, a wave whose sides are all deep and
// whose faces all lie below the still-water line takes a straight form
// without any of them: x- and y-faces of a 200 x 20 domain 10.6 -> 6.6
// thousand cycles; the stencil kernel as a whole, with roots and reciprocals
// at less than the correctly rounded cost, 13.0 -> 11.3 us there, 19.9 -> 18.0
// on 1024 x 256 and 26.9 -> 22.9 on 601 x 601.  (The fields' padding past a
// domain's end continues its depth, so the tiles there take it too.)  FP32
// does without: the test and the second form cost its mixed tiles (a beach's)
// 5 to 10 % of the kernel, more than they give the deep ones.
template <typename T, int N>
__device__ __forceinline__ void face_pass(const T* w, const T* qn, const T* qt, int st, const T (&Df)[N + 3], T ht,
                                          T eps, T g, T (&e)[N], T (&n)[N], T (&t)[N]) {
#pragma clang fp contract(off)
  // cell k - 1 at its low (l) and high (h) faces; limited (theta > 0) or
  // central slopes: one uniform branch per tile
  T wl[N + 2], wh[N + 2], pl[N + 2], ph[N + 2], ql[N + 2], qh[N + 2];
  auto recon = [&](auto lim) {
    constexpr bool LIM = decltype(lim)::value;
    auto ends = [&](const T* q, T& lo, T& hi) {
      const T s = hslope<LIM>(q[0], q[st], q[2 * st], ht);
      lo = q[st] - s;
      hi = q[st] + s;
    };
#pragma unroll
    for (int k = 0; k < N + 2; ++k) {
      ends(w + k * st, wl[k], wh[k]);
      if (sizeof(T) == 4) positive(w[(k + 1) * st], Df[k], Df[k + 1], wl[k], wh[k]);
      ends(qn + k * st, pl[k], ph[k]);
      ends(qt + k * st, ql[k], qh[k]);
    }
  };
  if (ht > T(0)) recon(std::true_type{});
  else recon(std::false_type{});
  T f0w = T(0), fnw = T(0), ftw = T(0), dvw = T(0);    // low face of the cell being closed
  if constexpr (sizeof(T) == 8) {
    T dmin = Df[0], hmin = wl[0] + Df[0];
#pragma unroll
    for (int k = 0; k < N + 2; ++k) {
      dmin = fmin(dmin, Df[k + 1]);
      hmin = fmin(hmin, fmin(wl[k] + Df[k], wh[k] + Df[k + 1]));
    }
    const T h2 = hmin * hmin;
    if (__all(dmin > T(0) && hmin > T(0) && h2 * h2 >= eps)) {
#pragma unroll
      for (int m = 0; m <= N; ++m) {
        const T D = Df[m + 1];
        auto side = [&](T ws, T a, T b) {
#pragma clang fp contract(off)
          Side<T> s;
          s.w = s.dev = ws;
          s.h = ws + D;
          side_speeds<true>(s, a, b, eps, g);
          s.pa = T(0.5) * g * ws;
          s.pb = s.h + D;
          return s;
        };
        const Side<T> L = side(wh[m], ph[m], qh[m]), R = side(wl[m + 1], pl[m + 1], ql[m + 1]);
        T f0, fn, ft;
        cu_flux<true>(L, R, g, D, f0, fn, ft);
        if (m > 0) {
          const T bed = g * (D - Df[m]) * (T(0.5) * (wh[m] + wl[m]));
          e[m - 1] = f0w - f0;
          n[m - 1] = bed - (fn - fnw);
          t[m - 1] = ftw - ft;
        }
        f0w = f0;
        fnw = fn;
        ftw = ft;
      }
      return;
    }
#pragma unroll
    for (int k = 0; k < N + 2; ++k) positive(w[(k + 1) * st], Df[k], Df[k + 1], wl[k], wh[k]);
  }
#pragma unroll
  for (int m = 0; m <= N; ++m) {
    const T D = Df[m + 1];
    const Side<T> L = make_side(wh[m], ph[m], qh[m], D, eps, g);
    const Side<T> R = make_side(wl[m + 1], pl[m + 1], ql[m + 1], D, eps, g);
    T f0, fn, ft;
    cu_flux<false>(L, R, g, D, f0, fn, ft);
    if (m > 0) {
      T bed = g * (D - Df[m]) * (T(0.5) * (L.dev + dvw));
      add_shore(bed, Df[m], D, g);
      e[m - 1] = f0w - f0;
      n[m - 1] = bed - (fn - fnw);
      t[m - 1] = ftw - ft;
    }
    f0w = f0;
    fnw = fn;
    ftw = ft;
    dvw = R.dev;
  }
}

// Coefficients of Eq. (21) at a cell from the still-water depths of the cell
// and its two neighbours along the line; tc = (1/(2h), (B+1/3)/h^2, 1/(6h)).
template <typename T>
__device__ __forceinline__ void tri_coef(T dm, T d0, T dp, const T* tc, T& a, T& b, T& c) {
  const T dd = (dp - dm) * tc[0];
  const T k = tc[1] * d0 * d0;
  const T s = d0 * dd * tc[2];
  a = s - k;
  b = T(1) + T(2) * k;
  c = -s - k;
}

// Chunk-local tridiagonal solve (zero coupling to the neighbouring chunks)
// of the m (<= M) unknowns of one chunk.  Dl[k * ds], k = 0..m+1, are the
// cell-average still-water depths of the chunk's cells with one neighbour on
// each side (d = max(D, 0)); tc are the Eq. (21) constants of the direction.
// fold_lo / fold_hi fold the odd mirror of a wall into the first / last
// diagonal.  rhs (stride rs) is overwritten with the solution; the forward
// sweep leaves y_k / u_k in rhs and keeps c_k / u_k in registers, so the
// backward sweep is one multiply-add per row (the loops are unrolled over M).
template <typename T, int M, bool FULL>
__device__ __forceinline__ void chunk_solve_db_(const T* Dl, int ds, int m, const T* tc, bool fold_lo, bool fold_hi,
                                                T* rhs, int rs) {
  if (FULL) m = M;
  T cu[M];                                     // c_k / u_k; rhs holds y_k / u_k
  T y_prev = T(0), iu_prev = T(1), c_prev = T(0);
#pragma unroll
  for (int k = 0; k < M; ++k) {
    if (FULL || k < m) {
      T a, b, c;
      tri_coef(dpos(Dl[k * ds]), dpos(Dl[(k + 1) * ds]), dpos(Dl[(k + 2) * ds]), tc, a, b, c);
      if (k == 0 && fold_lo) b -= a;
      if (k == m - 1 && fold_hi) b -= c;
      const T r = rhs[k * rs];
      T u, y;
      if (k == 0) {
        u = b;
        y = r;
      } else {
        const T l = a * iu_prev;
        u = b - l * c_prev;
        y = r - l * y_prev;
      }
      const T iu = frcp(u);
      cu[k] = c * iu;
      rhs[k * rs] = y * iu;
      y_prev = y;
      iu_prev = iu;
      c_prev = c;
    }
  }
  T x_next = T(0);
#pragma unroll
  for (int k = M - 1; k >= 0; --k) {
    if (FULL || k < m) {
      const T y = rhs[k * rs];
      const T x = (k == m - 1) ? y : y - cu[k] * x_next;
      rhs[k * rs] = x;
      x_next = x;
    }
  }
}
// full chunks (the common case) take a branch-free unrolled path, so the
// LDS reads can be issued ahead of the dependent arithmetic
template <typename T, int M>
__device__ __forceinline__ void chunk_solve_db(const T* Dl, int ds, int m, const T* tc, bool fold_lo, bool fold_hi,
                                               T* rhs, int rs) {
  if (m == M) chunk_solve_db_<T, M, true>(Dl, ds, m, tc, fold_lo, fold_hi, rhs, rs);
  else chunk_solve_db_<T, M, false>(Dl, ds, m, tc, fold_lo, fold_hi, rhs, rs);
}

// Chunk solve by a group of P lanes (P = 2 or 4 consecutive lanes; lane
// part = lane % P takes the part-th of P consecutive parts of the chunk's m
// rows, of (m + P - 1 - part) / P rows each, so that only trailing parts
// are empty).  Each lane eliminates its part with zero coupling to the
// other parts, for the right-hand side and for its two coupling columns:
// its last row couples to the next part's first unknown through c (response
// v), its first row to the previous part's last unknown through a (response
// w).  The group exchanges the parts' end values by lane shuffles, every
// lane solves the small system of the interface unknowns (L_i = x at part
// i's last row, R_i = x at part i+1's first row), and each lane corrects its
// part: x = x-hat - R_part v - L_{part-1} w.  This is the SPIKE construction
// of the line coupling applied inside the chunk: each serial sweep is 1/P as
// long.  Dl, ds, tc, fold_lo, fold_hi as in chunk_solve_db; rhs(k) is the
// right-hand side of chunk row k.  On return x[0 .. mh-1] holds the solution
// of chunk rows k0 .. k0+mh-1 and xlast that of row k0+mh-1.  Every lane of
// a group must make the call.
template <typename T, int H, int P, bool FULL, bool POS, typename RHS>
__device__ __forceinline__ void group_solve_(const T* Dl, int ds, int m, const T* tc, bool fold_lo, bool fold_hi,
                                             int part, RHS rhs, T (&x)[H], int& k0, int& mh, T& xlast) {
  static_assert(P == 2 || P == 4, "groups of two or four lanes");
  constexpr int N = 2 * (P - 1);              // interface unknowns L_0, R_0, L_1, R_1, ...
  auto size = [&](int q) { return FULL ? H : (m + P - 1 - q) / P; };
  k0 = 0;
#pragma unroll
  for (int q = 0; q < P - 1; ++q)
    if (q < part) k0 += size(q);
  mh = size(part);
  const int np = min(P, m);                   // parts that hold rows
  // the chunk's first row is this part's first when part == 0, its last row
  // this part's last when part == np - 1
  const bool lo = fold_lo && part == 0, hi = fold_hi && part == np - 1;
  T cu[H], wv[H], vv[H];                      // c_j / u_j; responses to the left / right couplings
  T y_prev = T(0), s_prev = T(0), iu_prev = T(1), c_prev = T(0), vy = T(0);
#pragma unroll
  for (int j = 0; j < H; ++j) {
    if (FULL || j < mh) {
      const int k = k0 + j;
      T a, b, c;
      if (POS) tri_coef(Dl[k * ds], Dl[(k + 1) * ds], Dl[(k + 2) * ds], tc, a, b, c);
      else tri_coef(dpos(Dl[k * ds]), dpos(Dl[(k + 1) * ds]), dpos(Dl[(k + 2) * ds]), tc, a, b, c);
      if (j == 0 && lo) b -= a;
      if (j == mh - 1 && hi) b -= c;
      const T r = rhs(k);
      T u, y, sw;
      if (j == 0) {
        u = b;
        y = r;
        sw = part > 0 ? a : T(0);
      } else {
        const T l = a * iu_prev;
        u = b - l * c_prev;
        y = r - l * y_prev;
        sw = -l * s_prev;
      }
      const T iu = rcp_n(u);
      cu[j] = c * iu;
      x[j] = y * iu;
      wv[j] = sw * iu;
      // the right coupling enters in the last row only (no elimination
      // reaches it before)
      if (j == mh - 1) vy = (part < np - 1 ? c : T(0)) * iu;
      y_prev = y;
      s_prev = sw;
      iu_prev = iu;
      c_prev = c;
    }
  }
  // backward sweeps; end values of the part (first and last row)
  T xn = T(0), wn = T(0), vn = T(0);
  T xL = T(0), wL = T(0), vL = T(0);
#pragma unroll
  for (int j = H - 1; j >= 0; --j) {
    if (FULL || j < mh) {
      const bool last = j == mh - 1;
      const T xv = last ? x[j] : x[j] - cu[j] * xn;
      const T wvv = last ? wv[j] : wv[j] - cu[j] * wn;
      const T vvv = last ? vy : -cu[j] * vn;
      x[j] = xv;
      wv[j] = wvv;
      vv[j] = vvv;
      xn = xv;
      wn = wvv;
      vn = vvv;
      if (last) {
        xL = xv;
        wL = wvv;
        vL = vvv;
      }
    }
  }
  const bool any = FULL || mh > 0;
  const T xF = any ? x[0] : T(0), wF = any ? wv[0] : T(0), vF = any ? vv[0] : T(0);
  // every part's end values, from the lanes of the group
  const int base = (int)(threadIdx.x & 63) & ~(P - 1);
  T gxL[P], gwL[P], gvL[P], gxF[P], gwF[P], gvF[P];
#pragma unroll
  for (int q = 0; q < P; ++q) {
    gxL[q] = __shfl(xL, base + q, 64);
    gwL[q] = __shfl(wL, base + q, 64);
    gvL[q] = __shfl(vL, base + q, 64);
    gxF[q] = __shfl(xF, base + q, 64);
    gwF[q] = __shfl(wF, base + q, 64);
    gvF[q] = __shfl(vF, base + q, 64);
  }
  // interface system M z = r, z = (L_0, R_0, L_1, R_1, ...); an interface
  // past the last part with rows has L = R = 0
  T M[N][N], rv[N];
#pragma unroll
  for (int e = 0; e < N; ++e) {
    rv[e] = T(0);
#pragma unroll
    for (int f = 0; f < N; ++f) M[e][f] = e == f ? T(1) : T(0);
  }
#pragma unroll
  for (int i = 0; i < P - 1; ++i) {
    if (i < np - 1) {
      // L_i + v_i(last) R_i + w_i(last) L_{i-1} = x-hat_i(last)
      M[2 * i][2 * i + 1] = gvL[i];
      if (i > 0) M[2 * i][2 * i - 2] = gwL[i];
      rv[2 * i] = gxL[i];
      // R_i + w_{i+1}(first) L_i + v_{i+1}(first) R_{i+1} = x-hat_{i+1}(first)
      M[2 * i + 1][2 * i] = gwF[i + 1];
      if (i + 1 < P - 1) M[2 * i + 1][2 * i + 3] = gvF[i + 1];
      rv[2 * i + 1] = gxF[i + 1];
    }
  }
  // Gaussian elimination (the matrix is the identity plus coupling
  // responses below one in size: no pivoting)
  T id[N];
#pragma unroll
  for (int e = 0; e < N; ++e) {
    id[e] = rcp_n(M[e][e]);
#pragma unroll
    for (int f = e + 1; f < N; ++f) {
      const T l = M[f][e] * id[e];
#pragma unroll
      for (int g = e; g < N; ++g) M[f][g] -= l * M[e][g];
      rv[f] -= l * rv[e];
    }
  }
  T z[N];
#pragma unroll
  for (int e = N - 1; e >= 0; --e) {
    T t = rv[e];
#pragma unroll
    for (int f = e + 1; f < N; ++f) t -= M[e][f] * z[f];
    z[e] = div_n(t, M[e][e], id[e]);
  }
  T Rp = T(0), Lm = T(0);                      // R_part, L_{part-1}
#pragma unroll
  for (int q = 0; q < P; ++q)
    if (q == part) {
      if (q < P - 1) Rp = z[2 * q + 1];
      if (q > 0) Lm = z[2 * q - 2];
    }
  xlast = T(0);
#pragma unroll
  for (int j = 0; j < H; ++j) {
    if (FULL || j < mh) {
      x[j] -= Rp * vv[j] + Lm * wv[j];
      if (j == mh - 1) xlast = x[j];
    }
  }
}
// full chunks (the common case) take the branch-free unrolled path.  POS:
// the depths Dl are already max(D, 0).
template <typename T, int H, int P, bool POS = false, typename RHS>
__device__ __forceinline__ void group_solve(const T* Dl, int ds, int m, const T* tc, bool fold_lo, bool fold_hi,
                                            int part, RHS rhs, T (&x)[H], int& k0, int& mh, T& xlast) {
  if (m == P * H) group_solve_<T, H, P, true, POS>(Dl, ds, m, tc, fold_lo, fold_hi, part, rhs, x, k0, mh, xlast);
  else group_solve_<T, H, P, false, POS>(Dl, ds, m, tc, fold_lo, fold_hi, part, rhs, x, k0, mh, xlast);
}

// The chunk system's response to its two neighbour-chunk values alone: the
// right-hand side is r0 in the chunk's first row and r1 in its last, zero
// elsewhere, solved by the same lane groups and parts as group_solve.  Every
// vector a part needs is then a combination of two: f and g, the part's
// responses to a unit value in its first and in its last row.  The part's
// own right-hand side is rf e_first + rl e_last (rf = r0 in the first part,
// rl = r1 in the last), its coupling columns are a e_first and c e_last, so
// x-hat = rf f + rl g, w = a f, v = c g, and the corrected solution is
// (rf - a L_{part-1}) f + (rl - c R_part) g: one forward and two backward
// sweeps per row instead of three of each.
template <typename T, int H, int P, bool FULL>
__device__ __forceinline__ void group_response_(const T* Dl, int ds, int m, const T* tc, bool fold_lo, bool fold_hi,
                                                int part, T r0, T r1, T (&x)[H], int& k0, int& mh) {
  static_assert(P == 2 || P == 4, "groups of two or four lanes");
  constexpr int N = 2 * (P - 1);
  auto size = [&](int q) { return FULL ? H : (m + P - 1 - q) / P; };
  k0 = 0;
#pragma unroll
  for (int q = 0; q < P - 1; ++q)
    if (q < part) k0 += size(q);
  mh = size(part);
  const int np = min(P, m);
  const bool lo = fold_lo && part == 0, hi = fold_hi && part == np - 1;
  // forward: LU of the part and the forward sweep of e_first (y_j / u_j in f)
  T cu[H], f[H], g[H];
  T iu_prev = T(1), c_prev = T(0), y_prev = T(1);
  T aF = T(0), cL = T(0), iuL = T(0);
#pragma unroll
  for (int j = 0; j < H; ++j) {
    if (FULL || j < mh) {
      const int k = k0 + j;
      T a, b, c;
      tri_coef(dpos(Dl[k * ds]), dpos(Dl[(k + 1) * ds]), dpos(Dl[(k + 2) * ds]), tc, a, b, c);
      if (j == 0 && lo) b -= a;
      if (j == mh - 1 && hi) b -= c;
      T u, y;
      if (j == 0) {
        u = b;
        y = T(1);
        aF = part > 0 ? a : T(0);
      } else {
        const T l = a * iu_prev;
        u = b - l * c_prev;
        y = -l * y_prev;
      }
      const T iu = rcp_n(u);
      cu[j] = c * iu;
      f[j] = y * iu;
      if (j == mh - 1) {
        cL = part < np - 1 ? c : T(0);
        iuL = iu;
      }
      y_prev = y;
      iu_prev = iu;
      c_prev = c;
    }
  }
  // backward sweeps of f and of g (g is iu at the last row, zero before it
  // in the forward sweep)
  T fn = T(0), gn = T(0);
#pragma unroll
  for (int j = H - 1; j >= 0; --j) {
    if (FULL || j < mh) {
      const bool last = j == mh - 1;
      const T fv = last ? f[j] : f[j] - cu[j] * fn;
      const T gv = last ? iuL : -cu[j] * gn;
      f[j] = fv;
      g[j] = gv;
      fn = fv;
      gn = gv;
    }
  }
  const bool any = FULL || mh > 0;
  const T fF = any ? f[0] : T(0), gF = any ? g[0] : T(0);
  T fL = T(0), gL = T(0);
#pragma unroll
  for (int j = 0; j < H; ++j)
    if ((FULL || j < mh) && j == mh - 1) {
      fL = f[j];
      gL = g[j];
    }
  const T rf = part == 0 ? r0 : T(0), rl = part == np - 1 ? r1 : T(0);
  // the end values group_solve gathers: x-hat, w, v at the first and last row
  const T xL = rf * fL + rl * gL, wL = aF * fL, vL = cL * gL;
  const T xF = rf * fF + rl * gF, wF = aF * fF, vF = cL * gF;
  const int base = (int)(threadIdx.x & 63) & ~(P - 1);
  T gxL[P], gwL[P], gvL[P], gxF[P], gwF[P], gvF[P];
#pragma unroll
  for (int q = 0; q < P; ++q) {
    gxL[q] = __shfl(xL, base + q, 64);
    gwL[q] = __shfl(wL, base + q, 64);
    gvL[q] = __shfl(vL, base + q, 64);
    gxF[q] = __shfl(xF, base + q, 64);
    gwF[q] = __shfl(wF, base + q, 64);
    gvF[q] = __shfl(vF, base + q, 64);
  }
  T M[N][N], rv[N];
#pragma unroll
  for (int e = 0; e < N; ++e) {
    rv[e] = T(0);
#pragma unroll
    for (int q = 0; q < N; ++q) M[e][q] = e == q ? T(1) : T(0);
  }
#pragma unroll
  for (int i = 0; i < P - 1; ++i) {
    if (i < np - 1) {
      M[2 * i][2 * i + 1] = gvL[i];
      if (i > 0) M[2 * i][2 * i - 2] = gwL[i];
      rv[2 * i] = gxL[i];
      M[2 * i + 1][2 * i] = gwF[i + 1];
      if (i + 1 < P - 1) M[2 * i + 1][2 * i + 3] = gvF[i + 1];
      rv[2 * i + 1] = gxF[i + 1];
    }
  }
  T id[N];
#pragma unroll
  for (int e = 0; e < N; ++e) {
    id[e] = rcp_n(M[e][e]);
#pragma unroll
    for (int q = e + 1; q < N; ++q) {
      const T l = M[q][e] * id[e];
#pragma unroll
      for (int h = e; h < N; ++h) M[q][h] -= l * M[e][h];
      rv[q] -= l * rv[e];
    }
  }
  T z[N];
#pragma unroll
  for (int e = N - 1; e >= 0; --e) {
    T t = rv[e];
#pragma unroll
    for (int q = e + 1; q < N; ++q) t -= M[e][q] * z[q];
    z[e] = div_n(t, M[e][e], id[e]);
  }
  T Rp = T(0), Lm = T(0);
#pragma unroll
  for (int q = 0; q < P; ++q)
    if (q == part) {
      if (q < P - 1) Rp = z[2 * q + 1];
      if (q > 0) Lm = z[2 * q - 2];
    }
  const T cf = rf - aF * Lm, cg = rl - cL * Rp;
#pragma unroll
  for (int j = 0; j < H; ++j)
    if (FULL || j < mh) x[j] = cf * f[j] + cg * g[j];
}
template <typename T, int H, int P>
__device__ __forceinline__ void group_response(const T* Dl, int ds, int m, const T* tc, bool fold_lo, bool fold_hi,
                                               int part, T r0, T r1, T (&x)[H], int& k0, int& mh) {
  if (m == P * H) group_response_<T, H, P, true>(Dl, ds, m, tc, fold_lo, fold_hi, part, r0, r1, x, k0, mh);
  else group_response_<T, H, P, false>(Dl, ds, m, tc, fold_lo, fold_hi, part, r0, r1, x, k0, mh);
}

// Work-groups of a launch are dealt round-robin to the 8 XCDs (each with its
// own L2): block b runs on XCD b % 8.  Renumber so that every XCD walks a
// contiguous run of tiles; a tile's halo rows and columns are then mostly
// the neighbour tiles' interiors, fetched from HBM once into the same L2.
constexpr int NXCD = 8;
__device__ __forceinline__ int xcd_tile(int b, int nb) {
  const int xcd = b % NXCD, local = b / NXCD;
  const int per = nb / NXCD, rem = nb % NXCD;
  return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// Work item (tile or line) of a launch -> (domain, index within it).  A
// batch carries a packed map, one word per item: domain << MAP_SHIFT | index
// (a single dependent load, no search); a single domain is the identity.
constexpr int MAP_SHIFT = 18;
__device__ __forceinline__ void locate(const int* map, int nd, int idx, int& dom, int& loc) {
  if (nd == 1) {
    dom = 0;
    loc = idx;
    return;
  }
  const int v = map[idx];
  dom = v >> MAP_SHIFT;
  loc = v & ((1 << MAP_SHIFT) - 1);
}

// ---------------------------------------------------------------------------
// k_dt: Delta t and weights of the step (one block per domain)
// ---------------------------------------------------------------------------

// whole-state copies through the global address space: one batch of loads
// or stores (a generic pointer would make them flat accesses, which also
// wait on the LDS counter)
__device__ __forceinline__ DevState load_state(const DevState* st) {
  constexpr int NW = (int)(sizeof(DevState) / 8);
  static_assert(sizeof(DevState) % 8 == 0, "state is whole 8-byte words");
  const gp<const unsigned long long> src = gbl((const unsigned long long*)st);
  unsigned long long w[NW];
#pragma unroll
  for (int k = 0; k < NW; ++k) w[k] = src[k];
  DevState S;
  __builtin_memcpy(&S, w, sizeof S);
  return S;
}
__device__ __forceinline__ void store_state(DevState* st, const DevState& S) {
  constexpr int NW = (int)(sizeof(DevState) / 8);
  unsigned long long w[NW];
  __builtin_memcpy(w, &S, sizeof S);
  const gp<unsigned long long> dst = gbl((unsigned long long*)st);
#pragma unroll
  for (int k = 0; k < NW; ++k) dst[k] = w[k];
}

__device__ __forceinline__ void commit(DevState& st) {
  if (st.pending) {
    st.t = st.t_next;
    st.dt3 = st.dt2;
    st.dt2 = st.dt1;
    st.dt1 = st.dt;
    st.n += 1;
    st.pending = 0;
  }
}

// f over the 64 lanes of a wave in the order of a butterfly (32, 16, ... 1
// lanes apart; f commutes), every lane with the result.  Row swaps and DPP
// instead of shuffles, which take an LDS trip per word and level.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
}
template <typename F>
__device__ __forceinline__ double wave_fold(double v, F f) {
  const auto both = [](auto lo, auto hi, int k) { return __hiloint2double((int)hi[k], (int)lo[k]); };
  {
    const unsigned l = (unsigned)__double2loint(v), h = (unsigned)__double2hiint(v);
    const auto lo = __builtin_amdgcn_permlane32_swap(l, l, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(h, h, false, false);
    v = f(both(lo, hi, 0), both(lo, hi, 1));
  }
  {
    const unsigned l = (unsigned)__double2loint(v), h = (unsigned)__double2hiint(v);
    const auto lo = __builtin_amdgcn_permlane16_swap(l, l, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(h, h, false, false);
    v = f(both(lo, hi, 0), both(lo, hi, 1));
  }
  v = f(v, dpp<0x128>(v));   // row_ror:8
  v = f(v, dpp<0x124>(v));   // row_ror:4, of a row that repeats after 8 lanes
  v = f(v, dpp<0x4e>(v));    // quad_perm 2 3 0 1
  return f(v, dpp<0xb1>(v)); // quad_perm 1 0 3 2
}

// one component of the incident wave train at west ghost column c = 0, 1 (its
// centre is at x = -(c + 1/2) dx)
struct WestTerm {
  double amp, om, ph, ck, hk;     // ck = om / k, hk = (c + 1/2) k
};
template <typename T>
__device__ __forceinline__ WestTerm west_term(const DomDev<T>& D, int m, int c) {
  const int nw = D.n_waves;
  const double k = D.wave[3 * nw + m], om = D.wave[nw + m];
  return {D.wave[m], om, D.wave[2 * nw + m], om / k, (c == 0 ? 0.5 : 1.5) * k};
}
__device__ __forceinline__ double west_ramp(double ramp, double t) {
  return ramp > 0.0 ? 1.0 - exp(-(t / ramp) * (t / ramp)) : 1.0;
}
// surface and flux that the wave train prescribes in ghost column c at time t,
// summed by one wave; w is its lanes' first component
template <typename T>
__device__ __forceinline__ void west_train(const DomDev<T>& D, double t, int c, WestTerm w, double& gw, double& gP) {
  const int lane = threadIdx.x & 63, nw = D.n_waves;
  const double r = west_ramp(D.wave_ramp, t);
  double a = 0, b = 0;
  for (int m = lane; m < nw; m += 64) {
    if (m != lane) w = west_term(D, m, c);
    const double s = r * w.amp * sin(fma_(w.hk, D.dx_d, w.om * t) + w.ph);
    a += s;
    b += w.ck * s;
  }
  const auto add = [](double x, double y) { return x + y; };
  gw = wave_fold(a, add);
  gP = wave_fold(b, add);
}
// a boundary series' values at time t: samples interpolated linearly in time,
// held outside their span; the same values in both ghost columns
template <typename T>
__device__ __forceinline__ void west_series(const DomDev<T>& D, double t, double& gw, double& gP) {
  const int n = D.ts_n;
  const double* se = D.wave;
  const double* sp = D.wave + n;
  const double s = t / D.ts_dt, r = west_ramp(D.wave_ramp, t);
  double e, p;
  if (!(s > 0.0)) {
    e = se[0];
    p = sp[0];
  } else if (s >= (double)(n - 1)) {
    e = se[n - 1];
    p = sp[n - 1];
  } else {
    const int k = (int)s;
    const double f = s - (double)k;
    e = se[k] + f * (se[k + 1] - se[k]);
    p = sp[k] + f * (sp[k + 1] - sp[k]);
  }
  gw = r * e;
  gP = r * p;
}

// one block of DT_THREADS per domain
constexpr int DT_THREADS = 256;

template <typename T>
__global__ void __launch_bounds__(DT_THREADS) k_dt(const DomDev<T>* __restrict__ doms, double dt_prescribed) {
  const DomDev<T>& D = doms[blockIdx.x];
  DevState* st = D.st;
  __shared__ int go;
  __shared__ double tn;
  // The state and the step controls are loaded first, in one batch, so their
  // latency overlaps the reduction below (the barrier in it keeps the state's
  // loads here); the decision further down is then register arithmetic.
  DevState S = load_state(st);
  const double t_end = D.t_end, cfl = D.cfl, ema = D.ema_alpha, dt_init = D.dt_init, dt_max = D.dt_max,
               dt_min = D.dt_min;
  const int fixed_dt = D.fixed_dt, fstar_order = D.fstar_order, corrector = D.corrector;
  __asm__ volatile("" ::"s"(t_end), "s"(cfl), "s"(ema), "s"(dt_init), "s"(dt_max), "s"(dt_min), "s"(fixed_dt),
                   "s"(fstar_order), "s"(corrector));
  // the wave train's components too, the waves 1 and 2 for a ghost column
  // each: what does not depend on the new time is formed while one thread
  // of wave 0 decides the step.  This kernel is latency alone: with both
  // columns in wave 0, loaded after the decision, a step took 35.4 us on 1024
  // x 256 FP64 for 34.9, 26.5 for 25.8 in FP32, 27.0 for 26.3 on 333 x 217
  const int bc0 = D.bc[0], nw = D.n_waves, lane = threadIdx.x & 63, col = uni((int)(threadIdx.x >> 6)) - 1;
  const bool train = (bc0 == SINE || bc0 == IRREGULAR) && (col == 0 || col == 1);
  WestTerm wt = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (train && lane < nw) wt = west_term(D, lane, col);
  // CFL maximum of the current state: the finalize kernel's per-tile maxima
  // (a NaN there is already +inf) and the initial state's value
  double tmax = 0.0;
  {
    // eight independent loads in flight per lane (a large domain has
    // thousands of tiles; one dependent load at a time would serialise them)
    const int ntiles = D.tiles_x * D.tiles_y;
    const gp<const double> sp = gbl((const double*)D.smax_tile);
    double tm[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) tm[u] = 0.0;
    for (int k0 = threadIdx.x; k0 < ntiles; k0 += 8 * DT_THREADS) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = k0 + DT_THREADS * u;
        tm[u] = fmax(tm[u], k < ntiles ? sp[k] : 0.0);
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) tmax = fmax(tmax, tm[u]);
    tmax = wave_fold(tmax, [](double x, double y) { return fmax(x, y); });
    __shared__ double wmax[DT_THREADS / 64];
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = tmax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < DT_THREADS / 64; ++w) tmax = fmax(tmax, wmax[w]);
  }
  if (threadIdx.x == 0) {
    // one thread decides the step on the register copy of the state and
    // stores it back in one batch
    commit(S);
    go = 0;
    S.halt = 1;
    if (S.status == ST_OK) {
      if (t_end > 0.0 && S.t >= t_end) {
        S.status = ST_EDONE;
      } else {
        const double s = fmax(__longlong_as_double((long long)S.smax_bits), tmax);
        if (!(s <= 1.79e308)) {
          S.status = ST_ENONFINITE;
        } else {
          const long long n = S.n;
          double dt;
          bool ok = true;
          if (dt_prescribed > 0.0) {
            dt = dt_prescribed;
          } else if (fixed_dt) {
            dt = dt_init;
          } else {
            const double cand = s > 0.0 ? cfl / s : dt_max;
            if (n == 0) dt = dt_init > 0.0 ? dt_init : cand;
            else dt = cand <= S.dt1 ? cand : ema * cand + (1.0 - ema) * S.dt1;
            dt = fmin(dt, dt_max);
            if (dt < dt_min) {
              S.status = ST_EDTMIN;
              ok = false;
            }
          }
          if (ok) {
            // one thread, FP64: the weights are formed from three
            // reciprocals (a division is a long dependent chain here)
            const double h0 = dt, h1 = S.dt1, h2 = S.dt2;
            const double i1 = 1.0 / h1, i2 = n >= 2 ? 1.0 / h2 : 0.0, h6 = h0 * (1.0 / 6.0);
            double a0 = h0, a1 = 0.0, a2 = 0.0, b0 = 0.0, b1 = 0.0, b2 = 0.0;
            if (n == 1) {
              b0 = h0 * i1;
              b1 = -b0;
            } else if (n >= 2) {
              // Eq. (42): integral over [t_n, t_n + h0] of the quadratic
              // through the three last nodes
              const double r1 = h0 * i1, s12 = h1 + h2, is = 1.0 / s12;
              a0 = h6 * (r1 * (2.0 * h0 + 6.0 * h1 + 3.0 * h2) * is + 6.0);
              a1 = -h6 * (r1 * (2.0 * h0 + 3.0 * h1 + 3.0 * h2) * i2);
              a2 = h6 * ((h0 * i2) * (2.0 * h0 + 3.0 * h1) * is);
              if (fstar_order == 1) {
                b0 = r1;
                b1 = -r1;
              } else {
                // Eq. (43) with (44)-(46) sum to the increment of the quadratic
                // through (t_{n-k}, F*^{n-k}) from t_n to t_n + h0
                b0 = (h0 + h1) * (h0 + s12) * (i1 * is) - 1.0;
                b1 = -h0 * (h0 + s12) * (i1 * i2);
                b2 = h0 * (h0 + h1) * (i2 * is);
              }
            }
            // Adams-Moulton corrector (domains that run it): integral over
            // [t_n, t_n + h0] of the Lagrange basis through t_{n+1}, t_n,
            // t_{n-1}, t_{n-2} (closed forms with a = h1, b = h1 + h2), the
            // cubic from n = 2 on, the quadratic at n = 1, the trapezoidal
            // rule at n = 0
            double g0 = 0.5 * h0, g1 = 0.5 * h0, g2 = 0.0, g3 = 0.0;
            if (corrector && n == 1) {
              const double a = h1;
              g0 = h0 * (2.0 * h0 + 3.0 * a) / (6.0 * (h0 + a));
              g1 = h0 * (h0 + 3.0 * a) / (6.0 * a);
              g2 = -h0 * h0 * h0 / (6.0 * a * (a + h0));
            } else if (corrector && n >= 2) {
              const double a = h1, b = h1 + h2, hh = h0 * h0 * h0;
              g0 = h0 * (3.0 * h0 * h0 + 4.0 * (a + b) * h0 + 6.0 * a * b) / (12.0 * (h0 + a) * (h0 + b));
              g1 = h0 * (h0 * h0 + 2.0 * (a + b) * h0 + 6.0 * a * b) / (12.0 * a * b);
              g2 = -hh * (h0 + 2.0 * b) / (12.0 * a * (a + h0) * h2);
              g3 = hh * (h0 + 2.0 * a) / (12.0 * b * (b + h0) * h2);
            }
            S.dt = dt;
            S.alpha[0] = a0; S.alpha[1] = a1; S.alpha[2] = a2;
            S.gamma[0] = g0; S.gamma[1] = g1; S.gamma[2] = g2; S.gamma[3] = g3;
            S.beta[0] = b0; S.beta[1] = b1; S.beta[2] = b2;
            S.t_next = S.t + dt;
            S.smax_used = s;
            S.slot = (int)(n % 3);
            S.smax_bits = 0ull;
            S.pending = 1;
            S.halt = 0;
            go = 1;
            tn = S.t_next;
          }
        }
      }
    }
    store_state(st, S);
  }
  __syncthreads();
  if (!go) return;
  double gw, gP;
  if (train) {
    west_train(D, tn, col, wt, gw, gP);
    if (lane == 0) {
      st->gw[col] = gw;
      st->gP[col] = gP;
    }
  } else if (bc0 == TIMESERIES && threadIdx.x == 0) {
    west_series(D, tn, gw, gP);
    st->gw[0] = st->gw[1] = gw;
    st->gP[0] = st->gP[1] = gP;
  }
}

template <typename T>
__global__ void k_commit(const DomDev<T>* __restrict__ doms, int nd) {
  const int d = blockIdx.x * blockDim.x + threadIdx.x;
  if (d < nd) commit(*doms[d].st);
}

// ---------------------------------------------------------------------------
// k_rhs: fused spatial operator, AB3 update and chunk-local line solves
// ---------------------------------------------------------------------------

template <typename T, int TY, int MX>
struct alignas(16) RhsSmem {
  static constexpr int WX = TX + 4, WY = TY + 4;      // radius-2 tiles
  static constexpr int BX = TX + 2, BY = TY + 2;      // radius-1 tiles
  static constexpr int CXN = TX + 5, CYN = TY + 5;    // corners
  static constexpr int TXP = TX + 1;                  // padded row of the solve buffers
  // LDS row pitch of the radius-2 tiles: 5 mod 32 words, so that the lane
  // layouts of the per-cell phases (cell_of: CPT-strided columns of CPT rows
  // per half-wave) and of the chunk solves hit 32 distinct banks
  static constexpr int LW = WX + 1;
  static constexpr int AXP = TX + 1;                  // row pitch of ay (same reason)
  // the corner tile is staged in pairs from corner i0 - 2, one corner past
  // the CXN used; its row pitch is 9 mod 32 words for the face passes
  static constexpr int CP = CXN + 4;
  // the weighted P/Q history is kept on radius-1 rows in the columns of the
  // radius-2 tile (its pairs load like the radius-2 rows), row pitch 5 mod
  // 32 words like LW (the F* reads of a thread's consecutive cells)
  static constexpr int PW = WX + 1;
  static_assert(LW % 32 == PITCH_MOD_TILE && PW % 32 == PITCH_MOD_TILE && AXP % 32 == PITCH_MOD_ROWS &&
                    TXP % 32 == PITCH_MOD_ROWS && CP % 32 == PITCH_MOD_CORNERS,
                "the lane layouts assume these row pitches");
  T w[WY * LW];
  T p[WY * LW];
  T q[WY * LW];
  T db[WY * LW];                                      // cell still-water depth
  union {
    struct {
      T pt[BY * PW];                                  // sum_k beta_k P^{n-k} (until the F* terms are formed)
      T qt[BY * PW];
    } h;
    T ay[3][TY * AXP];                                // y-direction parts of E, F, G per cell
    struct {
      T u[TY * TXP];
      T v[TY * TXP];
    } s;
  } x;
  T dc[CYN * CP];
};

// CORR = false: the AB3 step of Eq. (42)-(43) from level n (the predictor
// when the domain runs the corrector, which then writes the surface to w[2]).
// CORR = true: the Adams-Moulton corrector from the same base w^n, U*^n, V*^n
// with the spatial operator of the predicted level (slot of level n+1, w[2])
// and the F*, G* terms as their change F*(P*) - F*(P^n); domains without the
// corrector are skipped.
//
// THREADS: NT, or more in launches of few tiles (rhs_threads in the host code).
// BIG: some field of the domain exceeds 4 GiB, the reach of a lane's byte
// offset (ldu, ldv), so that every field is addressed from the tile's corner.
// The 60 scalar additions this takes cost 1 to 2 % of a step (333 x 217 FP64
// 5590 -> 5696 us for 200, 2048^2 FP32 80.0 -> 81.3 ms for 600): the launches
// of smaller fields go without.
template <typename T, int TY, int MX, bool CORR, int THREADS = NT, bool BIG = false>
__global__ void __launch_bounds__(THREADS) k_rhs(const DomDev<T>* __restrict__ doms, const int* __restrict__ tile_map,
                                           int nd, int swizzle) {
  using S = RhsSmem<T, TY, MX>;
  constexpr int WX = S::WX, LW = S::LW, AXP = S::AXP, CXN = S::CXN, CP = S::CP, PW = S::PW, TXP = S::TXP;
  constexpr int CPT = (TX * TY) / THREADS;                 // cells per thread
  static_assert((TX * TY) % THREADS == 0, "tile must be a multiple of the block");
  using V = Vec<T, CPT>;
  using V2 = Vec<T, 2>;
  __shared__ S sm;
  int dom, tile;
  // swizzle = 1: XCD-aware tile order (each XCD walks a contiguous run)
  locate(tile_map, nd, swizzle ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x, dom, tile);
  const DomDev<T>& D = doms[dom];
  const DevState* st = D.st;
  if (st->halt) return;
  if (CORR && !D.corrector) return;
  const int i0 = (tile % D.tiles_x) * TX, j0 = (tile / D.tiles_x) * TY;
  const int nx = D.nx, ny = D.ny, tid = threadIdx.x;
  // The step's scalars are read (and made wave-uniform) before any field
  // load is issued: the state is read through vector loads, whose waits are
  // in issue order and would otherwise also wait for the field loads.
  const int slot = uni(st->slot), par = uni((int)(st->n & 1));
  const int s1 = slot == 0 ? 2 : slot - 1, s2 = slot == 2 ? 0 : slot + 1;
  const double sb0 = uni(st->beta[0]), sb1 = uni(st->beta[1]), sb2 = uni(st->beta[2]);
  const double sa0 = uni(CORR ? st->gamma[0] : st->alpha[0]), sa1 = uni(CORR ? st->gamma[1] : st->alpha[1]);
  const double sa2 = uni(CORR ? st->gamma[2] : st->alpha[2]), sa3 = CORR ? uni(st->gamma[3]) : 0.0;
  const T beta0 = CORR ? T(1) : (T)sb0;
  const T beta1 = CORR ? T(-1) : (T)sb1;
  const T beta2 = CORR ? T(0) : (T)sb2;
  const bool hist = CORR || sb0 != 0.0 || sb1 != 0.0 || sb2 != 0.0;
  const int pitch = uni(D.pitch), xoff = uni(D.xoff), ipitch = uni(D.ipitch), cpitch = uni(D.cpitch);
  // Cells of a thread in the per-cell phases: row vr, columns vc .. vc+CPT-1
  // (consecutive columns: one vector access per field, and the x-face pass
  // below takes the same cells, so its results stay in registers).
  static_assert((TX / CPT) * TY == THREADS, "one row segment per thread");
  int vr, vc;
  cell_of<T, CPT>(tid, vr, vc);
  // BIG: the tile's corner in the fields, as scalars, from which the lanes
  // count; else they count from the fields' first element
  const int jl = BIG ? 0 : j0, il = BIG ? 0 : i0, xo = BIG ? 2 : xoff;
  const size_t tI = BIG ? (size_t)j0 * ipitch + i0 : 0;               // interior fields: cell (i0, j0)
  const size_t tG = BIG ? (size_t)j0 * pitch + xoff + i0 - 2 : 0;     // ghosted fields: cell (i0 - 2, j0 - 2)
  const size_t tC = BIG ? (size_t)j0 * cpitch + i0 : 0;               // corner (i0 - 2, j0 - 2)
  const unsigned oI = (unsigned)((jl + vr) * ipitch + il + vc);
  const unsigned oG = (unsigned)((jl + vr + 2) * pitch + xo + il + vc);

  // ---- phase 0: issue every load of the tile before the first LDS store ----
  // The halo tiles are read in pairs of cells (8 or 16 bytes per lane): a
  // radius-2 row is WX / 2 pairs from cell i0 - 2, a corner row (CXN + 1) / 2
  // pairs from corner i0 - 2, each staged by PairStaging (thread (r0, c)
  // loads rows r0 + RG k, so the LDS index is a per-thread base plus a
  // constant; repeated rows keep every round branch-free).  The workspace
  // pads every field to whole tiles plus the halo, so no index is clamped to
  // the domain: values outside it only reach cells outside it.
  using SW = PairStaging<WX / 2, S::WY, THREADS>;            // radius-2 rows
  using SB = PairStaging<WX / 2, S::BY, THREADS>;            // radius-1 rows, radius-2 columns
  using SC = PairStaging<(CXN + 1) / 2, S::CYN, THREADS>;    // corner rows
  constexpr int KW = SW::K, KB = SB::K, KC = SC::K;
  const int cP = SW::col(tid), cC = SC::col(tid);
  auto rowW = [&](int k) { return SW::row(tid, k); };
  auto rowB = [&](int k) { return SB::row(tid, k); };
  auto rowC = [&](int k) { return SC::row(tid, k); };
  // the history fields' addresses first (a wait for a descriptor read
  // would also wait for every field load issued before it)
  const int l1 = CORR ? slot : s1, l2 = CORR ? s1 : s2;
  const T* const pE1 = uni((const T*)D.E[l1]) + tI;
  const T* const pE2 = uni((const T*)D.E[l2]) + tI;
  const T* const pF1 = uni((const T*)D.F[l1]) + tI;
  const T* const pF2 = uni((const T*)D.F[l2]) + tI;
  const T* const pG1 = uni((const T*)D.G[l1]) + tI;
  const T* const pG2 = uni((const T*)D.G[l2]) + tI;
  const T* const pE3 = CORR ? uni((const T*)D.E[s2]) + tI : nullptr;
  const T* const pF3 = CORR ? uni((const T*)D.F[s2]) + tI : nullptr;
  const T* const pG3 = CORR ? uni((const T*)D.G[s2]) + tI : nullptr;
  V2 rw[KW], rp[KW], rq[KW], rc[KC], h1p[KB], h2p[KB], h1q[KB], h2q[KB];
  // keep the load groups in this order (the waits are in issue order)
  __builtin_amdgcn_sched_barrier(0);
  {
    // the state the spatial operator is taken of: level n, or the predicted level
    const T* w = uni((const T*)(CORR ? D.w[2] : D.w[par])) + tG;
    const T* Pn = uni((const T*)D.P[CORR ? s2 : slot]) + tG;
    const T* Qn = uni((const T*)D.Q[CORR ? s2 : slot]) + tG;
    const unsigned oW = (unsigned)(jl * pitch + xo + il - 2 + cP);         // radius-2 tile
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const unsigned o = oW + (unsigned)(rowW(k) * pitch);
      rw[k] = ldv<2>(w, o);
      rp[k] = ldv<2>(Pn, o);
      rq[k] = ldv<2>(Qn, o);
    }
    const T* Dc = uni((const T*)D.Dc) + tC;
    const unsigned oC = (unsigned)(jl * cpitch + il + cC);                 // corners from i0 - 2
#pragma unroll
    for (int k = 0; k < KC; ++k) rc[k] = ldv<2>(Dc, oC + (unsigned)(rowC(k) * cpitch));
    // radius-1 rows j0-1 .. j0+TY, in the radius-2 tile's columns
    const unsigned oB = (unsigned)((jl + 1) * pitch + xo + il - 2 + cP);
    if (CORR) {
      // level n, for the change of the F*, G* terms
      const T* P1 = uni((const T*)D.P[slot]) + tG;
      const T* Q1 = uni((const T*)D.Q[slot]) + tG;
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const unsigned o = oB + (unsigned)(rowB(k) * pitch);
        h1p[k] = ldv<2>(P1, o);
        h1q[k] = ldv<2>(Q1, o);
        h2p[k] = h2q[k] = V2{{T(0), T(0)}};
      }
    } else {
      // loaded also where a level's weight is zero (before the history
      // exists, and level n-2 with linear F* extrapolation): a branch here
      // would make the waits before the first LDS stores cover these loads
      // as well.  A level that is not needed repeats the addresses of a level
      // that is loaded anyway (n-1, else the staged level n), so its loads
      // hit the cache instead of reaching HBM.
      const int u1 = sb1 != 0.0 ? s1 : slot, u2 = sb2 != 0.0 ? s2 : u1;
      const T* P1 = uni((const T*)D.P[u1]) + tG;
      const T* P2 = uni((const T*)D.P[u2]) + tG;
      const T* Q1 = uni((const T*)D.Q[u1]) + tG;
      const T* Q2 = uni((const T*)D.Q[u2]) + tG;
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const unsigned o = oB + (unsigned)(rowB(k) * pitch);
        h1p[k] = ldv<2>(P1, o);
        h2p[k] = ldv<2>(P2, o);
        h1q[k] = ldv<2>(Q1, o);
        h2q[k] = ldv<2>(Q2, o);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  // E, F, G history of this thread's cells, issued last: they are consumed
  // only in phase 2, so the waits before the first LDS stores do not cover
  // them and their latency overlaps the phases in between
  const V e1 = ldv_nt<CPT>(pE1, oI), e2 = ldv_nt<CPT>(pE2, oI);
  const V f1 = ldv_nt<CPT>(pF1, oI), f2 = ldv_nt<CPT>(pF2, oI);
  const V g1 = ldv_nt<CPT>(pG1, oI), g2 = ldv_nt<CPT>(pG2, oI);
  V e3, f3, g3;
  if (CORR) {
    e3 = ldv_nt<CPT>(pE3, oI);
    f3 = ldv_nt<CPT>(pF3, oI);
    g3 = ldv_nt<CPT>(pG3, oI);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int e = rowW(k) * LW + cP;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      sm.w[e + u] = rw[k].v[u];
      sm.p[e + u] = rp[k].v[u];
      sm.q[e + u] = rq[k].v[u];
    }
  }
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    sm.dc[rowC(k) * CP + cC] = rc[k].v[0];
    sm.dc[rowC(k) * CP + cC + 1] = rc[k].v[1];
  }
  __syncthreads();
  // weighted P/Q history (level n from the staged tile) and cell depths
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    const int r = rowB(k);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t2 = (r + 1) * LW + cP + u;           // same cell in the radius-2 tile
      sm.x.h.pt[r * PW + cP + u] = hist ? beta0 * sm.p[t2] + beta1 * h1p[k].v[u] + beta2 * h2p[k].v[u] : T(0);
      sm.x.h.qt[r * PW + cP + u] = hist ? beta0 * sm.q[t2] + beta1 * h1q[k].v[u] + beta2 * h2q[k].v[u] : T(0);
    }
  }
#pragma unroll
  for (int k = 0; k < KW; ++k) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c0 = rowW(k) * CP + cP + u;
      sm.db[rowW(k) * LW + cP + u] = dbar4(sm.dc[c0], sm.dc[c0 + 1], sm.dc[c0 + CP], sm.dc[c0 + CP + 1]);
    }
  }

  __syncthreads();
  // F*, G* terms of this thread's cells (Eq. 14-15 are linear, so
  // sum_k beta_k F*^{n-k} = F*(sum_k beta_k Q^{n-k})), added to the AB3
  // history terms of U*, V* (Eq. 43) in phase 2; after them the history
  // tiles' LDS holds the y-parts of the face pass
  T fsF[CPT], fsG[CPT];
  {
    const T i2dx = D.i2dx, i2dy = D.i2dy, i4dxdy = D.i4dxdy, Bc = D.Bc;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int r = vr, c = vc + k;
      const int C0 = (r + 2) * LW + c + 2;
      const T d0 = dpos(sm.db[C0]);
      const T ddx = (dpos(sm.db[C0 + 1]) - dpos(sm.db[C0 - 1])) * i2dx;
      const T ddy = (dpos(sm.db[C0 + LW]) - dpos(sm.db[C0 - LW])) * i2dy;
      const int B0 = (r + 1) * PW + c + 2;
      const T qy = (sm.x.h.qt[B0 + PW] - sm.x.h.qt[B0 - PW]) * i2dy;
      const T qx = (sm.x.h.qt[B0 + 1] - sm.x.h.qt[B0 - 1]) * i2dx;
      const T qxy = ((sm.x.h.qt[B0 + PW + 1] - sm.x.h.qt[B0 - PW + 1]) -
                     (sm.x.h.qt[B0 + PW - 1] - sm.x.h.qt[B0 - PW - 1])) * i4dxdy;
      const T py = (sm.x.h.pt[B0 + PW] - sm.x.h.pt[B0 - PW]) * i2dy;
      const T px = (sm.x.h.pt[B0 + 1] - sm.x.h.pt[B0 - 1]) * i2dx;
      const T pxy = ((sm.x.h.pt[B0 + PW + 1] - sm.x.h.pt[B0 - PW + 1]) -
                     (sm.x.h.pt[B0 + PW - 1] - sm.x.h.pt[B0 - PW - 1])) * i4dxdy;
      fsF[k] = d0 * ddx * qy * T(1.0 / 6.0) + d0 * ddy * qx * T(1.0 / 6.0) + Bc * d0 * d0 * qxy;
      fsG[k] = d0 * ddx * py * T(1.0 / 6.0) + d0 * ddy * px * T(1.0 / 6.0) + Bc * d0 * d0 * pxy;
      pin(fsF[k]);
      pin(fsG[k]);
    }
  }
  // AB3 history terms alpha_1 X^{n-1} + alpha_2 X^{n-2} (Eq. 42), the
  // corrector's gamma_1 X^n + gamma_2 X^{n-1} + gamma_3 X^{n-2}.  FP64 forms
  // them here: the loads have had the F* phase to arrive, and the face passes
  // then run with 24 registers in the place of 64 (1024 x 256: 19.9 -> 18.4
  // us); FP32 after the face passes, where they cost it nothing.
  T hE[CPT], hF[CPT], hG[CPT];
  auto history = [&]() {
    const T a1 = (T)sa1, a2 = (T)sa2;
    const T a3 = CORR ? (T)sa3 : T(0);
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      hE[k] = a1 * e1.v[k] + a2 * e2.v[k];
      hF[k] = a1 * f1.v[k] + a2 * f2.v[k];
      hG[k] = a1 * g1.v[k] + a2 * g2.v[k];
      if (CORR) {
        hE[k] += a3 * e3.v[k];
        hF[k] += a3 * f3.v[k];
        hG[k] += a3 * g3.v[k];
      }
      hF[k] += fsF[k];
      hG[k] += fsG[k];
    }
  };
  if constexpr (sizeof(T) == 8) {
    history();
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      pin(hE[k]);
      pin(hF[k]);
      pin(hG[k]);
    }
  }
  __syncthreads();
  const T g = D.g, eps = D.eps, ht = T(0.5) * D.theta;
  const T idx = D.idx, idy = D.idy;
  // ---- phase 1x: x-faces by row segments, kept in registers -----------------
  // The thread's own cells (the last face is also its right neighbour's
  // first); it keeps the x-parts of its cells' E, F, G.
  T acc_e[CPT], acc_f[CPT], acc_g[CPT];
  {
    const T* c0 = sm.dc + (vr + 2) * CP + vc + 1;     // corners of face vc - 1
    T Dfx[CPT + 3];                                   // still-water depth of face vc - 1 + k
#pragma unroll
    for (int k = 0; k < CPT + 3; ++k) Dfx[k] = T(0.5) * (c0[k] + c0[k + CP]);
    const int o = (vr + 2) * LW + vc;                 // tile column vc = cell vc - 2
    face_pass<T, CPT>(sm.w + o, sm.p + o, sm.q + o, 1, Dfx, ht, eps, g, acc_e, acc_f, acc_g);
  }
  // ---- phase 1y: y-faces by column segments, parts to LDS -------------------
  // normal = Q, tangential = P; thread cells (rY0 + q, cY)
  {
    const int cY = tid % TX, rY0 = (tid / TX) * CPT;
    const T* c0 = sm.dc + (rY0 + 1) * CP + cY + 2;    // corners of face rY0 - 1
    T Dfy[CPT + 3];
#pragma unroll
    for (int k = 0; k < CPT + 3; ++k) Dfy[k] = T(0.5) * (c0[k * CP] + c0[k * CP + 1]);
    const int o = rY0 * LW + cY + 2;                  // tile row rY0 = row rY0 - 2
    T ye[CPT], yg[CPT], yf[CPT];
    face_pass<T, CPT>(sm.w + o, sm.q + o, sm.p + o, LW, Dfy, ht, eps, g, ye, yg, yf);
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int oy = (rY0 + k) * AXP + cY;
      sm.x.ay[0][oy] = ye[k] * idy;
      sm.x.ay[1][oy] = yf[k] * idy;                   // x-momentum through y-faces
      sm.x.ay[2][oy] = yg[k] * idy;                   // y-momentum
    }
  }
  __syncthreads();

  // ---- phase 2: per-cell right-hand sides and AB3 update -------------------
  const T B = D.B, gn2 = D.gn2, cf = D.cf;
  const T a0 = (T)sa0;
  T* const wn = uni(CORR ? D.w[par ^ 1] : (D.corrector ? D.w[2] : D.w[par ^ 1])) + tG;
  const T* const wbase = uni((const T*)D.w[par]) + tG;   // w^n (the corrector's base)
  // The thread's cells are consecutive columns of one row, and the body is
  // branch-free, so the stencil reads and the eta / depth values they share
  // are formed once for all of them (cells outside the domain compute
  // harmless values and store nothing).
  const T i2dx = D.i2dx, i2dy = D.i2dy, idx2 = D.idx2, idy2 = D.idy2, i4dxdy = D.i4dxdy;
  const T i2dx3 = D.i2dx3, i2dy3 = D.i2dy3, i2dxdy2 = D.i2dxdy2, i2dx2dy = D.i2dx2dy;
  const T Bg = B * g;
  static_assert(S::AXP == TXP, "U*, V* alias the y-parts cell by cell");
  const bool row_in = j0 + vr < ny;
  const bool all_in = row_in && i0 + vc + CPT <= nx;
  if constexpr (sizeof(T) == 4) history();
  // eta = w + min(D, 0) over the radius-2 tile, formed once per cell for the
  // dispersive stencils below (in the staging's cell mapping) into the
  // corner tile's words, which nothing reads after the face passes; the
  // depth tile keeps d = max(D, 0) from here on (h = w + D = eta + d)
  T* const eta = sm.dc;
  static_assert(S::CYN * S::CP >= S::WY * LW, "the eta tile fits in the corner tile");
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    // every cell by one thread only: the staging's repeated rows (threads
    // past the last whole row, rows past the tile) would read a depth that
    // another wave has already clamped
    if (SW::owns(tid, k)) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int e = rowW(k) * LW + cP + u;
        const T De = sm.db[e];
        eta[e] = sm.w[e] + dneg(De);
        sm.db[e] = dpos(De);
      }
    }
  }
  __syncthreads();
  V ve, vf, vg, vw;
  V wb;
  if (CORR) wb = ldv<CPT>(wbase, oG);
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int r = vr, c = vc + k;
    const bool in = row_in & (i0 + c < nx);
    const int C0 = (r + 2) * LW + c + 2;   // radius-2 tile index of the cell
    const int o = r * AXP + c;
    T e_ = fma_(acc_e[k], idx, sm.x.ay[0][o]);
    T f_ = fma_(acc_f[k], idx, sm.x.ay[1][o]);
    T g_ = fma_(acc_g[k], idx, sm.x.ay[2][o]);
    const T d0 = sm.db[C0];
    const T dxm = sm.db[C0 - 1], dxp = sm.db[C0 + 1];
    const T dym = sm.db[C0 - LW], dyp = sm.db[C0 + LW];
    const T ddx = (dxp - dxm) * i2dx, ddy = (dyp - dym) * i2dy;
    // dispersive terms of Eq. (12)-(13): eta = h - d = w + min(D, 0); they
    // vanish with d0 on land
    {
#define ETA(o) eta[C0 + (o)]
      const T e00 = ETA(0);
      const T exm = ETA(-1), exp_ = ETA(1), eym = ETA(-LW), eyp = ETA(LW);
      const T emm = ETA(-LW - 1), epm = ETA(-LW + 1), emp = ETA(LW - 1), epp = ETA(LW + 1);
      const T exm2 = ETA(-2), exp2 = ETA(2), eym2 = ETA(-2 * LW), eyp2 = ETA(2 * LW);
#undef ETA
      const T exx = (exp_ - T(2) * e00 + exm) * idx2;
      const T eyy = (eyp - T(2) * e00 + eym) * idy2;
      const T exy = ((epp - epm) - (emp - emm)) * i4dxdy;
      const T exxx = ((exp2 - exm2) - T(2) * (exp_ - exm)) * i2dx3;
      const T eyyy = ((eyp2 - eym2) - T(2) * (eyp - eym)) * i2dy3;
      const T exyy = ((epp - T(2) * exp_ + epm) - (emp - T(2) * exm + emm)) * i2dxdy2;
      const T exxy = ((epp - T(2) * eyp + emp) - (epm - T(2) * eym + emm)) * i2dx2dy;
      const T bg = Bg * d0 * d0;
      f_ += bg * d0 * (exxx + exyy) + bg * (ddx * (T(2) * exx + eyy) + ddy * exy);
      g_ += bg * d0 * (eyyy + exxy) + bg * (ddy * (T(2) * eyy + exx) + ddx * exy);
    }
    // bottom friction f1, f2 at the cell centre: Manning g n^2 u |U| / h^(1/3)
    // plus the quadratic law f u |U|
    const T Pc = sm.p[C0], Qc = sm.q[C0];
    if (gn2 > T(0) || cf > T(0)) {
      const T h = fmax(eta[C0] + d0, T(0));
      const T vfc = vfac(h, eps);
      const T u = Pc * vfc, v = Qc * vfc;
      const T kf = h > T(0) ? (gn2 * frcbrt(h) + cf) * fsqrt(u * u + v * v) : T(0);
      f_ -= kf * u;
      g_ -= kf * v;
    }
    // Eq. (42)-(43)
    ve.v[k] = e_;
    vf.v[k] = f_;
    vg.v[k] = g_;
    vw.v[k] = (CORR ? wb.v[k] : sm.w[C0]) + (a0 * e_ + hE[k]);
    // increments U*^{n+1} - U*^n, V*^{n+1} - V*^n (Eq. 43); the line solves
    // below act on them: P^{n+1} = P^n + T^-1 (U*^{n+1} - U*^n) since
    // U*^n = T P^n with the same matrix.  They overwrite this cell's own
    // y-parts (same word of the union), which no other thread reads, so no
    // barrier is needed between the two.
    sm.x.s.u[o] = in ? a0 * f_ + hF[k] : T(0);
    sm.x.s.v[o] = in ? a0 * g_ + hG[k] : T(0);
  }
  {
    T* const E0 = uni(D.E[slot]) + tI;
    T* const F0 = uni(D.F[slot]) + tI;
    T* const G0 = uni(D.G[slot]) + tI;
    if (all_in) {
      if (!CORR) {
        stv_nt(E0, oI, ve);
        stv_nt(F0, oI, vf);
        stv_nt(G0, oI, vg);
      }
      stv_nt(wn, oG, vw);
    } else if (row_in) {
      // the domain's last cells end inside this vector
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        if (i0 + vc + k >= nx) break;
        if (!CORR) {
          stu(E0, oI + k, ve.v[k]);
          stu(F0, oI + k, vf.v[k]);
          stu(G0, oI + k, vg.v[k]);
        }
        stu(wn, oG + k, vw.v[k]);
      }
    }
  }
  __syncthreads();

  // ---- phase 3: chunk-local solves of Eq. (19) (x) and Eq. (20) (y) -------
  // lane groups per chunk (group_solve; parts of 8 rows along x, two
  // halves along y): the x-chunks in the first PX TY NCX threads, the
  // y-chunks (tile columns) in the last 2 TX
  constexpr int NCX = TX / MX;                  // x-chunks per tile row
  constexpr int PX = MX / 8;                    // lanes per x-chunk
  static_assert(TX % MX == 0, "chunks must tile the tile width");
  static_assert(PX * TY * NCX <= THREADS - 2 * TX, "x- and y-chunk solver groups must fit the block");
  const bool wave_w = west_driven(D.bc[0]);
  if (tid < PX * TY * NCX) {
    const int qq = tid / PX, part = tid - qq * PX;
    int r, qc;
    xchunk_of<T, TY, NCX, PX>(qq, r, qc);
    const int j = j0 + r, is = i0 + qc * MX;
    if (j < ny && is < nx) {
      const int m = min(MX, nx - is);
      // depths of cells is-1 .. is+m (tile columns qc*MX+1 ..)
      const T* dlx = sm.db + (r + 2) * LW + qc * MX + 1;
      T* rhs = sm.x.s.u + r * TXP + qc * MX;
      if (is == 0 && wave_w && part == 0) {
        // Dirichlet ghost: the increment of P_{-1} from t_n to t_{n+1}
        T a, b, c;
        tri_coef(dlx[0], dlx[1], dlx[2], D.tcx, a, b, c);
        const T pg = CORR ? D.P[slot][(size_t)(j + 2) * pitch + xoff - 1] : sm.p[(r + 2) * LW + 1];
        rhs[0] -= a * ((T)st->gP[0] - pg);
      }
      T xs[8], xlast;
      int k0, mh;
      group_solve<T, 8, PX, true>(dlx, 1, m, D.tcx, is == 0 && !wave_w, is + m == nx, part,
                                  [&](int k) { return rhs[k]; }, xs, k0, mh, xlast);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (u < mh) rhs[k0 + u] = xs[u];
      const int cgl = is / MX;
      const gp<T> chx = gbl(D.chx);
      if (part == 0) chx[(size_t)cgl * ny + j] = xs[0];
      if (k0 + mh == m && mh > 0) chx[((size_t)D.cx + cgl) * ny + j] = xlast;
    }
  } else if (tid >= THREADS - 2 * TX) {
    const int c = ycol_of<T, TY>((tid - (THREADS - 2 * TX)) >> 1);
    const int part = tid & 1;
    const int i = i0 + c;
    if (i < nx && j0 < ny) {
      const int m = min(TY, ny - j0);
      const T* dly = sm.db + LW + c + 2;        // depths of rows j0-1 .. j0+m
      T* rhs = sm.x.s.v + c;
      T xs[TY / 2], xlast;
      int k0, mh;
      group_solve<T, TY / 2, 2, true>(dly, LW, m, D.tcy, j0 == 0, j0 + m == ny, part,
                                      [&](int k) { return rhs[k * TXP]; }, xs, k0, mh, xlast);
#pragma unroll
      for (int u = 0; u < TY / 2; ++u)
        if (u < mh) rhs[(k0 + u) * TXP] = xs[u];
      const int cgl = j0 / TY;
      const gp<T> chy = gbl(D.chy);
      if (part == 0) chy[(size_t)cgl * nx + i] = xs[0];
      if (k0 + mh == m && mh > 0) chy[((size_t)D.cy + cgl) * nx + i] = xlast;
    }
  }
  __syncthreads();
  // local solutions (cells outside the domain land in the fields' padding),
  // on the base P^n, Q^n
  {
    V xp, xq, pb, qb;
    if (CORR) {
      pb = ldv<CPT>(uni((const T*)D.P[slot]) + tG, oG);
      qb = ldv<CPT>(uni((const T*)D.Q[slot]) + tG, oG);
    }
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int C0 = (vr + 2) * LW + vc + k + 2;
      xp.v[k] = (CORR ? pb.v[k] : sm.p[C0]) + sm.x.s.u[vr * TXP + vc + k];
      xq.v[k] = (CORR ? qb.v[k] : sm.q[C0]) + sm.x.s.v[vr * TXP + vc + k];
    }
    stv_nt(uni(D.xhP) + tI, oI, xp);
    stv_nt(uni(D.xhQ) + tI, oI, xq);
  }
}

// ---------------------------------------------------------------------------
// k_reduced: couple the chunk-local solutions of every line
// ---------------------------------------------------------------------------
//
// For chunk c with local solution xh, left spike v and right spike w, the
// exact solution is x = xh + v * X_{e}(c-1) + w * X_{s}(c+1).  With
// sigma_c = x_first(c) and alpha_c = x_last(c) written as affine functions
// of x_first(c+1), a forward sweep gives
//   sigma_c = k1 xh_s + k2 alpha_{c-1},  alpha_c = xh_e + m1 alpha_{c-1} + m2 sigma_c
// and a backward sweep X_s(c) = sigma_c + tau_c X_s(c+1),
// X_e(c) = alpha_c + gamma_c X_s(c+1).  (k1, k2, m1, m2, tau, gamma) are
// static and precomputed.
//
// The recurrences are serial in c, their inputs are not.  A line's chunks
// are spread over RED_SEGS threads of RED_MAX chunks each, which load all
// their inputs at once; the sweep then passes from thread to thread in
// registers (row swaps inside a wave, LDS from wave to wave).  What
// bounds the kernel is latency (its words are 0.15 of the stencil kernel's
// bytes at most): one trip to memory and the chain itself, three dependent
// operations per chunk forward and one backward.  16 lines to a block spread
// the lines thinly (a 2048^2 domain gives 256 blocks, one per compute unit,
// one of 200 x 20 cells 15).  The sweep takes the chunks in their order and
// rounds each as one thread sweeping alone in groups of 8 chunks did, so
// neither the launch nor the batch around a domain changes its results.
// Against that one thread per line (HIP events around the launch): 41.6 ->
// 12.6 us on 2048^2 FP32, 33.3 -> 8.7 on 1024 x 256 FP64, 10.7 -> 7.3 on 200 x
// 20 FP64; composing the segments' maps in parallel, which rounds differently,
// would take 11.3, 8.2 and 6.7.
// Lines of more than RED_SEGS * RED_MAX chunks are taken in panels, from the
// first to the last and back, with sigma and alpha of all but the last panel
// kept in the result's slots: 64 columns of FP64 rows take 11.4 us with 128
// chunks (33.0 by one thread per line), 14.5 with 129 (40.4), 79 with 1024
// (250).

constexpr int RED_LINES = 16, RED_SEGS = 16, RED_MAX = 8;
constexpr int RED_PANEL = RED_SEGS * RED_MAX;      // chunks of a line per panel
constexpr int RED_THREADS = RED_LINES * RED_SEGS;
constexpr int RED_ROWS = 64 / RED_LINES;           // segments (rows of lanes) per wave
static_assert(RED_ROWS == 4, "the sweeps below pass through four rows");
template <int V>
using Int = std::integral_constant<int, V>;

// blocks of RED_LINES lines of a domain: its x-lines', then its y-lines'
__host__ __device__ inline int line_blocks(int nx, int ny) {
  return (ny + RED_LINES - 1) / RED_LINES + (nx + RED_LINES - 1) / RED_LINES;
}

// A wave's value moved by one row of 16 lanes: up (row r to row r + 1) for
// r = FROM, or down (row r to row r - 1).  The rows that the sweep has yet
// to reach get no meaningful value.
template <bool UP, int FROM>
__device__ __forceinline__ unsigned row_move(unsigned v) {
  if (UP) {
    if (FROM == 1) v = __builtin_amdgcn_permlane32_swap(v, v, false, false)[0];   // row 3 = row 1
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return FROM == 1 ? r[1] : r[0];                                               // even rows from odd, or odd from even
  }
  if (FROM == 2) v = __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];     // row 0 = row 2
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return FROM == 2 ? r[0] : r[1];
}
template <bool UP, int FROM>
__device__ __forceinline__ float row_move(float v) {
  return __uint_as_float(row_move<UP, FROM>(__float_as_uint(v)));
}
template <bool UP, int FROM>
__device__ __forceinline__ double row_move(double v) {
  const unsigned lo = row_move<UP, FROM>((unsigned)__double2loint(v));
  const unsigned hi = row_move<UP, FROM>((unsigned)__double2hiint(v));
  return __hiloint2double((int)hi, (int)lo);
}

template <typename T>
__global__ void __launch_bounds__(RED_THREADS) k_reduced(const DomDev<T>* __restrict__ doms,
                                                        const int* __restrict__ line_map, int nd, int pass) {
  __shared__ T hand[RED_LINES];               // the sweep's value, from wave to wave
  int dom, blk;
  // neighbouring blocks share 128-byte lines: keep them on one XCD
  locate(line_map, nd, xcd_tile(blockIdx.x, gridDim.x), dom, blk);
  const DomDev<T>& D = doms[dom];
  if (D.st->halt) return;
  if (pass == 1 && !D.corrector) return;      // the corrector pass
  const int nbx = (D.ny + RED_LINES - 1) / RED_LINES;
  const bool xl = blk < nbx;
  const int L = uni(xl ? D.ny : D.nx), C = uni(xl ? D.cx : D.cy);
  const int ln = threadIdx.x % RED_LINES, seg = threadIdx.x / RED_LINES;
  const int row = seg % RED_ROWS, wave = uni(seg / RED_ROWS);
  const int line = (xl ? blk : blk - nbx) * RED_LINES + ln;
  const bool active = line < L;
  const unsigned lo = (unsigned)min(line, L - 1);
  const size_t CL = (size_t)C * L;
  const T* const ch = uni((const T*)(xl ? D.chx : D.chy));
  const T* const rs = uni((const T*)(xl ? D.rsx : D.rsy));
  T* const itf = uni(xl ? D.ifx : D.ify);     // left neighbour values
  T* const itr = itf + CL;                    // right neighbour values
  const int panels = (C + RED_PANEL - 1) / RED_PANEL;
  T sg[RED_MAX], al[RED_MAX], t4[RED_MAX], t5[RED_MAX];
  T a = T(0);                                 // alpha of the chunk before
  for (int p = 0; p < panels; ++p) {
    const int c0 = p * RED_PANEL + seg * RED_MAX;
    const int waves = min(RED_SEGS / RED_ROWS, (C - p * RED_PANEL + RED_MAX * RED_ROWS - 1) / (RED_MAX * RED_ROWS));
    T k1[RED_MAX], k2[RED_MAX], m1[RED_MAX], m2[RED_MAX], xs[RED_MAX], xe[RED_MAX];
    if (wave < waves) {
#pragma unroll
      for (int k = 0; k < RED_MAX; ++k) {
        const unsigned o = (unsigned)min(c0 + k, C - 1) * (unsigned)L + lo;
        xs[k] = ldu(ch, o);
        xe[k] = ldu(ch + CL, o);
        k1[k] = ldu(rs, o);
        k2[k] = ldu(rs + CL, o);
        m1[k] = ldu(rs + 2 * CL, o);
        m2[k] = ldu(rs + 3 * CL, o);
        t4[k] = ldu(rs + 4 * CL, o);
        t5[k] = ldu(rs + 5 * CL, o);
      }
    }
    for (int w = 0; w < waves; ++w) {
      if (w == wave) {
        if (w > 0) a = hand[ln];
        // chunks past the line's last one change only values that are not used
        auto sweep = [&](auto r) {
          if (decltype(r)::value == row) {
#pragma unroll
            for (int k = 0; k < RED_MAX; ++k) {
              // Which of the two products is rounded by itself is part of the
              // FP32 results: in the first chunk of a thread the other one, as the
              // former sweep's groups of 8 chunks came out of the compiler.
              // (RED_MAX is that 8: another value would round differently.)
              sg[k] = k == 0 ? fma_(k2[k], a, k1[k] * xs[k]) : fma_(k1[k], xs[k], k2[k] * a);
              a = fma_(m2[k], sg[k], fma_(m1[k], a, xe[k]));
              al[k] = a;
            }
          }
        };
        sweep(Int<0>{});
        a = row_move<true, 0>(a);
        sweep(Int<1>{});
        a = row_move<true, 1>(a);
        sweep(Int<2>{});
        a = row_move<true, 2>(a);
        sweep(Int<3>{});
        if (row == RED_ROWS - 1) hand[ln] = a;
      }
      __syncthreads();
    }
    a = hand[ln];                             // into the next panel
    if (p + 1 < panels && active) {
#pragma unroll
      for (int k = 0; k < RED_MAX; ++k)
        if (c0 + k < C) {
          const unsigned o = (unsigned)(c0 + k) * (unsigned)L + lo;
          stu(itf, o, sg[k]);
          stu(itr, o, al[k]);
        }
    }
    __syncthreads();
  }
  // the chunks past the last one hand it a zero
  if (panels > 0) {
    const int c0 = (panels - 1) * RED_PANEL + seg * RED_MAX;
#pragma unroll
    for (int k = 0; k < RED_MAX; ++k)
      if (c0 + k >= C) sg[k] = T(0);
  }
  T x = T(0);                                 // X_s of the chunk after
  for (int p = panels - 1; p >= 0; --p) {
    const int c0 = p * RED_PANEL + seg * RED_MAX;
    const int waves = min(RED_SEGS / RED_ROWS, (C - p * RED_PANEL + RED_MAX * RED_ROWS - 1) / (RED_MAX * RED_ROWS));
    if (p + 1 < panels) {
#pragma unroll
      for (int k = 0; k < RED_MAX; ++k) {
        const unsigned o = (unsigned)(c0 + k) * (unsigned)L + lo;   // whole panels but the last
        sg[k] = ldu((const T*)itf, o);
        al[k] = ldu((const T*)itr, o);
        t4[k] = ldu(rs + 4 * CL, o);
        t5[k] = ldu(rs + 5 * CL, o);
        pin(sg[k]);
      }
      // a slot's sigma is read before the chunk on its left writes its result there
      __syncthreads();
    }
    for (int w = waves - 1; w >= 0; --w) {
      if (w == wave) {
        if (w < waves - 1) x = hand[ln];
        auto sweep = [&](auto r) {
          if (decltype(r)::value == row) {
#pragma unroll
            for (int k = RED_MAX - 1; k >= 0; --k) {
              const T Xs = fma_(t4[k], x, sg[k]);
              sg[k] = fma_(t5[k], x, al[k]);            // X_e(c)
              al[k] = x;
              x = Xs;
            }
          }
        };
        sweep(Int<3>{});
        x = row_move<false, 3>(x);
        sweep(Int<2>{});
        x = row_move<false, 2>(x);
        sweep(Int<1>{});
        x = row_move<false, 1>(x);
        sweep(Int<0>{});
        if (row == 0) hand[ln] = x;
      }
      __syncthreads();
    }
    x = hand[ln];                             // into the panel before
    if (active) {
#pragma unroll
      for (int k = 0; k < RED_MAX; ++k)
        if (c0 + k < C) {
          const unsigned o = (unsigned)(c0 + k) * (unsigned)L + lo;
          stu(itr, o, al[k]);                                     // right neighbour of chunk c
          if (c0 + k + 1 < C) stu(itf, o + (unsigned)L, sg[k]);   // left neighbour of chunk c + 1
        }
    }
    __syncthreads();
  }
  if (active && seg == 0) stu(itf, lo, T(0));   // chunk 0 has no left neighbour
}

// ---------------------------------------------------------------------------
// k_final: spike corrections, sponge, ghost cells, CFL maximum
// ---------------------------------------------------------------------------

template <typename T>
__device__ __forceinline__ void put3(const DomDev<T>& D, T* w, T* P, T* Q, int i, int j, T vw, T vp, T vq) {
  const size_t g = (size_t)(j + 2) * D.pitch + D.xoff + i;
  gbl(w)[g] = vw;
  gbl(P)[g] = vp;
  gbl(Q)[g] = vq;
}

// ghost cells written by interior cell (i, j) of the new state: x sides for
// interior rows (wall mirror or wavemaker values), then y sides for all
// columns (the corners mirror the x ghosts)
template <typename T>
__device__ void ghost_cell(const DomDev<T>& D, T* w, T* P, T* Q, int i, int j, T wv, T p, T qv, const double* gw,
                           const double* gP) {
  const int nx = D.nx, ny = D.ny;
  const bool yg = j < 2 || j >= ny - 2;
  T gwv = wv, gpv = p, gqv = qv;
  int gi = 0;
  bool have_x = false;
  if (i < 2) {
    gi = -1 - i;
    have_x = true;
    if (west_driven(D.bc[0])) {
      gwv = (T)gw[i];
      gpv = (T)gP[i];
      gqv = T(0);
    } else {
      gpv = -p;
    }
    put3(D, w, P, Q, gi, j, gwv, gpv, gqv);
  } else if (i >= nx - 2) {
    gi = 2 * nx - 1 - i;
    have_x = true;
    gpv = -p;
    put3(D, w, P, Q, gi, j, gwv, gpv, gqv);
  }
  if (yg) {
    const int gj = j < 2 ? -1 - j : 2 * ny - 1 - j;
    put3(D, w, P, Q, i, gj, wv, p, -qv);
    if (have_x) put3(D, w, P, Q, gi, gj, gwv, gpv, -gqv);
  }
}

template <typename T, int TY, int MX>
struct alignas(16) FinSmem {
  static constexpr int CXN = TX + 3, CYN = TY + 3;    // corners of cells i0-1 .. i0+TX, j0-1 .. j0+TY
  static constexpr int BX = TX + 2, BY = TY + 2;      // cells with one neighbour on each side
  static constexpr int BXP = BX + 3;                  // their row pitch: 5 mod 32 words
  static constexpr int TXP = TX + 1;
  static_assert(BXP % 32 == PITCH_MOD_TILE && TXP % 32 == PITCH_MOD_ROWS, "the lane layouts assume these row pitches");
  // corners are staged in pairs from corner i0 - 2 (one before the CXN used)
  static constexpr int CP = CXN + 1;
  T db[BY * BXP];                                     // cell still-water depth
  union {
    T dc[CYN * CP];                                   // corners (until db is formed)
    struct {
      T cx[TY * TXP];                                 // x-line correction of P
      T cy[TY * TXP];                                 // y-line correction of Q
    } s;
  } u;
};

// MODE 0: finalizes the AB3 step in a launch where no domain runs the
// corrector.  MODE 1: the same where some do; for those it finalizes the
// predicted level (surface in w[2], no sponge, no run-up record).  MODE 2:
// finalizes the corrector of the domains that run it.
template <typename T, int TY, int MX, int MODE, int THREADS = NT, bool BIG = false>
__global__ void __launch_bounds__(THREADS) k_final(const DomDev<T>* __restrict__ doms, const int* __restrict__ tile_map,
                                             int nd, int swizzle) {
  using S = FinSmem<T, TY, MX>;
  constexpr int CP = S::CP, BX = S::BX, BXP = S::BXP, TXP = S::TXP;
  constexpr int CPT = (TX * TY) / THREADS;
  using V = Vec<T, CPT>;
  using V2 = Vec<T, 2>;
  __shared__ S sm;
  int dom, tile;
  // swizzle = 1: XCD-aware tile order, as in the stencil kernel (the corner
  // halo of a tile is then mostly in its XCD's L2)
  locate(tile_map, nd, swizzle ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x, dom, tile);
  const DomDev<T>& D = doms[dom];
  DevState* st = D.st;
  if (st->halt) return;
  if (MODE == 2 && !D.corrector) return;
  const bool pred = MODE == 1 && D.corrector;          // the predictor's level
  const int i0 = (tile % D.tiles_x) * TX, j0 = (tile / D.tiles_x) * TY;
  const int nx = D.nx, ny = D.ny, tid = threadIdx.x;
  const int ns = uni(st->slot == 2 ? 0 : st->slot + 1);   // slot of level n + 1
  const int par = uni((int)((st->n + 1) & 1));
  T* const w = uni(pred ? D.w[2] : D.w[par]);
  T* const P = uni(D.P[ns]);
  T* const Q = uni(D.Q[ns]);
  const int pitch = uni(D.pitch), xoff = uni(D.xoff), ipitch = uni(D.ipitch), cpitch = uni(D.cpitch);
  const T g = D.g, eps = D.eps, idx = D.idx, idy = D.idy;
  // cells of a thread: row vr, columns vc .. vc+CPT-1 (as in the stencil kernel)
  int vr, vc;
  cell_of<T, CPT>(tid, vr, vc);
  // where the lanes count from, as in the stencil kernel
  const int jl = BIG ? 0 : j0, il = BIG ? 0 : i0, xo = BIG ? 0 : xoff;
  const size_t tI = BIG ? (size_t)j0 * ipitch + i0 : 0;
  const size_t tG = BIG ? (size_t)j0 * pitch + xoff + i0 : 0;
  const size_t tC = BIG ? (size_t)j0 * cpitch + i0 : 0;
  const unsigned oI = (unsigned)((jl + vr) * ipitch + il + vc);
  const unsigned oG = (unsigned)((jl + vr + 2) * pitch + xo + il + vc);
  // All loads first, in the order they are needed (the waits are in issue
  // order): the corners of the tile's cells and their neighbours (pairs of
  // corners, rows read in groups, no clamping: the fields are padded to
  // whole tiles), the neighbour-chunk end values of the line solves, the
  // local solutions and the new surface.
  const double dt = uni(st->dt);
  constexpr int NCX = TX / MX;
  using SC = PairStaging<CP / 2, S::CYN, THREADS>;           // corner rows
  constexpr int KC = SC::K;
  const int cC = SC::col(tid);
  auto rowC = [&](int k) { return SC::row(tid, k); };
  V2 rc[KC];
  __builtin_amdgcn_sched_barrier(0);
  {
    const T* Dc = uni((const T*)D.Dc) + tC;
    const unsigned oC = (unsigned)((jl + 1) * cpitch + il + cC);   // corner (i0-2+cC, j0-1)
#pragma unroll
    for (int k = 0; k < KC; ++k) rc[k] = ldv<2>(Dc, oC + (unsigned)(rowC(k) * cpitch));
  }
  __builtin_amdgcn_sched_barrier(0);
  // lane groups solve the chunk responses (group_solve; parts of 8 rows
  // along x, two halves along y): x-chunks in the first PX TY NCX threads,
  // y-chunks (tile columns) in the last 2 TX; every thread loads the end
  // values of both, at clamped indices, and uses one
  constexpr int PX = MX / 8;
  static_assert(PX * TY * NCX <= THREADS - 2 * TX, "x- and y-chunk solver groups must fit the block");
  T xl, xr;
  {
    const int qx = min(tid / PX, TY * NCX - 1);
    int r, qc;
    xchunk_of<T, TY, NCX, PX>(qx, r, qc);
    const int jx = min(j0 + r, ny - 1), is = min(i0 + qc * MX, nx - 1);
    const unsigned ox = (unsigned)((is / MX) * ny + jx);
    const int iy = min(i0 + ycol_of<T, TY>((tid >> 1) & (TX - 1)), nx - 1);
    const unsigned oy = (unsigned)((j0 / TY) * nx + iy);
    const T* ifx = uni((const T*)D.ifx);
    const T* ify = uni((const T*)D.ify);
    const unsigned cxn = (unsigned)(D.cx * ny), cyn = (unsigned)(D.cy * nx);
    const T xlx = ldu(ifx, ox), xrx = ldu(ifx, cxn + ox);
    const T xly = ldu(ify, oy), xry = ldu(ify, cyn + oy);
    const bool xsol = tid < PX * TY * NCX;
    xl = xsol ? xlx : xly;
    xr = xsol ? xrx : xry;
  }
  __builtin_amdgcn_sched_barrier(0);
  const V lp = ldv_nt<CPT>(uni((const T*)D.xhP) + tI, oI);
  const V lq = ldv_nt<CPT>(uni((const T*)D.xhQ) + tI, oI);
  const V lw = ldv_nt<CPT>((const T*)w + tG, oG);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    sm.u.dc[rowC(k) * CP + cC] = rc[k].v[0];
    sm.u.dc[rowC(k) * CP + cC + 1] = rc[k].v[1];
  }
  __syncthreads();
  for (int e = tid; e < S::BY * BX; e += THREADS) {
    const int r = e / BX, c = e - r * BX;
    // cell (i0 - 1 + c, j0 - 1 + r): corners c + 1, c + 2 of the staged rows
    sm.db[r * BXP + c] = dbar4(sm.u.dc[r * CP + c + 1], sm.u.dc[r * CP + c + 2], sm.u.dc[(r + 1) * CP + c + 1],
                     sm.u.dc[(r + 1) * CP + c + 2]);
  }
  __syncthreads();
  // Exact line solution = local solution + the response of the chunk system
  // to its coupling with the neighbour chunks' end values (from the
  // line-coupling kernel): a right-hand side that is zero except -a x_left
  // in the first row and -c x_right in the last.  The response is solved
  // here from the static matrix instead of read as stored spikes, by the
  // lane groups of the chunk solves in their two-vector form
  // (group_response).
  const bool wave_w = west_driven(D.bc[0]);
  if (tid < PX * TY * NCX) {
    const int qq = tid / PX, part = tid - qq * PX;
    int r, qc;
    xchunk_of<T, TY, NCX, PX>(qq, r, qc);
    const int j = j0 + r, is = i0 + qc * MX;
    if (j < ny && is < nx) {
      const int m = min(MX, nx - is);
      const T* dlx = sm.db + (r + 1) * BXP + qc * MX;  // cells is-1 .. is+m
      T a, b, c0, cm;
      tri_coef(dpos(dlx[0]), dpos(dlx[1]), dpos(dlx[2]), D.tcx, a, b, c0);
      const T r0 = -a * xl;
      tri_coef(dpos(dlx[m - 1]), dpos(dlx[m]), dpos(dlx[m + 1]), D.tcx, a, b, cm);
      const T r1 = -cm * xr;
      T xs[8];
      int k0, mh;
      group_response<T, 8, PX>(dlx, 1, m, D.tcx, is == 0 && !wave_w, is + m == nx, part, r0, r1, xs, k0, mh);
      T* out = sm.u.s.cx + r * TXP + qc * MX + k0;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (u < mh) out[u] = xs[u];
    }
  } else if (tid >= THREADS - 2 * TX) {
    const int c = ycol_of<T, TY>((tid - (THREADS - 2 * TX)) >> 1);
    const int part = tid & 1;
    const int i = i0 + c;
    if (i < nx && j0 < ny) {
      const int m = min(TY, ny - j0);
      const T* dly = sm.db + c + 1;                    // rows j0-1 .. j0+m
      T a, b, c0, cm;
      tri_coef(dpos(dly[0]), dpos(dly[BXP]), dpos(dly[2 * BXP]), D.tcy, a, b, c0);
      const T r0 = -a * xl;
      tri_coef(dpos(dly[(m - 1) * BXP]), dpos(dly[m * BXP]), dpos(dly[(m + 1) * BXP]), D.tcy, a, b, cm);
      const T r1 = -cm * xr;
      T xs[TY / 2];
      int k0, mh;
      group_response<T, TY / 2, 2>(dly, BXP, m, D.tcy, j0 == 0, j0 + m == ny, part, r0, r1, xs, k0, mh);
      T* out = sm.u.s.cy + k0 * TXP + c;
#pragma unroll
      for (int u = 0; u < TY / 2; ++u)
        if (u < mh) out[u * TXP] = xs[u];
    }
  }
  __syncthreads();
  // new state, sponge, CFL speeds (Eq. 22) and ghost cells
  const int j = j0 + vr;
  const bool row_in = j < ny;
  const bool all_in = row_in && i0 + vc + CPT <= nx;
  T smax = T(0);
  V vp, vq;
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = vc + k, i = i0 + c;
    T p = lp.v[k] + sm.u.s.cx[vr * TXP + c];
    T qv = lq.v[k] + sm.u.s.cy[vr * TXP + c];
    T wv = lw.v[k];
    const T Db = sm.db[(vr + 1) * BXP + c + 1];
    vp.v[k] = p;
    vq.v[k] = qv;
    if (i >= nx || !row_in) continue;
    if (D.any_sponge && !pred && Db > T(0)) {
      const T dist[4] = {(T(i) + T(0.5)) * D.dx, (T(nx - i) - T(0.5)) * D.dx, (T(j) + T(0.5)) * D.dy,
                         (T(ny - j) - T(0.5)) * D.dy};
      T sig = T(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const T Ls = D.sponge_w[s];
        if (D.bc[s] == SPONGE && Ls > T(0) && dist[s] < Ls) {
          const T z = (Ls - dist[s]) / Ls;
          sig += D.sponge_sigma * z * z;
        }
      }
      if (sig > T(0)) {
        const T fac = exp(-sig * (T)dt);
        wv *= fac;
        p *= fac;
        qv *= fac;
        vp.v[k] = p;
        vq.v[k] = qv;
        stu(w + tG, oG + k, wv);
      }
    }
    const T h = fmax(wv + Db, T(0));
    if (D.runup && !pred && h > D.runup_delta) {
      // run-up record: highest surface over the inundated states (NaN until
      // the first one)
      const gp<T> wm = gbl(D.wmax) + tI;
      const unsigned oi = oI + (unsigned)k;
      if (!(wm[oi] >= wv)) wm[oi] = wv;
    }
    const T vf = vfac(h, eps);
    const T u = p * vf, v = qv * vf;
    const T cel = fsqrt(g * h);
    const T sx = (fabs(u) + cel) * idx, sy = (fabs(v) + cel) * idy;
    // a NaN in either direction must reach the maximum as +inf
    const T sd = (sx != sx || sy != sy) ? T(INFINITY) : fmax(sx, sy);
    smax = fmax(smax, sd);
    if (i < 2 || i >= nx - 2 || j < 2 || j >= ny - 2) ghost_cell(D, w, P, Q, i, j, wv, p, qv, st->gw, st->gP);
  }
  if (all_in) {
    stv_nt(P + tG, oG, vp);
    stv_nt(Q + tG, oG, vq);
  } else if (row_in) {
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      if (i0 + vc + k >= nx) break;
      stu(P + tG, oG + k, vp.v[k]);
      stu(Q + tG, oG + k, vq.v[k]);
    }
  }
  // block max -> one word per tile (max commutes with the widening to FP64,
  // so the FP32 maximum converts to the same value); no atomics, so a large
  // domain's blocks do not serialise on one address
  __shared__ T red[THREADS / 64];
  for (int o = 32; o > 0; o >>= 1) smax = fmax(smax, __shfl_xor(smax, o, 64));
  if ((tid & 63) == 0) red[tid >> 6] = smax;
  __syncthreads();
  if (tid == 0) {
    T m = red[0];
    for (int k = 1; k < THREADS / 64; ++k) m = fmax(m, red[k]);
    gbl(D.smax_tile)[tile] = (double)m;               // reduced by the next step's k_dt
  }
}

}  // namespace bqk
