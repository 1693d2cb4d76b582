// Device-side numerics of the ideal-MHD step (gfx950).
//
// Everything here is a __device__ inline function templated on the face
// scalar R (double, or float in the mixed-precision path) so that the
// reconstruction / Riemann / EMF chain is instantiated twice from one source.
// Primitive recovery and all accumulation stay in double.
//
// Paper: arXiv 2511.20337 (gPLUTO). Sec. 2.1 Eqs. (mhd), (Energy): state,
// flux and EOS; Sec. 2.2: primitive inversion, reconstruction (Eq.
// reconstruct), Riemann flux, constrained transport; Secs. 4.1/4.2 cite the
// HLLD solver of Miyoshi & Kusano (2005), written out below.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Every floating-point operation is evaluated as written: no automatic fusion
// of a multiply and an add into an FMA (explicit __builtin_fma calls stay).
// The adjoint re-evaluates reconstruction and the Riemann solver in other
// kernels and in dual numbers; with contraction left to the compiler, the same
// source could round differently there than in the forward kernels, and at
// near-ties (a limiter at a local extremum, min/max of equal wave speeds,
// the sign of the contact speed) take the other branch. This pragma applies
// to every function defined after it in the translation unit.
#pragma clang fp contract(off)

namespace mhd {

enum : int { F_RHO = 0, F_MX = 1, F_MY = 2, F_MZ = 3, F_EN = 4, F_BX = 5, F_BY = 6, F_BZ = 7 };

// Workgroup order of the 3D kernels that take cells in storage order, of the CT
// kernel and of the adjoint's gather kernels: the hardware deals workgroups
// round-robin to the 8 XCDs, each with its own L2. Within every full group of
// 512 workgroups, XCD x is given the 64 consecutive ones x*64 .. x*64+63, so
// that neighbouring rows (the stencil's reach along y) are mostly read through
// the same L2, while all XCDs still advance together through the domain and
// share the Infinity Cache. A permutation of 0 .. nb-1; a last partial group
// keeps its order. (Measured slower for the z-marching face kernel, whose
// neighbouring columns share the Infinity Cache better round-robin.)
__device__ __forceinline__ unsigned xcd_grouped(unsigned b, unsigned nb) {
  const unsigned grp = b / 512u;
  if ((grp + 1u) * 512u > nb) return b;
  const unsigned w = b % 512u;
  return grp * 512u + (w % 8u) * 64u + w / 8u;
}

// Per-face record slots (one array of N values per slot, per direction):
// fluxes of the cell-averaged fields, then the quantities the edge EMF needs.
// With the UCT-HLLD average, S_AP holds its weight om, S_AM its diffusion
// coefficient d^L and S_DR d^R, and S_V1/S_V2 the om-weighted velocities.
enum : int {
  S_RHO = 0, S_MX = 1, S_MY = 2, S_MZ = 3, S_EN = 4, S_BZ = 5,  // S_BZ: 2D only
  S_AP = 6, S_AM = 7, S_V1 = 8, S_V2 = 9, S_DR = 10, NSLOT = 11
};

struct Geom {
  int nx, ny, nz;
  int64_t n;            // cells
  double dx, dy, dz;    // spacings
  double gamma;
};

// FP64 reciprocal, quotient and square root from the hardware estimates
// (v_rcp_f64 / v_rsq_f64, about 5e-8 relative), refined by a third-order step
// (reciprocal; what is left of the estimate's error is 1e-22, below its last
// rounding) or a Newton step and a residual correction: on 2^20 random
// operands the quotient and the square root reproduce the IEEE result bit for
// bit, at well under the instruction count of the IEEE sequences. Operands:
// finite, nonzero divisors and non-negative radicands in the normal range.
__device__ __forceinline__ double rcp_r(double b) {
  const double r = __builtin_amdgcn_rcp(b);
  const double e = __builtin_fma(-b, r, 1.0);
  return __builtin_fma(r, __builtin_fma(e, e, e), r);  // r (1 + e + e^2)
}
// Quotient a/b; r receives the refined reciprocal of b it was formed with.
__device__ __forceinline__ double div_r_rcp(double a, double b, double& r) {
  r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}
__device__ __forceinline__ double div_r(double a, double b) {
  double r;
  return div_r_rcp(a, b, r);
}
// Square root of x >= 0; h receives about 1/(2 sqrt(x)) (one Newton step).
__device__ __forceinline__ double sqrt_r_half(double x, double& h) {
  const double y = __builtin_amdgcn_rsq(x);
  double s = x * y;
  h = 0.5 * y;
  const double t = __builtin_fma(-s, h, 0.5);
  s = __builtin_fma(s, t, s);
  h = __builtin_fma(h, t, h);
  const double r = __builtin_fma(__builtin_fma(-s, s, x), h, s);
  return x > 0.0 ? r : 0.0;  // the estimate is infinite at 0
}
__device__ __forceinline__ double sqrt_r(double x) {
  double h;
  return sqrt_r_half(x, h);
}
// a * b + c with one rounding. With contraction off, these are the only fused
// multiply-adds; the adjoint's dual numbers overload fma_r with the same value.
__device__ __forceinline__ double fma_r(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}
__device__ __forceinline__ float fma_r(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}
// FP32 (mixed precision): the one-ulp hardware reciprocal and square root.
__device__ __forceinline__ float rcp_r(float b) {
  const float r = __builtin_amdgcn_rcpf(b);
  return __builtin_fmaf(r, __builtin_fmaf(-b, r, 1.0f), r);
}
__device__ __forceinline__ float div_r(float a, float b) {
  const float r = __builtin_amdgcn_rcpf(b);
  const float q = a * r;
  return __builtin_fmaf(__builtin_fmaf(-b, q, a), r, q);
}
__device__ __forceinline__ float sqrt_r(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double abs_r(double x) { return __builtin_fabs(x); }
__device__ __forceinline__ float abs_r(float x) { return __builtin_fabsf(x); }
template <class R> __device__ __forceinline__ R max_r(R a, R b) { return (b > a) ? b : a; }
// max_r(0, x) (0 for a NaN too) in one instruction instead of three
__device__ __forceinline__ double max0_r(double x) { return __builtin_fmax(x, 0.0); }
__device__ __forceinline__ float max0_r(float x) { return __builtin_fmaxf(x, 0.0f); }
template <class R> __device__ __forceinline__ R min_r(R a, R b) { return (b < a) ? b : a; }

// Limited slope of piecewise-linear reconstruction, zero at extrema: minmod
// (LIM 0), or half the harmonic van Leer slope (LIM 1; the half comes free: the
// slope 2 dm dp / (dm + dp) times 1/2, bit for bit, without its two products by
// two). plm_up / plm_lo: the values x + slope/2 and x - slope/2.
template <int LIM, class R>
__device__ __forceinline__ R plm_slope(R dm, R dp) {
  const R pr = dm * dp;
  if (LIM == 0) return (pr <= R(0)) ? R(0) : ((abs_r(dm) <= abs_r(dp)) ? dm : dp);
  const R q = div_r(pr, dm + dp);  // unused (maybe not finite) at extrema
  return (pr <= R(0)) ? R(0) : q;
}
template <int LIM, class R>
__device__ __forceinline__ R plm_up(R slope, R x) {
  return LIM == 0 ? fma_r(R(0.5), slope, x) : x + slope;
}
template <int LIM, class R>
__device__ __forceinline__ R plm_lo(R slope, R x) {
  return LIM == 0 ? fma_r(R(-0.5), slope, x) : x - slope;
}
// Left and right value at a face from the four cells about it.
template <int LIM, class R>
__device__ __forceinline__ void plm_pair(R a, R b, R c, R d, R& l, R& r) {
  l = plm_up<LIM, R>(plm_slope<LIM, R>(b - a, c - b), b);
  r = plm_lo<LIM, R>(plm_slope<LIM, R>(c - b, d - c), c);
}

// Fifth-order WENO-Z reconstruction (Borges et al. 2008, one of the operators
// R+- cited with Eq. (reconstruct)), FP64: the value at the upper interface of
// the middle cell of v0..v4 (cells i-2..i+2), a convex combination of the three
// third-order candidate values with Z weights d_k (1 + tau5 / (beta_k + eps)),
// Jiang-Shu smoothness indicators beta_k, tau5 = |beta0 - beta2|, ideal
// weights (1, 6, 3)/10, eps = 1e-40. The lower interface value is the same
// function of the cells in reverse order. The weights are formed over a common
// denominator, which moves the result by a few ulps from the textbook order of
// operations, and so do the fused multiply-adds.
__device__ __forceinline__ double wenoz_upper(double v0, double v1, double v2, double v3,
                                              double v4) {
  // six times the three candidate values (fused multiply-adds throughout:
  // this reconstruction has no adjoint whose roundings must match)
  const double q0 = __builtin_fma(2.0, v0, __builtin_fma(-7.0, v1, 11.0 * v2));
  const double q1 = __builtin_fma(5.0, v2, __builtin_fma(2.0, v3, -v1));
  const double q2 = __builtin_fma(2.0, v2, __builtin_fma(5.0, v3, -v4));
  const double c1 = 13.0 / 12.0, c2 = 1.0 / 4.0;
  const double a0 = __builtin_fma(-2.0, v1, v0 + v2);
  const double b0 = __builtin_fma(-4.0, v1, __builtin_fma(3.0, v2, v0));
  const double a1 = __builtin_fma(-2.0, v2, v1 + v3), b1 = v1 - v3;
  const double a2 = __builtin_fma(-2.0, v3, v2 + v4);
  const double b2 = __builtin_fma(3.0, v2, __builtin_fma(-4.0, v3, v4));
  const double eps = 1e-40;
  const double beta0 = __builtin_fma(c1 * a0, a0, __builtin_fma(c2 * b0, b0, eps));
  const double beta1 = __builtin_fma(c1 * a1, a1, __builtin_fma(c2 * b1, b1, eps));
  const double beta2 = __builtin_fma(c1 * a2, a2, __builtin_fma(c2 * b2, b2, eps));
  const double tau5 = __builtin_fabs(beta0 - beta2);
  // d_k (1 + tau5 / beta_k) times beta0 beta1 beta2 (> 0, which the
  // normalisation cancels), so that one division remains instead of seven;
  // beta_k >= eps keeps the products normal, and they stay finite while the
  // differences of the five values are below about 1e50
  const double al0 = 0.1 * (beta0 + tau5) * (beta1 * beta2);
  const double al1 = 0.6 * (beta1 + tau5) * (beta0 * beta2);
  const double al2 = 0.3 * (beta2 + tau5) * (beta0 * beta1);
  return div_r(__builtin_fma(al0, q0, __builtin_fma(al1, q1, al2 * q2)), 6.0 * (al0 + al1 + al2));
}

// The values at the lower and the upper interface of the middle cell: the two
// share the smoothness indicators (in reverse order), their products and the
// middle weight. Equal to two wenoz_upper up to rounding, not bit for bit: a value
// that is formed at two places takes the same function at both.
__device__ __forceinline__ void wenoz_both(double v0, double v1, double v2, double v3, double v4,
                                           double& lo, double& up) {
  const double c1 = 13.0 / 12.0, c2 = 1.0 / 4.0, eps = 1e-40;
  const double a0 = __builtin_fma(-2.0, v1, v0 + v2), a1 = __builtin_fma(-2.0, v2, v1 + v3);
  const double a2 = __builtin_fma(-2.0, v3, v2 + v4), b1 = v1 - v3;
  const double b0 = __builtin_fma(-4.0, v1, __builtin_fma(3.0, v2, v0));
  const double b2 = __builtin_fma(3.0, v2, __builtin_fma(-4.0, v3, v4));
  const double e0 = __builtin_fma(c1 * a0, a0, __builtin_fma(c2 * b0, b0, eps));
  const double e1 = __builtin_fma(c1 * a1, a1, __builtin_fma(c2 * b1, b1, eps));
  const double e2 = __builtin_fma(c1 * a2, a2, __builtin_fma(c2 * b2, b2, eps));
  const double tau5 = __builtin_fabs(e0 - e2);
  const double w0 = (e0 + tau5) * (e1 * e2), w2 = (e2 + tau5) * (e0 * e1);
  const double al1 = 0.6 * (e1 + tau5) * (e0 * e2);
  {
    const double al0 = 0.1 * w0, al2 = 0.3 * w2;
    const double q0 = __builtin_fma(2.0, v0, __builtin_fma(-7.0, v1, 11.0 * v2));
    const double q1 = __builtin_fma(5.0, v2, __builtin_fma(2.0, v3, -v1));
    const double q2 = __builtin_fma(2.0, v2, __builtin_fma(5.0, v3, -v4));
    up = div_r(__builtin_fma(al0, q0, __builtin_fma(al1, q1, al2 * q2)), 6.0 * (al0 + al1 + al2));
  }
  {
    const double al0 = 0.1 * w2, al2 = 0.3 * w0;
    const double q0 = __builtin_fma(2.0, v4, __builtin_fma(-7.0, v3, 11.0 * v2));
    const double q1 = __builtin_fma(5.0, v2, __builtin_fma(2.0, v1, -v3));
    const double q2 = __builtin_fma(2.0, v2, __builtin_fma(5.0, v1, -v0));
    lo = div_r(__builtin_fma(al0, q0, __builtin_fma(al1, q1, al2 * q2)), 6.0 * (al0 + al1 + al2));
  }
}

// Face-frame primitive state: (rho, u_n, v_t1, v_t2, B_t1, B_t2, p).
template <class R> struct FState { R w[7]; };

template <class R> struct RiemannOut {
  R f[7];        // flux of (rho, m_n, m_t1, m_t2, B_t1, B_t2, E)
  R ap, am;      // max(0, S_R), max(0, -S_L)
  R v1, v2;      // HLL-weighted transverse velocities (EM 1: om-weighted)
  R om, dl, dr;  // EM 1: UCT-HLLD weight of the left state, diffusion coefficients
};

// Fast magnetosonic speed along the normal, and its square.
template <class R>
__device__ __forceinline__ R cfast2(R g, R rho, R p, R bn, R b1, R b2) {
  const R gp = g * p;
  const R bn2 = bn * bn;
  const R bb = fma_r(b2, b2, fma_r(b1, b1, bn2));
  const R a = gp + bb;
  const R disc = max0_r(fma_r(a, a, -(R(4) * gp) * bn2));
  return div_r(a + sqrt_r(disc), R(2) * rho);
}
template <class R>
__device__ __forceinline__ R cfast(R g, R rho, R p, R bn, R b1, R b2) {
  return sqrt_r(cfast2(g, rho, p, bn, b1, b2));
}

// Conserved vector, normal flux and total pressure of a face-frame state.
template <class R>
__device__ __forceinline__ void phys(R igm1, const R* w, R bn, R* u, R* f, R& pt) {
  const R rho = w[0], vn = w[1], v1 = w[2], v2 = w[3], b1 = w[4], b2 = w[5], p = w[6];
  const R bb = fma_r(b2, b2, fma_r(b1, b1, bn * bn));
  pt = fma_r(R(0.5), bb, p);
  const R v2s = fma_r(v2, v2, fma_r(v1, v1, vn * vn));
  const R en = fma_r(R(0.5), bb, fma_r(R(0.5) * rho, v2s, p * igm1));
  const R mn = rho * vn;
  u[0] = rho; u[1] = mn; u[2] = rho * v1; u[3] = rho * v2; u[4] = b1; u[5] = b2; u[6] = en;
  const R vb = fma_r(v2, b2, fma_r(v1, b1, vn * bn));
  f[0] = mn;
  f[1] = fma_r(mn, vn, fma_r(-bn, bn, pt));
  f[2] = fma_r(mn, v1, -bn * b1);
  f[3] = fma_r(mn, v2, -bn * b2);
  f[4] = fma_r(vn, b1, -v1 * bn);
  f[5] = fma_r(vn, b2, -v2 * bn);
  f[6] = fma_r(en + pt, vn, -bn * vb);
}

// Relative tolerance below which the HLLD star state is treated as
// degenerate: 1e-12 in FP64; the same number of units of the working
// precision in FP32 (1e-12 * 2^29), where D = rho (S-u)(S-S_M) - bn^2 is
// the small difference of two large terms at low plasma beta.
template <class R> struct DegenerateTol { static constexpr double value = 1e-12; };
template <> struct DegenerateTol<float> { static constexpr double value = 1e-12 * 536870912.0; };

// Intermediate values of one HLL solve, recorded for the adjoint's reverse sweep
// (RiemannTape) or not at all (NoTape; the compiler drops every store).
struct NoTape {
  static constexpr bool on = false;
};
struct RiemannTape {
  static constexpr bool on = true;
  int region;  // 0 F_L, 1 F_R (outside the fan), 2 HLL fan
  double ul[7], fl[7], ur[7], fr[7], cl, cr, sl, sr, ap, am, isum, v1, v2;
  double idn;  // HLL fan
};

// Riemann fluxes between face-frame states wl | wr with continuous normal field
// bn: HLL (riemann_core) or HLLD (hlld_flux). Wave-speed bounds of both: S_L =
// min(u_L,u_R) - c, S_R = max(u_L,u_R) + c, c = max(c_f,L, c_f,R). HLLD: the
// four-state solver of Miyoshi & Kusano (contact S_M, Alfven fronts S*_L,
// S*_R); when rho (S-u)(S-S_M) - bn^2 vanishes (relative DegenerateTol) the
// tangential fields of that side's star state are left unchanged. Region ties
// go left.
//
// EM 1 with HLL: the UCT-HLLD coefficients om = alpha+/(alpha+ + alpha-), d^L =
// d^R = alpha+ alpha-/(alpha+ + alpha-).
template <class R, class T, int EM = 0>
__device__ __forceinline__ void riemann_core(R g, const R* wl, const R* wr, R bn,
                                             RiemannOut<R>& o, T& tp) {
  R ul[7], fl[7], ur[7], fr[7], ptl, ptr;
  const R igm1 = rcp_r(g - R(1));  // 1/(gamma-1)
  phys(igm1, wl, bn, ul, fl, ptl);
  phys(igm1, wr, bn, ur, fr, ptr);
  const R cl = cfast(g, wl[0], wl[6], bn, wl[4], wl[5]);
  const R cr = cfast(g, wr[0], wr[6], bn, wr[4], wr[5]);
  const R cm = max_r(cl, cr);
  const R sl = min_r(wl[1], wr[1]) - cm;
  const R sr = max_r(wl[1], wr[1]) + cm;
  o.ap = max_r(R(0), sr);
  o.am = max_r(R(0), -sl);
  const R isum = rcp_r(o.ap + o.am);
  o.v1 = fma_r(o.ap, wl[2], o.am * wr[2]) * isum;
  o.v2 = fma_r(o.ap, wl[3], o.am * wr[3]) * isum;
  if constexpr (T::on) {
#pragma unroll
    for (int q = 0; q < 7; ++q) {
      tp.ul[q] = ul[q]; tp.fl[q] = fl[q]; tp.ur[q] = ur[q]; tp.fr[q] = fr[q];
    }
    tp.cl = cl; tp.cr = cr; tp.sl = sl; tp.sr = sr;
    tp.ap = o.ap; tp.am = o.am; tp.isum = isum; tp.v1 = o.v1; tp.v2 = o.v2;
  }
  if (EM == 1) {
    o.om = o.ap * isum;
    o.dl = o.ap * o.am * isum;
    o.dr = o.dl;
  }
  if (sl >= R(0)) {
    if constexpr (T::on) tp.region = 0;
#pragma unroll
    for (int q = 0; q < 7; ++q) o.f[q] = fl[q];
  } else if (sr <= R(0)) {
    if constexpr (T::on) tp.region = 1;
#pragma unroll
    for (int q = 0; q < 7; ++q) o.f[q] = fr[q];
  } else {
    const R idn = rcp_r(sr - sl);
    if constexpr (T::on) { tp.region = 2; tp.idn = idn; }
#pragma unroll
    for (int q = 0; q < 7; ++q)
      o.f[q] = fma_r(sl * sr, ur[q] - ul[q], fma_r(sr, fl[q], -sl * fr[q])) * idn;
  }
}

// The parts of the HLLD solver that decide its branches, shared by hlld_flux and the
// adjoint's reverse sweep, which has to take the branch that the flux took.
template <class R> struct HlldFan {
  R ptl, ptr, c2l, c2r;  // total pressures, squares of the fast speeds
  R sl, sr, sm, pts;     // outer fronts, contact, star total pressure
  R iden;                // 1 / (m_R - m_L), m = rho (S - u)
  bool fan, rt;          // between the outer fronts; right of the contact, or (not in
                         // the fan) in the right state
};
template <class R>
__device__ __forceinline__ HlldFan<R> hlld_fan(R g, const R* wl, const R* wr, R bn, R bn2) {
  HlldFan<R> o;
  o.ptl = fma_r(R(0.5), fma_r(wl[5], wl[5], fma_r(wl[4], wl[4], bn2)), wl[6]);
  o.ptr = fma_r(R(0.5), fma_r(wr[5], wr[5], fma_r(wr[4], wr[4], bn2)), wr[6]);
  // the larger of the two fast speeds: the root of the larger square
  o.c2l = cfast2(g, wl[0], wl[6], bn, wl[4], wl[5]);
  o.c2r = cfast2(g, wr[0], wr[6], bn, wr[4], wr[5]);
  const R cm = sqrt_r(max_r(o.c2l, o.c2r));
  o.sl = min_r(wl[1], wr[1]) - cm;
  o.sr = max_r(wl[1], wr[1]) + cm;
  const R ml = (o.sl - wl[1]) * wl[0], mr = (o.sr - wr[1]) * wr[0];
  o.iden = rcp_r(mr - ml);
  o.sm = fma_r(mr, wr[1], fma_r(-ml, wl[1], o.ptl - o.ptr)) * o.iden;
  o.pts = fma_r(ml * mr, wr[1] - wl[1], fma_r(mr, o.ptl, -ml * o.ptr)) * o.iden;
  // the side the face lies on: outside the fan the upwind one
  const bool outl = o.sl > R(0), outr = !outl && o.sr < R(0);
  o.fan = !outl && !outr;
  o.rt = outr || (o.fan && !(o.sm >= R(0)));
  return o;
}
// Tangential star state of one side with front S, m = d rho, d = S - u, u = un: v*_t
// = v_t - eta B_t, B*_t = zeta B_t (degenerate: v*_t = v_t, B*_t = B_t).
template <class R> struct HlldStar {
  R eta, zeta, iden2;
  bool deg;
};
template <class R>
__device__ __forceinline__ HlldStar<R> hlld_star(R m, R d, R S, R un, R sm, R bn, R bn2) {
  HlldStar<R> o;
  const R big = m * (S - sm);
  const R den = big - bn2;
  o.deg = abs_r(den) <= R(DegenerateTol<R>::value) * (abs_r(big) + bn2);
  o.iden2 = rcp_r(den);  // dropped (maybe not finite) when degenerate
  const R fv = bn * (sm - un) * o.iden2;
  const R fb = fma_r(m, d, -bn2) * o.iden2;
  o.eta = o.deg ? R(0) : fv;
  o.zeta = o.deg ? R(1) : fb;
  return o;
}
// The Alfven front of the side rt, sq the root of its star density; between the
// fronts lies the face where (front >= 0) == rt.
template <class R>
__device__ __forceinline__ R hlld_front(R sm, R abn, R sq, bool rt) {
  const R qa = div_r(abn, sq);
  return sm + (rt ? qa : -qa);
}

// HLLD flux. It needs the physical flux, the energy star state and (unless the face lies
// between the Alfven fronts) the star state of one side only, the side of the
// contact S_M the face lies on: that side is selected first and only its
// quantities are formed; the other side's tangential star state and the
// double-star state follow where a lane of the wave lies between the fronts.
// (What bounds the face kernels is their FP64 instruction count.)
//
// EM 1 also gives the coefficients of the UCT-HLLD edge average. At the wave
// structure of the face the flux of each transverse field component is
// linear in the outer transverse fields and velocities,
//   F[B_t] = chiL B_t^L + chiR B_t^R - bn (om v_t^L + (1 - om) v_t^R);
// the EMF takes om, 1 - om as the weights of v_n B_t on either side,
// d^L = chiL - om u_L and d^R = (1 - om) u_R - chiR as its diffusion
// coefficients, and v1, v2 become the om-weighted velocities. Per region
// (B*_t = zeta B_t and v*_t = v_t - eta B_t on each side; w = 1/(sql + sqr)):
//   F_L, F*_L:  om = 1, chiL = u_L + S_L (zeta_L - 1), chiR = 0;
//   F**_L:      om = 1 + S*_L w sql sqr / |bn|,
//               chiL = u_L + S_L (zeta_L - 1) + S*_L (w (sqr zeta_L + s sql sqr eta_L) - zeta_L),
//               chiR = S*_L w (sql zeta_R - s sql sqr eta_R), s = sign(bn);
//   F**_R, F*_R, F_R: the mirror images.
template <class R, int EM>
__device__ __forceinline__ void hlld_flux(R g, const R* wl, const R* wr, R bn, RiemannOut<R>& o) {
  const R igm1 = rcp_r(g - R(1));  // 1/(gamma-1)
  const R bn2 = bn * bn;
  const HlldFan<R> fn = hlld_fan<R>(g, wl, wr, bn, bn2);
  const R sl = fn.sl, sr = fn.sr, sm = fn.sm, pts = fn.pts;
  const bool rt = fn.rt;
  if (EM == 0) {
    o.ap = max0_r(sr);
    o.am = max0_r(-sl);
    const R isum = rcp_r(o.ap + o.am);
    o.v1 = fma_r(o.ap, wl[2], o.am * wr[2]) * isum;
    o.v2 = fma_r(o.ap, wl[3], o.am * wr[3]) * isum;
  }
  R w[7], u[7], f[7], pt;
#pragma unroll
  for (int q = 0; q < 7; ++q) w[q] = rt ? wr[q] : wl[q];
  phys(igm1, w, bn, u, f, pt);
  if (EM == 1) {
    o.om = rt ? R(0) : R(1);
    o.dl = R(0);
    o.dr = R(0);
    o.v1 = w[2];
    o.v2 = w[3];
  }
#pragma unroll
  for (int q = 0; q < 7; ++q) o.f[q] = f[q];
  if (!fn.fan) return;
  // star state of that side
  const R S = rt ? sr : sl;
  const R d = S - w[1], m = d * w[0];
  const R ism = rcp_r(S - sm);
  const R rs = m * ism;
  const R sq = sqrt_r(rs);
  const R abn = abs_r(bn);
  const R sa = hlld_front(sm, abn, sq, rt);
  const HlldStar<R> st = hlld_star(m, d, S, w[1], sm, bn, bn2);
  const R zeta = st.zeta, eta = st.eta;
  const R vs = fma_r(-w[4], eta, w[2]), ws = fma_r(-w[5], eta, w[3]);
  const R b1s = w[4] * zeta, b2s = w[5] * zeta;
  const R vb = fma_r(w[3], w[5], fma_r(w[2], w[4], w[1] * bn));
  const R vbs = fma_r(ws, b2s, fma_r(vs, b1s, sm * bn));
  const R es = fma_r(bn, vb - vbs, fma_r(pts, sm, fma_r(d, u[6], -pt * w[1]))) * ism;
  const R us[7] = {rs, rs * sm, rs * vs, rs * ws, b1s, b2s, es};
#pragma unroll
  for (int q = 0; q < 7; ++q) o.f[q] = fma_r(S, us[q] - u[q], f[q]);
  if (EM == 1) {
    const R t = S * (zeta - R(1));
    o.dl = rt ? R(0) : t;
    o.dr = rt ? -t : R(0);
  }
  if ((sa >= R(0)) != rt) return;  // outside the Alfven fronts
  // F**: the other side's star state, then the double-star state
  const R so = rt ? sl : sr, uo = rt ? wl[1] : wr[1], rho_o = rt ? wl[0] : wr[0];
  const R vo = rt ? wl[2] : wr[2], wo = rt ? wl[3] : wr[3];
  const R b1o = rt ? wl[4] : wr[4], b2o = rt ? wl[5] : wr[5];
  const R d_o = so - uo, m_o = d_o * rho_o;
  const R sqo = sqrt_r(m_o * rcp_r(so - sm));
  const HlldStar<R> sto = hlld_star(m_o, d_o, so, uo, sm, bn, bn2);
  const R zo = sto.zeta, eo = sto.eta;
  const R vso = fma_r(-b1o, eo, vo), wso = fma_r(-b2o, eo, wo);
  const R b1so = b1o * zo, b2so = b2o * zo;
  // left and right in their places
  const R sql = rt ? sqo : sq, sqr = rt ? sq : sqo;
  const R vl = rt ? vso : vs, vr = rt ? vs : vso, wsl = rt ? wso : ws, wsr = rt ? ws : wso;
  const R b1l = rt ? b1so : b1s, b1r = rt ? b1s : b1so;
  const R b2l = rt ? b2so : b2s, b2r = rt ? b2s : b2so;
  const R sgn = (bn > R(0)) ? R(1) : ((bn < R(0)) ? R(-1) : R(0));
  const R isq = rcp_r(sql + sqr);
  const R ssq = sgn * sql * sqr;
  const R vss = fma_r(sgn, b1r - b1l, fma_r(sql, vl, sqr * vr)) * isq;
  const R wss = fma_r(sgn, b2r - b2l, fma_r(sql, wsl, sqr * wsr)) * isq;
  const R b1ss = fma_r(ssq, vr - vl, fma_r(sql, b1r, sqr * b1l)) * isq;
  const R b2ss = fma_r(ssq, wsr - wsl, fma_r(sql, b2r, sqr * b2l)) * isq;
  const R vbss = fma_r(vss, b1ss, wss * b2ss);
  const R sa_sgn = (rt ? sgn : -sgn) * sq;
  const R ess = fma_r(sa_sgn, fma_r(vs, b1s, ws * b2s) - vbss, es);
  const R uss[7] = {rs, rs * sm, rs * vss, rs * wss, b1ss, b2ss, ess};
#pragma unroll
  for (int q = 0; q < 7; ++q) o.f[q] = fma_r(sa, uss[q] - us[q], o.f[q]);
  if (EM == 1) {
    // (|bn| > 0 there: S*_L < 0 <= S_M or S_M < 0 <= S*_R)
    const R zl = rt ? zo : zeta, zr = rt ? zeta : zo, el = rt ? eo : eta, er = rt ? eta : eo;
    const R ww = isq * sql * sqr;
    const R cl = fma_r(sgn * sql * sqr, el, sqr * zl) * isq;   // B** per B_t^L
    const R cr = fma_r(-sgn * sql * sqr, er, sql * zr) * isq;  // B** per B_t^R
    const R ca = rt ? cr : cl, co = rt ? cl : cr;
    const R t = sa * ww;
    const R q = div_r(rt ? t : -t, abn);
    const R chia = fma_r(sa, ca - zeta, fma_r(S, zeta - R(1), w[1])), chio = sa * co;
    o.om = rt ? q : R(1) - q;
    const R chiL = rt ? chio : chia, chiR = rt ? chia : chio;
    const R omr = R(1) - o.om;
    o.dl = fma_r(-o.om, wl[1], chiL);
    o.dr = fma_r(omr, wr[1], -chiR);
    o.v1 = fma_r(o.om, wl[2], omr * wr[2]);
    o.v2 = fma_r(o.om, wl[3], omr * wr[3]);
  }
}

template <int RS, class R, int EM = 0>
__device__ __forceinline__ void riemann(R g, const R* wl, const R* wr, R bn, RiemannOut<R>& o) {
  if constexpr (RS == 0) {
    hlld_flux<R, EM>(g, wl, wr, bn, o);
  } else {
    NoTape tp;
    riemann_core<R, NoTape, EM>(g, wl, wr, bn, o, tp);
  }
}

// Solve of a face with normal field bn, or (GLM) the exact interface values of
// the (B_n, psi) subsystem from the reconstructed wl[7..8] | wr[7..8],
//   bn = (bn_L + bn_R)/2 - (psi_R - psi_L)/(2 c_h),
//   psi = (psi_L + psi_R)/2 - c_h (bn_R - bn_L)/2,
// then the MHD solve with bn; psi and c_h^2 bn are the fluxes of B_n and psi.
template <int RS, class R, int EM>
__device__ __forceinline__ void face_solve(R gam, const R* wl, const R* wr, R bn, R ch,
                                            RiemannOut<R>& o, R& psi, R& fpsi) {
  if constexpr (EM == 2) {
    bn = R(0.5) * (wl[7] + wr[7]) - div_r(wr[8] - wl[8], R(2) * ch);
    psi = R(0.5) * (wl[8] + wr[8]) - R(0.5) * ch * (wr[7] - wl[7]);
    fpsi = ch * ch * bn;
    riemann<RS, R, 0>(gam, wl, wr, bn, o);
  } else {
    riemann<RS, R, EM>(gam, wl, wr, bn, o);
  }
}

// Upwind edge EMF for component c with cyclic pair (a, b); the exact value
// is v_b B_a - v_a B_b. a-bracket: v_a B_b upwinded along a from the two
// b-faces (W, E) reconstructed toward the edge, with the largest alpha+-
// of the two a-faces touching the edge; b-bracket likewise along b.
template <class R>
__device__ __forceinline__ R uct(R apa, R ama, R vW, R bW, R vE, R bE,
                                 R apb, R amb, R vS, R bS, R vN, R bN) {
  const R ta = div_r(apa * vW * bW + ama * vE * bE - apa * ama * (bE - bW), apa + ama);
  const R tb = div_r(apb * vS * bS + amb * vN * bN - apb * amb * (bN - bS), apb + amb);
  return tb - ta;
}

// UCT-HLLD edge EMF for component c with cyclic pair (a, b): the weights
// (aa, 1 - aa) and diffusion coefficients dla, dra (averaged over the two
// a-faces touching the edge) act on v_a B_b from the two b-faces
// reconstructed along a (W, E); the b-bracket likewise.
template <class R>
__device__ __forceinline__ R uct_hlld(R aa, R dla, R dra, R vW, R bW, R vE, R bE, R ab, R dlb,
                                      R drb, R vS, R bS, R vN, R bN) {
  const R ta = aa * vW * bW + (R(1) - aa) * vE * bE - (dra * bE - dla * bW);
  const R tb = ab * vS * bS + (R(1) - ab) * vN * bN - (drb * bN - dlb * bS);
  return tb - ta;
}

// Values of a face quantity reconstructed toward an edge from the two faces
// beside it: lo = x(-1) + slope(-1)/2 (upper extrapolation of the lower face),
// hi = x(0) - slope(0)/2, from the four faces x(-2), x(-1), x(0), x(+1).
template <int LIM, class R>
__device__ __forceinline__ void edge_pair(R xm2, R xm1, R x0, R xp1, R& lo, R& hi) {
  plm_pair<LIM, R>(xm2, xm1, x0, xp1, lo, hi);
}

// Upwind edge EMF from its inputs: alpha+- of the two a-faces touching the
// edge (below the edge along B, then the cell's own), of the two b-faces
// (below along A, then own); the face velocity v_A and the field b_B on the
// b-faces at A-offsets -2..+1, and v_B and b_A on the a-faces at B-offsets
// -2..+1, each reconstructed toward the edge.
template <int LIM, class R>
__device__ __forceinline__ R emf_core(R apa_m, R apa_c, R ama_m, R ama_c, R apb_m, R apb_c,
                                      R amb_m, R amb_c, const R* vbA, const R* bB, const R* vaB,
                                      const R* bA) {
  const R apa = max_r(apa_m, apa_c), ama = max_r(ama_m, ama_c);
  const R apb = max_r(apb_m, apb_c), amb = max_r(amb_m, amb_c);
  R vW, vE, bW, bE, vS, vN, bS, bN;
  edge_pair<LIM, R>(vbA[0], vbA[1], vbA[2], vbA[3], vW, vE);
  edge_pair<LIM, R>(bB[0], bB[1], bB[2], bB[3], bW, bE);
  edge_pair<LIM, R>(vaB[0], vaB[1], vaB[2], vaB[3], vS, vN);
  edge_pair<LIM, R>(bA[0], bA[1], bA[2], bA[3], bS, bN);
  return uct<R>(apa, ama, vW, bW, vE, bE, apb, amb, vS, bS, vN, bN);
}

// UCT-HLLD edge EMF from its inputs: om, d^L, d^R of the two a-faces (below
// the edge along B, then the cell's own) and of the two b-faces, averaged;
// the reconstructed values as for emf_core.
template <int LIM, class R>
__device__ __forceinline__ R emf_core_hlld(R oma_m, R oma_c, R dla_m, R dla_c, R dra_m, R dra_c,
                                           R omb_m, R omb_c, R dlb_m, R dlb_c, R drb_m, R drb_c,
                                           const R* vbA, const R* bB, const R* vaB,
                                           const R* bA) {
  const R aa = R(0.5) * (oma_m + oma_c), dla = R(0.5) * (dla_m + dla_c);
  const R dra = R(0.5) * (dra_m + dra_c);
  const R ab = R(0.5) * (omb_m + omb_c), dlb = R(0.5) * (dlb_m + dlb_c);
  const R drb = R(0.5) * (drb_m + drb_c);
  R vW, vE, bW, bE, vS, vN, bS, bN;
  edge_pair<LIM, R>(vbA[0], vbA[1], vbA[2], vbA[3], vW, vE);
  edge_pair<LIM, R>(bB[0], bB[1], bB[2], bB[3], bW, bE);
  edge_pair<LIM, R>(vaB[0], vaB[1], vaB[2], vaB[3], vS, vN);
  edge_pair<LIM, R>(bA[0], bA[1], bA[2], bA[3], bS, bN);
  return uct_hlld<R>(aa, dla, dra, vW, bW, vE, bE, ab, dlb, drb, vS, bS, vN, bN);
}

}  // namespace mhd
