// Index helpers and primitive recovery shared by the forward and adjoint
// kernels (periodic Cartesian grid, field-major SoA, x fastest).
#pragma once
#include "mhd_device.hpp"

namespace mhd {

constexpr int kBlock = 256;

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

__device__ __forceinline__ int64_t lin(const Geom& g, int i, int j, int k) {
  return ((int64_t)k * g.ny + j) * g.nx + i;
}

__device__ __forceinline__ void coords(const Geom& g, int64_t c, int& i, int& j, int& k) {
  i = (int)(c % g.nx);
  const int64_t r = c / g.nx;
  j = (int)(r % g.ny);
  k = (int)(r / g.ny);
}

// Cell shifted by s (|s| <= 2) along direction D, periodic.
template <int D>
__device__ __forceinline__ int64_t shifted(const Geom& g, int i, int j, int k, int s) {
  if (D == 0) return lin(g, wrap(i + s, g.nx), j, k);
  if (D == 1) return lin(g, i, wrap(j + s, g.ny), k);
  return lin(g, i, j, wrap(k + s, g.nz));
}

// The same value, of which the compiler does not know that it is: what is
// derived from it is formed where it is used instead of being hoisted out of a
// loop, or shared between faces, in registers that the solves need (and an
// offset is seen as the zero-extended 32 bits that the scalar-base addressing
// form takes).
template <class T>
__device__ __forceinline__ T here(T v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A value that every lane holds alike, in scalar registers.
__device__ __forceinline__ double uni(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float uni(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
// The value at byte offset off of the uniform base b.
__device__ __forceinline__ double ld_at(const double* __restrict__ b, uint32_t off) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(b) + off);
}
// The stored values primitive recovery at a cell reads: its 8 fields and
// the staggered field on its three upper faces.
struct RawCell {
  double u[8];
  double bxp, byp, bzp;
};

template <int DIM>
__device__ __forceinline__ RawCell load_raw(const double* __restrict__ U, const Geom& g, int i,
                                            int j, int k) {
  const int64_t n = g.n;
  const int64_t c = lin(g, i, j, k);
  RawCell r;
#pragma unroll
  for (int q = 0; q < 8; ++q) r.u[q] = U[q * n + c];
  r.bxp = U[5 * n + lin(g, wrap(i + 1, g.nx), j, k)];
  r.byp = U[6 * n + lin(g, i, wrap(j + 1, g.ny), k)];
  r.bzp = (DIM == 3) ? U[7 * n + lin(g, i, j, wrap(k + 1, g.nz))] : 0.0;
  return r;
}

// Primitive recovery (always FP64): V = (rho, vx, vy, vz, p, Bx, By, Bz), B
// cell-centred as the mean of the two faces (2D: field 7 is already
// cell-centred). Returns false for an unphysical cell.
template <int DIM>
__device__ __forceinline__ bool prim_from_raw(const RawCell& r, double gamma, double* V) {
  const double rho = r.u[0];
  const double mx = r.u[1], my = r.u[2], mz = r.u[3], en = r.u[4];
  const double bx = 0.5 * (r.u[5] + r.bxp);
  const double by = 0.5 * (r.u[6] + r.byp);
  const double bz = (DIM == 3) ? 0.5 * (r.u[7] + r.bzp) : r.u[7];
  const double irho = rcp_r(rho);
  const double vx = mx * irho, vy = my * irho, vz = mz * irho;
  const double kin = 0.5 * fma_r(mz, vz, fma_r(my, vy, mx * vx));
  const double mag = 0.5 * fma_r(bz, bz, fma_r(by, by, bx * bx));
  const double p = (gamma - 1.0) * (en - kin - mag);
  V[0] = rho; V[1] = vx; V[2] = vy; V[3] = vz; V[4] = p; V[5] = bx; V[6] = by; V[7] = bz;
  return (rho > 0.0) && (p > 0.0) && __builtin_isfinite(p) && __builtin_isfinite(vx) &&
         __builtin_isfinite(vy) && __builtin_isfinite(vz);
}

// Primitive recovery at cell (i,j,k).
template <int DIM>
__device__ __forceinline__ bool prim_at(const double* __restrict__ U, const Geom& g, int i, int j,
                                        int k, double* V) {
  return prim_from_raw<DIM>(load_raw<DIM>(U, g, i, j, k), g.gamma, V);
}

// Partial derivatives (d slope/d dm, d slope/d dp) of the limited slope.
template <int LIM>
__device__ __forceinline__ void plm_slope_grad(double dm, double dp, double& s1, double& s2) {
  const bool ext = dm * dp <= 0.0;
  if (LIM == 0) {
    const bool left = __builtin_fabs(dm) <= __builtin_fabs(dp);
    s1 = (ext || !left) ? 0.0 : 1.0;
    s2 = (ext || left) ? 0.0 : 1.0;
  } else {
    // branch-free: at extrema (where dm + dp may vanish) the select drops the
    // value of the refined reciprocal
    const double is = rcp_r(dm + dp);
    s1 = ext ? 0.0 : 2.0 * dp * dp * is * is;
    s2 = ext ? 0.0 : 2.0 * dm * dm * is * is;
  }
}

// Adjoint of piecewise-linear extrapolation along one line. x[0..4] are the
// values at positions -2..+2 around position 0; xp[p], xm[p] (p = 0,1,2 for
// positions -1, 0, +1) are the cotangents of the upper extrapolation
// x + slope/2 and the lower one x - slope/2 at those positions. Returns the
// cotangent of x at position 0.
template <int LIM>
__device__ __forceinline__ double plm_adjoint(const double* x, const double* xp,
                                              const double* xm) {
  double s1[3], s2[3], sb[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    plm_slope_grad<LIM>(x[p + 1] - x[p], x[p + 2] - x[p + 1], s1[p], s2[p]);
    sb[p] = 0.5 * (xp[p] - xm[p]);
  }
  return xp[1] + xm[1] + sb[1] * (s1[1] - s2[1]) - sb[2] * s1[2] + sb[0] * s2[0];
}

__device__ __forceinline__ int wrap_any(int i, int n) {
  int r = i % n;
  return r < 0 ? r + n : r;
}

// Face records (fluxes, alpha+-, HLL-weighted velocities) and edge EMFs are
// stored in the precision they were computed in: FP64, or FP32 in the mixed
// mode (exact, and half the bytes for the kernels that read them). The
// workspace holds dim * NSLOT * n and 3 * n doubles either way.
template <class R>
__device__ __forceinline__ R* stored(double* buf) {
  return reinterpret_cast<R*>(buf);
}
template <class R>
__device__ __forceinline__ const R* stored(const double* buf) {
  return reinterpret_cast<const R*>(buf);
}

// CFL bound of one cell from its FP64 primitives: min over directions of
// dx_d / (|v_d| + c_f,d).
template <int DIM>
__device__ __forceinline__ double cfl_bound(const Geom& g, const double* W, double m) {
  const double dd[3] = {g.dx, g.dy, g.dz};
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const double cf = cfast<double>(g.gamma, W[0], W[4], W[5 + d], W[5 + (d + 1) % 3],
                                    W[5 + (d + 2) % 3]);
    const double t = div_r(dd[d], __builtin_fabs(W[1 + d]) + cf);
    m = (t < m) ? t : m;
  }
  return m;
}

// Minimum of v over the kBlock threads of the workgroup, stored by thread 0
// to *out. Every thread of the workgroup must call it.
__device__ __forceinline__ void workgroup_min_store(double v, double* __restrict__ out) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(v, off, 64);
    v = (o < v) ? o : v;
  }
  __shared__ double red[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = red[0];
#pragma unroll
    for (int w = 1; w < kBlock / 64; ++w) r = (red[w] < r) ? red[w] : r;
    *out = r;
  }
}

// The stages' combinations of u, the state L was formed at, and u0, the state at
// the start of the step: 0: L; 1: u + h L; 2: (u0 + (u + h L)) / 2; 4: (3 u0 + (u +
// h L)) / 4; 5: (u0 + 2 (u + h L)) / 3. By coefficients, for a stage known at run
// time without a branch per value: (ca u0 + cb (cu u + h L)) / cd, the quotient by
// the divisors 1, 2, 4 exact and by 3 corrected to the rounded one.
struct RkCoef {
  double cu, h, ca, cb, cc, cd;
};
__device__ __forceinline__ RkCoef rk_coef(int stage, double h) {
  RkCoef c = {1.0, h, 0.0, 1.0, 1.0, 1.0};
  if (stage == 0) { c.cu = 0.0; c.h = 1.0; }
  if (stage == 2) { c.ca = 1.0; c.cc = 0.5; c.cd = 2.0; }
  if (stage == 4) { c.ca = 3.0; c.cc = 0.25; c.cd = 4.0; }
  if (stage == 5) { c.ca = 1.0; c.cb = 2.0; c.cc = 1.0 / 3.0; c.cd = 3.0; }
  return c;
}
__device__ __forceinline__ double rk_apply(const RkCoef& c, double u, double u0, double L) {
  const double v = c.ca * u0 + c.cb * (c.cu * u + c.h * L);
  const double q = v * c.cc;
  return fma_r(fma_r(-c.cd, q, v), c.cc, q);
}

}  // namespace mhd
