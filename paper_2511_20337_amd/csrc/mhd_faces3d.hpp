// 3D stage: the z-marching face kernel, which also differences the fluxes of the
// cell-averaged fields.
//
// A workgroup owns a 32 x 8 column of cells and walks a run of planes
// k0 <= k < k1, one cell of each plane per thread. Per plane each thread
// solves the lower z-, x- and y-face of its cell; the faces above the column
// (32 y-faces, 8 x-faces) are solved once more by one wave, in turn, so that
// every flux the column's cells need is at hand: only the inputs of the edge
// EMFs (alpha+- or the UCT-HLLD coefficients, two velocities: 12 or 15 values
// per cell) go to memory, and the five flux divergences end in the new state
// directly. A face solved twice gives the same bits both times.
//
// With GLM cleaning (nine cell-centred fields, no edge EMFs) this kernel is the
// whole stage. WENO-Z reads the primitives k_prim left: its stencil is three
// cells either way, and recovering them again at each plane's halo cost more.
//
// What bounds it: the instruction count (1840 per cell at 256^3 in FP64, the
// vector units 67 % busy; WENO-Z 3450 and 75 %). Measured against the split it replaces (a face
// kernel that stored the fluxes, 27 values per cell, and an update that read
// them back): faces 1.52 -> 1.60 ms, update 0.96 -> 0.43 ms per launch at 256^3
// in FP64, the step 6.32 -> 5.35 ms; 384^3 mixed 13.9 -> 12.4 ms; with GLM (before:
// primitives 0.44, faces 1.97 and update 1.32 ms per stage through memory) 1.62
// ms per stage, the step 7.50 -> 3.40 ms. WENO-Z (before: a face kernel without
// LDS and an update that read all its fluxes back): 352^3 with RK3 and UCT-HLLD
// faces 6.5 -> 6.4, update 2.7 -> 0.68 ms a stage, the step 35.8 -> 30.2 ms;
// 150 x 131 x 97 with GLM 1112 -> 900 us. Choices:
//  - 32 x 8 columns: the extra faces fit one wave (40 lanes; 64 x 4 needs 68),
//    the halo is 160 cells a plane (64 x 4: 272), and a ragged nx wastes less.
//  - LDS holds two planes of the column (by the parity of k - k0; the values a
//    thread needs of planes k-1 and k+1 are its own), one cross halo and the
//    exchanged fluxes.
//  - Two waves per SIMD in FP64 (214 VGPRs, GLM and WENO-Z with GLM 254), three in
//    mixed precision: one more spills (FP64 1.95 ms against 1.52, mixed 384^3 3.73
//    against 3.39).
//  - Fluxes are differenced before they are added up, so a uniform flow has L = 0 and
//    a cell's result does not depend on its place in the column (a running sum over
//    the faces has neither, and takes as long). The lower z-flux waits for the upper
//    one in registers; with HLL in FP64, which would need 176 (with 168 or fewer three
//    workgroups fit a CU), and in WENO-Z with GLM, which would spill, in the thread's
//    own slot of fy, free between the exchanges (GLM that way: 256^3 3311 against 3254
//    us a step).
//  - Two barriers a plane: before the first one everybody reads plane k; then
//    the halo of plane k+1 and the exchanged fluxes are written; the second
//    publishes them.
//  - Lanes past a ragged grid hold the periodic images of the first cells, so
//    their faces are those of the cells they repeat: they are solved and their
//    edge inputs stored like any other (the same bits to the same place),
//    which keeps every path through a plane alike. Only the new state, which
//    may be updated in place, is written by its owner alone.
#pragma once
#include <algorithm>

#include "mhd_device.hpp"
#include "mhd_grid.hpp"
#include "mhd_kernels.hpp"

namespace mhd {

namespace {

struct March {
  static constexpr int TX = 32, TY = 8, NCORE = TX * TY;
};
static_assert(March::NCORE == kBlock, "one column cell per thread");
static_assert(March::TX + March::TY <= 64, "the faces above the column fit one wave");
static_assert(March::TX == 32, "a wave holds two rows");

// The cross halo of S cells below and S above (PLM 2, WENO-Z 3) and the LDS
// offsets. One stride for every quantity, core or halo, so that a stencil cell
// is one offset and its quantities lie at constant distances from it.
template <int S>
struct Halo {
  static constexpr int NX = 2 * S * March::TY;         // columns -S .. -1, TX .. TX + S - 1
  static constexpr int N = NX + 2 * S * March::TX;     // then the rows
  static constexpr int OFF = 2 * March::NCORE;         // offset, after the core of two planes
  static constexpr int Q = 2 * March::NCORE + N;       // quantity stride
  static_assert(N <= March::NCORE, "at most one halo cell per thread");
  // Position of halo entry h relative to the column origin.
  static __device__ __forceinline__ void pos(int h, int& x, int& y) {
    if (h < NX) {
      const int s = h / March::TY;
      y = h % March::TY;
      x = (s < S) ? s - S : March::TX + s - S;
    } else {
      h -= NX;
      const int s = h / March::TX;
      x = h % March::TX;
      y = (s < S) ? s - S : March::TY + s - S;
    }
  }
  // Offset of cell (xx, yy) of the plane whose core starts at cp (at most one
  // coordinate outside the column).
  static __device__ __forceinline__ int at(int cp, int xx, int yy) {
    const int hx = OFF + ((xx < 0) ? xx + S : xx - March::TX + S) * March::TY + yy;
    const int hy = OFF + NX + ((yy < 0) ? yy + S : yy - March::TY + S) * March::TX + xx;
    const int in = cp + yy * March::TX + xx;
    return (xx < 0 || xx >= March::TX) ? hx : (yy < 0 || yy >= March::TY) ? hy : in;
  }
};

template <class R, int S, int NQ, int NF>
struct MarchLds {
  R v[NQ][Halo<S>::Q];     // core of two planes, halo
  R fy[NF][March::NCORE];  // y-fluxes of rows 1 .. TY (row r at (r - 1) * TX)
  R fx[NF][March::TY];     // x-fluxes at column TX
  double red[March::NCORE / 64];
};

// Byte offsets within a plane of one field (FP64) of the values the primitive
// recovery of cell (i, j) reads (indices wrapped): the cell, and its upper x
// and y neighbours (staggered B_x, B_y). The staggered B_z above is the
// cell's own offset in the next plane. 32 bits: a plane holds fewer than
// 2^29 cells.
struct PlaneOffs {
  uint32_t c, xp, yp;
};
__device__ __forceinline__ PlaneOffs plane_offs(const Geom& g, int i, int j, bool wide) {
  const int iw = wide ? wrap(i, g.nx) : wrap_any(i, g.nx);
  const int jw = wide ? wrap(j, g.ny) : wrap_any(j, g.ny);
  PlaneOffs p;
  p.c = (uint32_t)(jw * g.nx + iw) * 8u;
  p.xp = (uint32_t)(jw * g.nx + wrap(iw + 1, g.nx)) * 8u;
  p.yp = (uint32_t)(wrap(jw + 1, g.ny) * g.nx + iw) * 8u;
  return p;
}
// Raw values of the cell at offsets p in plane kw; the staggered B_z above
// from plane kw1 (both wrapped into 0..nz-1). GLM (EM 2): the nine
// cell-centred values, psi in bzp. WENO-Z (LIM 2): the primitives, from U = PW.
template <int LIM, int EM>
__device__ __forceinline__ RawCell load_raw_plane(const double* __restrict__ U, const Geom& g,
                                                  int64_t nxy, int kw, int kw1,
                                                  const PlaneOffs& p) {
  const double* pl = U + kw * nxy;
  const uint32_t c = here(p.c), xp = here(p.xp), yp = here(p.yp);
  RawCell r;
#pragma unroll
  for (int q = 0; q < 8; ++q) r.u[q] = ld_at(pl + q * g.n, c);
  if constexpr (EM == 2 || LIM == 2) {
    r.bxp = r.byp = 0.0;
    r.bzp = (EM == 2) ? ld_at(pl + 8 * g.n, c) : 0.0;
    return r;
  }
  r.bxp = ld_at(pl + 5 * g.n, xp);
  r.byp = ld_at(pl + 6 * g.n, yp);
  r.bzp = ld_at(U + 7 * g.n + kw1 * nxy, c);
  return r;
}

// The primitives of a raw cell (GLM: with psi as the ninth).
template <int LIM, int EM>
__device__ __forceinline__ bool march_prim(const RawCell& r, double gamma, double* W) {
  if constexpr (LIM == 2) {  // recovered (and checked) already
#pragma unroll
    for (int q = 0; q < 8; ++q) W[q] = r.u[q];
    W[8] = r.bzp;
    return true;
  } else if constexpr (EM == 2) {
    RawCell c = r;  // a mean of two equal faces is the cell's field, exactly
    c.bxp = r.u[5];
    c.byp = r.u[6];
    c.bzp = r.u[7];
    W[8] = r.bzp;
    return prim_from_raw<3>(c, gamma, W);
  } else {
    return prim_from_raw<3>(r, gamma, W);
  }
}

// The edge inputs of a lower D-face of the plane whose records start at fwp
// (slot 0 of direction 0), the cell at byte offset boff.
template <int D, int EM, class R>
__device__ __forceinline__ void put_edge(R* __restrict__ fwp, int64_t n, uint32_t boff,
                                         const RiemannOut<R>& o) {
  const uint32_t off = here(boff);
  auto put = [&](int slot, R v) {
    *reinterpret_cast<R*>(reinterpret_cast<char*>(fwp + ((int64_t)D * NSLOT + slot) * n) +
                          off) = v;
  };
  if (EM == 1) {
    put(S_AP, o.om);
    put(S_AM, o.dl);
    put(S_DR, o.dr);
  } else {
    put(S_AP, o.ap);
    put(S_AM, o.am);
  }
  put(S_V1, o.v1);
  put(S_V2, o.v2);
}

// Fluxes of (rho, m_x, m_y, m_z, E), with GLM also of (B_x, B_y, B_z, psi),
// through a D-face.
template <int D, int EM, class R>
__device__ __forceinline__ void cell_fluxes(const RiemannOut<R>& o, R psi, R fpsi, R* F) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  F[0] = o.f[0];
  F[1 + D] = o.f[1];
  F[1 + T1] = o.f[2];
  F[1 + T2] = o.f[3];
  F[4] = o.f[6];
  if constexpr (EM == 2) {
    F[5 + D] = psi;
    F[5 + T1] = o.f[4];
    F[5 + T2] = o.f[5];
    F[8] = fpsi;
  }
}

// Left and right value of quantity q at a face from its stencil cells (offsets
// o), S of them on either side.
template <int LIM, int S, class R>
__device__ __forceinline__ void march_pair(const R* lds, const int* o, int q, R& l, R& r) {
  R v[2 * S];
#pragma unroll
  for (int s = 0; s < 2 * S; ++s) v[s] = lds[o[s] + q * Halo<S>::Q];
  if constexpr (LIM == 2) {
    l = wenoz_upper(v[0], v[1], v[2], v[3], v[4]);
    r = wenoz_upper(v[5], v[4], v[3], v[2], v[1]);
  } else {
    plm_pair<LIM, R>(v[0], v[1], v[2], v[3], l, r);
  }
}

// stage: as rk_coef, for the five cell-averaged fields (U0 not null: U
// where the stage does not use it); 3: no state. Lc != nullptr: their L too, into
// Lc[5][n]. EM 2: GLM cleaning, nine cell-centred fields and no edge inputs, c_h =
// ch0 / dt, psi times decay in a step's last stage. cflp != nullptr:
// dt = cfl times the minimum of the npart CFL partials of U, also to *dt_out.
template <int LIM, int RS, class R, int EM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 2 : 3)))
void k_faces_march(const double* __restrict__ U, const double* __restrict__ PW,
                   const double* U0, double* out,
                   double* __restrict__ FW, Geom g, MarchGrid mg, int stage, double dt,
                   const double* __restrict__ dtp, int* __restrict__ flag,
                   double* __restrict__ Lc, double ch0, double decay,
                   const double* __restrict__ cflp, int npart, double cfl, double* dt_out) {
  using M = March;
  constexpr bool GLM = EM == 2, WZ = LIM == 2;
  // the lower z-flux waits in LDS where registers are short (see above)
  constexpr bool ZL = GLM ? WZ : (!WZ && RS == 1 && sizeof(R) == 8);
  constexpr int S = WZ ? 3 : 2;
  using HL = Halo<S>;
  const double* __restrict__ const src = WZ ? PW : U;
  constexpr int NQ = GLM ? 9 : 8, NF = GLM ? 9 : 5, NW = GLM ? 9 : 7;
  // face frames (rho, v_n, v_t1, v_t2, B_t1, B_t2, p), GLM: and (B_n, psi)
  constexpr int xslot[9] = {0, 1, 2, 3, 6, 7, 4, 5, 8}, yslot[9] = {0, 2, 3, 1, 7, 5, 4, 6, 8};
  constexpr int zslot[9] = {0, 3, 1, 2, 5, 6, 4, 7, 8};
  __shared__ MarchLds<R, S, NQ, NF> L;
  R* lds = &L.v[0][0];
  const unsigned b = blockIdx.x;
  const int tx = (int)(b % (unsigned)mg.ntx);
  const unsigned r = b / (unsigned)mg.ntx;
  const int ty = (int)(r % (unsigned)mg.nty);
  const int zc = (int)(r / (unsigned)mg.nty);
  const int i0 = tx * M::TX, j0 = ty * M::TY;
  const int k0 = zc * mg.lz;
  const int k1 = min(k0 + mg.lz, g.nz);
  const int t = (int)threadIdx.x;
  const int x = t % M::TX, y = t / M::TX;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const bool inside = (i0 + x < g.nx) && (j0 + y < g.ny);
  const int64_t n = g.n, nxy = (int64_t)g.nx * g.ny;
  const R gam = (R)g.gamma;
  // (a remainder only where the grid is smaller than what its last column reaches)
  const bool wide = mg.ntx * M::TX + S <= 2 * g.nx && mg.nty * M::TY + S <= 2 * g.ny;
  const PlaneOffs po = plane_offs(g, i0 + x, j0 + y, wide);
  const uint32_t boff = po.c / 8u * (uint32_t)sizeof(R);
  // halo cell (threads past the halo load a valid cell and drop it)
  const bool haloer = t < HL::N;
  int hx, hy;
  HL::pos(haloer ? t : HL::N - 1, hx, hy);
  const PlaneOffs ph = plane_offs(g, i0 + hx, j0 + hy, wide);
  // face above the column of this lane: y-faces of lanes 0 .. 31, x-faces of
  // lanes 32 .. 39 (further lanes repeat the last); the offset of its cell
  uint32_t eoff;
  {
    const bool ey = lane < M::TX;
    const int e = ey ? lane : min(lane - M::TX, M::TY - 1);
    eoff = plane_offs(g, i0 + (ey ? e : M::TX), j0 + (ey ? M::TY : e), wide).c;
  }
  const double idx = uni(1.0 / g.dx), idy = uni(1.0 / g.dy), idz = uni(1.0 / g.dz);
  bool bad = false;
  if (cflp) {
    double m = __builtin_inf();
    for (int e = t; e < npart; e += M::NCORE) m = (cflp[e] < m) ? cflp[e] : m;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(m, off, 64);
      m = (o < m) ? o : m;
    }
    if (lane == 0) L.red[wave] = m;
  }
  // Prologue: plane k0 (core and halo), V_{k0-1} of the own cell in the other
  // core plane, the left state of the first z-face, the raw cell of k0 + 1.
  R zl[NW];
  double bn[3];  // normal fields of the own cell's lower faces, plane k
  // WENO-Z: the own column's z-face quantities of planes k - 2 and k + 2, the
  // normal fields of plane k + 1
  double zm2[NW], zp2[NW], nb[3] = {0.0, 0.0, 0.0};
  {
    const int km2 = wrap(k0 - 2, g.nz), km1 = wrap(k0 - 1, g.nz);
    const int kp1 = wrap(k0 + 1, g.nz);
    const RawCell rm2 = load_raw_plane<LIM, EM>(src, g, nxy, km2, km1, po);
    const RawCell rm1 = load_raw_plane<LIM, EM>(src, g, nxy, km1, k0, po);
    const RawCell rc = load_raw_plane<LIM, EM>(src, g, nxy, k0, kp1, po);
    const RawCell rh = load_raw_plane<LIM, EM>(src, g, nxy, k0, kp1, ph);
    double Wm2[9], Wm1[9], W[9];
    bad |= !march_prim<LIM, EM>(rm2, g.gamma, Wm2);
    bad |= !march_prim<LIM, EM>(rm1, g.gamma, Wm1);
    bad |= !march_prim<LIM, EM>(rc, g.gamma, W);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      lds[q * HL::Q + M::NCORE + t] = (R)Wm1[q];
      lds[q * HL::Q + t] = (R)W[q];
    }
    if constexpr (WZ) {
      // the upper value of cell k0 - 1, from planes k0 - 3 .. k0 + 1, as the run below
      // forms it (wenoz_both, its lower value unused): the face between two runs is
      // solved by either, to the same bits
      const double* const pm3 = PW + wrap(k0 - 3, g.nz) * nxy;
      const double* const pp1 = PW + kp1 * nxy;
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const int sq = zslot[q];
        double lo;
        wenoz_both(ld_at(pm3 + sq * n, po.c), Wm2[sq], Wm1[sq], W[sq], ld_at(pp1 + sq * n, po.c),
                   lo, zl[q]);
        zm2[q] = Wm2[sq];
        zp2[q] = ld_at(PW + sq * n + wrap(k0 + 2, g.nz) * nxy, po.c);
      }
    } else {
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const R a = (R)Wm2[zslot[q]], bb = (R)Wm1[zslot[q]], c = (R)W[zslot[q]];
        zl[q] = plm_up<LIM, R>(plm_slope<LIM, R>(bb - a, c - bb), bb);
      }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      bn[d] = WZ ? (GLM ? 0.0 : ld_at(U + (F_BX + d) * n + k0 * nxy, po.c)) : rc.u[5 + d];
      if (WZ && !GLM) nb[d] = ld_at(U + (F_BX + d) * n + kp1 * nxy, po.c);
    }
    if (haloer) {
      bad |= !march_prim<LIM, EM>(rh, g.gamma, W);
#pragma unroll
      for (int q = 0; q < NQ; ++q) lds[q * HL::Q + HL::OFF + t] = (R)W[q];
    }
  }
  RawCell nxt =
      load_raw_plane<LIM, EM>(src, g, nxy, wrap(k0 + 1, g.nz), wrap(k0 + 2, g.nz), po);
  __syncthreads();
  double h = 0.0;
  if (cflp) {
    double m = L.red[0];
#pragma unroll
    for (int w = 1; w < M::NCORE / 64; ++w) m = (L.red[w] < m) ? L.red[w] : m;
    h = uni(cfl * m);
    if (b == 0 && t == 0) *dt_out = h;
  } else if (stage != 0 && stage != 3) {
    h = uni(dtp ? *dtp : dt);
  }
  const RkCoef rk = rk_coef(stage, h);
  const R ch = GLM ? uni((R)(ch0 / h)) : R(0);
  int cp = 0;  // core offset of plane k
  double acc[NF];  // flux differences along x and y of the own cell
  R fz[NF];        // its lower z-flux; ZL: in L.fy[.][t] but for the exchange
  R* const fw0 = reinterpret_cast<R*>(FW);
  for (int k = k0;; ++k) {
    const int kw = wrap(k, g.nz);
    R* const fwp = fw0 + kw * nxy;
    R wl[NW], wr[NW], psi = R(0), fpsi = R(0);
    RiemannOut<R> o;
    // z-face: the own cell of plane k + 1, then the reconstruction of cell k,
    // which gives the right state and the next plane's left state
    double bnn[3];
    {
      double W[9];
      bad |= !march_prim<LIM, EM>(nxt, g.gamma, W);
#pragma unroll
      for (int d = 0; d < 3; ++d) bnn[d] = WZ ? nb[d] : nxt.u[5 + d];
      const int cn = M::NCORE - cp + t;  // own cell in the other core plane: k - 1, then k + 1
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const int sq = zslot[q];
        const R a = lds[cn + sq * HL::Q];
        const R bb = lds[cp + t + sq * HL::Q];
        const R c = (R)W[sq];
        wl[q] = zl[q];
        if constexpr (WZ) {
          wenoz_both(zm2[q], a, bb, c, zp2[q], wr[q], zl[q]);
        } else {
          const R dlt = plm_slope<LIM, R>(bb - a, c - bb);
          wr[q] = plm_lo<LIM, R>(dlt, bb);
          zl[q] = plm_up<LIM, R>(dlt, bb);
        }
        // formed here: the compiler otherwise moves the arithmetic of the next
        // plane's left state behind the faces and keeps its inputs until then
        // (WENO-Z spilled 200 B a lane and took 9.5 ms instead of 6.4 at 352^3)
        zl[q] = here(zl[q]);
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) lds[cn + q * HL::Q] = (R)W[q];
    }
    face_solve<RS, R, EM>(gam, wl, wr, (R)bn[2], ch, o, psi, fpsi);
    {
      R F[NF];
      cell_fluxes<2, EM>(o, psi, fpsi, F);
      // the cell below is finished
      const int64_t cb = (int64_t)(k - 1) * nxy;
      if (k > k0 && inside) {
        const uint32_t c = here(po.c);
        auto put = [&](double* p, double v) {
          *reinterpret_cast<double*>(reinterpret_cast<char*>(p + cb) + c) = v;
        };
#pragma unroll
        for (int q = 0; q < NF; ++q)
          acc[q] = -(acc[q] + ((double)F[q] - (double)(ZL ? L.fy[q][t] : fz[q])) * idz);
        if (stage != 3) {
          double u[NF], u0[NF];
#pragma unroll
          for (int q = 0; q < NF; ++q) {
            u[q] = ld_at(U + q * n + cb, c);
            u0[q] = ld_at(U0 + q * n + cb, c);
          }
#pragma unroll
          for (int q = 0; q < NF; ++q) {
            double v = rk_apply(rk, u[q], u0[q], acc[q]);
            if (GLM && q == 8) v *= decay;
            put(out + q * n, v);
          }
        }
        if (Lc) {
#pragma unroll
          for (int q = 0; q < NF; ++q) put(Lc + q * n, acc[q]);
        }
      }
      if (k == k1) break;
#pragma unroll
      for (int q = 0; q < NF; ++q) (ZL ? L.fy[q][t] : fz[q]) = F[q];
    }
    if constexpr (!GLM) put_edge<2, EM>(fwp, n, boff, o);
    const int ka = wrap(k + 1, g.nz), kb = wrap(k + 2, g.nz), kc = wrap(k + 3, g.nz);
    // x-face
    {
      const int tt = here(t), xx = tt & (M::TX - 1), yy = tt / M::TX;
      int os[2 * S];
#pragma unroll
      for (int s = 0; s < 2 * S; ++s) os[s] = HL::at(cp, xx - S + s, yy);
#pragma unroll
      for (int q = 0; q < NW; ++q) march_pair<LIM, S, R>(lds, os, xslot[q], wl[q], wr[q]);
    }
    face_solve<RS, R, EM>(gam, wl, wr, (R)bn[0], ch, o, psi, fpsi);
    if constexpr (!GLM) put_edge<0, EM>(fwp, n, boff, o);
    {
      R F[NF];
      cell_fluxes<0, EM>(o, psi, fpsi, F);
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        // the upper face; the last column keeps the lower one until it is exchanged
        const R up = __shfl_down(F[q], 1, 64);
        acc[q] = (x == M::TX - 1) ? (double)F[q] : ((double)up - (double)F[q]) * idx;
      }
    }
    // y-face
    {
      const int tt = here(t), xx = tt & (M::TX - 1), yy = tt / M::TX;
      int os[2 * S];
#pragma unroll
      for (int s = 0; s < 2 * S; ++s) os[s] = HL::at(cp, xx, yy - S + s);
#pragma unroll
      for (int q = 0; q < NW; ++q) march_pair<LIM, S, R>(lds, os, yslot[q], wl[q], wr[q]);
    }
    face_solve<RS, R, EM>(gam, wl, wr, (R)bn[1], ch, o, psi, fpsi);
    if constexpr (!GLM) put_edge<1, EM>(fwp, n, boff, o);
    R fy[NF];
    cell_fluxes<1, EM>(o, psi, fpsi, fy);
    // the faces above the column: one wave, in turn
    const bool helper = wave == ((k - k0) & 3);
    R fe[NF];
    if (helper) {
      const int l = here(lane);
      const bool ey = l < M::TX;
      const int e = ey ? l : min(l - M::TX, M::TY - 1);
      const double ebn =
          GLM ? 0.0 : ld_at(U + (ey ? F_BY : F_BX) * n + kw * nxy, here(eoff));
      // slots: the x frame's, plus 1 at (v_n, v_t1, B_t1, B_n) and minus 2 at
      // (v_t2, B_t2) for a y-face
      const int up = ey ? HL::Q : 0, dn = ey ? -2 * HL::Q : 0;
      int os[3][2 * S];
#pragma unroll
      for (int s = 0; s < 2 * S; ++s) {
        os[0][s] = HL::at(cp, ey ? e : M::TX - S + s, ey ? M::TY - S + s : e);
        os[1][s] = os[0][s] + up;
        os[2][s] = os[0][s] + dn;
      }
      constexpr int kind[9] = {0, 1, 1, 2, 1, 2, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < NW; ++q)
        march_pair<LIM, S, R>(lds, os[kind[q]], xslot[q], wl[q], wr[q]);
      face_solve<RS, R, EM>(gam, wl, wr, (R)ebn, ch, o, psi, fpsi);
      fe[0] = o.f[0];
      fe[1] = ey ? o.f[3] : o.f[1];
      fe[2] = ey ? o.f[1] : o.f[2];
      fe[3] = ey ? o.f[2] : o.f[3];
      fe[4] = o.f[6];
      if constexpr (GLM) {
        fe[5] = ey ? o.f[5] : psi;
        fe[6] = ey ? psi : o.f[4];
        fe[7] = ey ? o.f[4] : o.f[5];
        fe[8] = fpsi;
      }
    }
    // the raw halo cell of plane k + 1 and own cell of plane k + 2 (their
    // latency passes at the barriers)
    const RawCell hr = load_raw_plane<LIM, EM>(src, g, nxy, ka, kb, ph);
    nxt = load_raw_plane<LIM, EM>(src, g, nxy, kb, kc, po);
    if constexpr (WZ) {
      const uint32_t c = here(po.c);
      const int km1 = wrap(k - 1, g.nz);
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        zm2[q] = ld_at(PW + zslot[q] * n + km1 * nxy, c);
        zp2[q] = ld_at(PW + zslot[q] * n + kc * nxy, c);
      }
      if constexpr (!GLM) {
#pragma unroll
        for (int d = 0; d < 3; ++d) nb[d] = ld_at(U + (F_BX + d) * n + kb * nxy, c);
      }
    }
#pragma unroll
    for (int q = 0; q < NF; ++q)
      if (ZL) fz[q] = L.fy[q][t];
    __syncthreads();
    if (y > 0) {
#pragma unroll
      for (int q = 0; q < NF; ++q) L.fy[q][t - M::TX] = fy[q];
    }
    if (helper && lane < M::TX + M::TY) {
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        if (lane < M::TX) L.fy[q][M::NCORE - M::TX + lane] = fe[q];
        else L.fx[q][lane - M::TX] = fe[q];
      }
    }
    if (haloer) {
      double W[9];
      bad |= !march_prim<LIM, EM>(hr, g.gamma, W);
#pragma unroll
      for (int q = 0; q < NQ; ++q) lds[q * HL::Q + HL::OFF + t] = (R)W[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      if (x == M::TX - 1) acc[q] = ((double)L.fx[q][y] - acc[q]) * idx;
      acc[q] += ((double)L.fy[q][t] - (double)fy[q]) * idy;
      if (ZL) L.fy[q][t] = fz[q];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) bn[d] = bnn[d];
    cp = M::NCORE - cp;
  }
  if (bad) atomicOr(flag, 1);
}

// ---------------------------------------------------------------------------
// WENO-Z, and PLM with GLM, on grids that the columns of the march would pad or whose
// runs would be short and solve up to half of the z-faces twice (faces_by_cells): one
// thread per cell, in storage order, solves its three lower faces from the primitives
// and stores their fluxes, and a second kernel differences them. On small grids the
// fluxes' way through memory is short (they stay in the caches).

// The lower D-face of cell (i, j, k): fluxes to FL[D], CT: its edge inputs to FW.
template <int D, int LIM, int RS, class R, int EM>
__device__ __forceinline__ void cell_face(const double* __restrict__ U,
                                          const double* __restrict__ PW, R* __restrict__ FW,
                                          const Geom& g, int i, int j, int k, int64_t c, R ch) {
  constexpr bool GLM = EM == 2;
  constexpr int NW = GLM ? 9 : 7, NF = GLM ? 9 : 5, T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  constexpr int slot[9] = {0, 1 + D, 1 + T1, 1 + T2, 5 + T1, 5 + T2, 4, 5 + D, 8};
  const int64_t n = g.n;
  // all values of the stencil before a scheduling barrier: one wait per face. (32-bit
  // byte offsets, the grid is small: 64 x 52 x 175 with GLM 1381 -> 1301 us a pass)
  constexpr int S = LIM == 2 ? 3 : 2;
  double v[NW][2 * S];
#pragma unroll
  for (int s = 0; s < 2 * S; ++s) {
    const int o = s - S;
    const uint32_t cs =
        8u * (uint32_t)lin(g, D == 0 ? wrap(i + o, g.nx) : i, D == 1 ? wrap(j + o, g.ny) : j,
                           D == 2 ? wrap(k + o, g.nz) : k);
    const uint32_t off = here(cs);
#pragma unroll
    for (int q = 0; q < NW; ++q) v[q][s] = ld_at(PW + slot[q] * n, off);
  }
  const uint32_t co = here(8u * (uint32_t)c);
  const double bn = GLM ? 0.0 : ld_at(U + (F_BX + D) * n, co);
  __builtin_amdgcn_sched_barrier(0);
  R wl[NW], wr[NW], psi = R(0), fpsi = R(0), F[NF];
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    if constexpr (LIM == 2) {
      wl[q] = wenoz_upper(v[q][0], v[q][1], v[q][2], v[q][3], v[q][4]);
      wr[q] = wenoz_upper(v[q][5], v[q][4], v[q][3], v[q][2], v[q][1]);
    } else {
      plm_pair<LIM, R>((R)v[q][0], (R)v[q][1], (R)v[q][2], (R)v[q][3], wl[q], wr[q]);
    }
  }
  RiemannOut<R> o;
  face_solve<RS, R, EM>((R)g.gamma, wl, wr, (R)bn, ch, o, psi, fpsi);
  cell_fluxes<D, EM>(o, psi, fpsi, F);
  R* const fw = FW + (int64_t)D * (GLM ? 9 : (int)NSLOT) * n;
  const uint32_t fo = co / (uint32_t)(8 / sizeof(R));
  auto put = [&](int q, R v) {
    *reinterpret_cast<R*>(reinterpret_cast<char*>(fw + q * n) + fo) = v;
  };
#pragma unroll
  for (int q = 0; q < NF; ++q) put(q, F[q]);
  if constexpr (!GLM) {
    put(S_AP, EM == 1 ? o.om : o.ap);
    put(S_AM, EM == 1 ? o.dl : o.am);
    if constexpr (EM == 1) put(S_DR, o.dr);
    put(S_V1, o.v1);
    put(S_V2, o.v2);
  }
}

// Cell of this thread: kBlock consecutive cells per workgroup, in the XCD-grouped
// order (rows three away stay in an XCD's L2).
__device__ __forceinline__ bool linear_cell(const Geom& g, int& i, int& j, int& k, int64_t& c) {
  const uint32_t t = xcd_grouped(blockIdx.x, gridDim.x) * (uint32_t)kBlock + threadIdx.x;
  if ((int64_t)t >= g.n) return false;
  const uint32_t r = t / (uint32_t)g.nx;
  i = (int)(t - r * (uint32_t)g.nx);
  k = (int)(r / (uint32_t)g.ny);
  j = (int)(r - (uint32_t)k * (uint32_t)g.ny);
  c = t;
  return true;
}

template <int LIM, int RS, class R, int EM>
__global__ __launch_bounds__(kBlock) void k_faces_cells(const double* __restrict__ U,
                                                        const double* __restrict__ PW,
                                                        double* __restrict__ FW, Geom g,
                                                        double ch0, double dt,
                                                        const double* __restrict__ dtp) {
  int i, j, k;
  int64_t c;
  if (!linear_cell(g, i, j, k, c)) return;
  const R ch = EM == 2 ? (R)(ch0 / (dtp ? *dtp : dt)) : R(0);
  R* const fw = stored<R>(FW);
  cell_face<0, LIM, RS, R, EM>(U, PW, fw, g, i, j, k, c, ch);
  cell_face<1, LIM, RS, R, EM>(U, PW, fw, g, i, j, k, c, ch);
  cell_face<2, LIM, RS, R, EM>(U, PW, fw, g, i, j, k, c, ch);
}

// The update of the cell-averaged fields from the fluxes (stage: as rk_coef, U0 = U
// where it does not use it; psi times decay).
template <class R, int EM>
__global__ __launch_bounds__(kBlock) void k_update_cells(const double* __restrict__ U,
                                                         const double* U0, double* out,
                                                         const double* __restrict__ FW, Geom g,
                                                         int stage, double dt,
                                                         const double* __restrict__ dtp,
                                                         double decay) {
  constexpr bool GLM = EM == 2;
  constexpr int NF = GLM ? 9 : 5;
  int i, j, k;
  int64_t c;
  if (!linear_cell(g, i, j, k, c)) return;
  const int64_t n = g.n;
  const int64_t xp = lin(g, wrap(i + 1, g.nx), j, k), yp = lin(g, i, wrap(j + 1, g.ny), k);
  const int64_t zp = lin(g, i, j, wrap(k + 1, g.nz));
  const RkCoef rk = rk_coef(stage, stage == 0 ? 0.0 : (dtp ? *dtp : dt));
  const double idx = 1.0 / g.dx, idy = 1.0 / g.dy, idz = 1.0 / g.dz;
  const R* fx = stored<R>(FW);
  const R* fy = fx + (int64_t)(GLM ? 9 : (int)NSLOT) * n;
  const R* fz = fy + (int64_t)(GLM ? 9 : (int)NSLOT) * n;
  const bool two = stage == 2 || stage == 4 || stage == 5;
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    const double L = -(((double)fx[q * n + xp] - (double)fx[q * n + c]) * idx +
                       ((double)fy[q * n + yp] - (double)fy[q * n + c]) * idy +
                       ((double)fz[q * n + zp] - (double)fz[q * n + c]) * idz);
    const double u = U[q * n + c];
    double v = rk_apply(rk, u, two ? U0[q * n + c] : u, L);
    if (GLM && q == 8) v *= decay;
    out[q * n + c] = v;
  }
}

template <int LIM, int RS, class R, int EM>
void cells_impl(const StageArgs& a) {
  const unsigned nb = (unsigned)((a.g.n + kBlock - 1) / kBlock);
  MHD_TIMED(a, K_FACES,
            hipLaunchKernelGGL((k_faces_cells<LIM, RS, R, EM>), dim3(nb), dim3(kBlock), 0, a.stream, a.U,
                               a.PW, a.FW, a.g, a.cfl * a.glm_dmin, a.dt, a.dtp));
  MHD_TIMED(a, K_UPDATE,
            hipLaunchKernelGGL((k_update_cells<R, EM>), dim3(nb), dim3(kBlock), 0, a.stream, a.U,
                               a.U0 ? a.U0 : a.U, a.out, a.FW, a.g, a.stage, a.dt, a.dtp,
                               (a.stage == 2 || a.stage == 5) ? a.glm_decay : 1.0));
}

template <int LIM, int RS, class R, int EM>
void faces_impl(const StageArgs& a, const double* cflp, int npart) {
  const MarchGrid mg = march_grid(a.g, a.limiter);
  hipLaunchKernelGGL((k_faces_march<LIM, RS, R, EM>), dim3(mg.nblocks), dim3(kBlock), 0, a.stream,
                     a.U, a.PW, a.U0 ? a.U0 : a.U, a.out, a.FW, a.g, mg, a.stage, a.dt, a.dtp,
                     a.flag, a.keep_rhs ? a.FW : nullptr, a.cfl * a.glm_dmin,
                     (a.stage == 2 || a.stage == 5) ? a.glm_decay : 1.0, cflp, npart, a.cfl,
                     a.dt_out);
}
template <int LIM, int RS, class R>
void faces_em(const StageArgs& a, const double* cflp, int npart) {
  if (a.glm) faces_impl<LIM, RS, R, 2>(a, cflp, npart);
  else if (a.emf == 1) faces_impl<LIM, RS, R, 1>(a, cflp, npart);
  else faces_impl<LIM, RS, R, 0>(a, cflp, npart);
}
template <int LIM, int RS>
void faces_prec(const StageArgs& a, const double* cflp, int npart) {
  if constexpr (LIM == 2) faces_em<LIM, RS, double>(a, cflp, npart);
  else if (a.precision == 1) faces_em<LIM, RS, float>(a, cflp, npart);
  else faces_em<LIM, RS, double>(a, cflp, npart);
}

}  // namespace

// Planes per run: a run costs about a plane more (its prologue and the z-faces above
// it; less of one with WENO-Z, whose primitives are there), a longer one leaves fewer
// workgroups, counted as two to each of the 256 CUs (in mixed precision, and in FP64
// for HLL with PLM and CT, three fit; the rule does not tell them apart). The power of two up to 16 that
// minimises (runs per slot + 0.4) (planes + extra), the longer of two that differ by
// less than 2 %. Measured, us a launch: 32^3 1: 17, 2: 23, 4: 38; 64^3 1: 46, 2: 40, 4:
// 45; 150 x 131 x 97 1: 243, 2: 214, 4: 193, 8: 185; 60 x 50 x 40 WENO-Z 1: 51, 2: 56,
// 4: 59; 60 x 64 x 27 WENO-Z with GLM 1: 41, 2: 44, 4: 69; 256^3 4: 1742, 8: 1654, 16:
// 1608, 32: 1601.
MarchGrid march_grid(const Geom& g, int limiter, double* turns) {
  MarchGrid mg;
  mg.ntx = (g.nx + March::TX - 1) / March::TX;
  mg.nty = (g.ny + March::TY - 1) / March::TY;
  const double extra = limiter == 2 ? 0.6 : 1.0;
  double best = 0.0;
  mg.lz = 0;
  for (int lz = 16; lz >= 1; lz /= 2) {
    const int64_t nb = (int64_t)mg.ntx * mg.nty * ((g.nz + lz - 1) / lz);
    const double t = ((double)nb / 512.0 + 0.4) * (lz + extra);
    if (mg.lz == 0 || t < 0.98 * best) {
      best = t;
      mg.lz = lz;
    }
  }
  if (turns) *turns = best;
  mg.nzc = (g.nz + mg.lz - 1) / mg.lz;
  mg.nblocks = (unsigned)mg.ntx * (unsigned)mg.nty * (unsigned)mg.nzc;
  return mg;
}

// Which of the two is estimated to take less, in microseconds a stage. march: its
// turns, which count its padding; cells: latency, the L2, or the memory. Fitted to 120
// grids from 4^3 to 4 million cells, cubes, slabs and bars, with HLL and mixed
// precision, which move both sides alike; the worse one is taken near the line only
// (PLM 15 to 25 % at most, 1 % on average; WENO-Z 5 %, 0.1 %). Measured, march / cells:
// PLM with GLM 4 x 4 x 4000 110 / 22, 33 x 9 x 861 118 / 52, 48^3 37 / 31, 64^3 38 / 49,
// 128^3 227 / 466; WENO-Z 48^3 68 / 51, 100^3 340 / 282, 112^3 392 / 376, 128^3 507 /
// 583, 4 x 4 x 125000 4937 / 1251; with GLM 48^3 59 / 40, 100 x 40 x 100 130 / 111, 128^3
// 435 / 568.
bool faces_by_cells(const Geom& g, int limiter, bool glm) {
  if (limiter != 2 && !glm) return false;     // PLM with CT marches
  if (g.n >= (int64_t)1 << 29) return false;  // 32-bit byte offsets
  struct {
    double march, turn, cells, l2, mem;
  } t = {3.5, 10.5, 17.0, 0.12, 0.22};
  if (limiter == 2 && glm) t = {8.0, 22.0, 0.0, 0.0, 0.28};
  else if (limiter == 2) t = {12.0, 22.0, 0.0, 0.0, 0.25};
  const double k = 1e-3 * (double)g.n;
  double turns;
  march_grid(g, limiter, &turns);
  return std::max(t.cells + t.l2 * k, t.mem * k) < t.march + t.turn * turns;
}

namespace {

template <int RS>
void cells_rs(const StageArgs& a) {
  const bool mixed = a.precision == 1;
  if (a.limiter == 2) {
    if (a.glm) cells_impl<2, RS, double, 2>(a);
    else if (a.emf == 1) cells_impl<2, RS, double, 1>(a);
    else cells_impl<2, RS, double, 0>(a);
  } else if (a.limiter == 1) {
    if (mixed) cells_impl<1, RS, float, 2>(a);
    else cells_impl<1, RS, double, 2>(a);
  } else {
    if (mixed) cells_impl<0, RS, float, 2>(a);
    else cells_impl<0, RS, double, 2>(a);
  }
}

}  // namespace

void launch_faces_cells(const StageArgs& a) {
  if (a.riemann == 0) cells_rs<0>(a);
  else cells_rs<1>(a);
}

void launch_faces_march(const StageArgs& a, const double* cflp, int npart) {
  if (a.limiter == 2) {
    if (a.riemann == 0) faces_prec<2, 0>(a, cflp, npart);
    else faces_prec<2, 1>(a, cflp, npart);
  } else if (a.limiter == 0) {
    if (a.riemann == 0) faces_prec<0, 0>(a, cflp, npart);
    else faces_prec<0, 1>(a, cflp, npart);
  } else {
    if (a.riemann == 0) faces_prec<1, 0>(a, cflp, npart);
    else faces_prec<1, 1>(a, cflp, npart);
  }
}

}  // namespace mhd
