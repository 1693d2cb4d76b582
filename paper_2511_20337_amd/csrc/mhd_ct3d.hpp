// 3D constrained transport, the second kernel of a stage: the edge EMFs from the
// face kernel's edge inputs, and from them the update of the staggered field.
//
// A workgroup owns a column of up to 31 x 7 cells and walks a run of planes. Its
// 32 x 8 threads form the three EMFs on the lower edges of their cell, the last
// column's and the last row's once more than their owner does, so that the
// differences along x and y come from LDS and those along z from the thread's
// own EMFs of the plane before: the EMFs never go to memory. Per plane every input
// is loaded once into LDS, with the halo (up to three values a thread), and read
// from there by the threads around; v and b that E_x and E_y reconstruct along z,
// and the coefficients one plane down, ride in registers. The next plane's loads
// are on the way while this one's EMFs are formed.
//
// What bounds it: HBM (256^3 FP64 with U0: 227 B per cell counted, 168 of them
// needed, 4.6 TB/s; a large copy reaches 4.76). Measured against the two kernels it replaces (EMFs to
// memory, 0.65 ms; the update that read them back, 0.31 ms, 0.56 where it also
// finished the cell fields): 256^3 0.79 ms a stage, 384^3 mixed 2.68 -> 1.73, 352^3
// UCT-HLLD 2.65 -> 2.25. Choices:
//  - Inputs through LDS: with every thread loading its neighbours' values itself (47
//    loads a plane instead of 18) the vector cache was the bound, 1.22 ms at 256^3.
//  - Workgroups in the XCD-grouped order, neighbours on one L2: 352^3 2.50 -> 2.27.
//  - Results stored a plane later, before the loads that are waited for next: no
//    gain. Three waves per SIMD in FP64 spill.
#pragma once
#include "mhd_device.hpp"
#include "mhd_grid.hpp"
#include "mhd_kernels.hpp"

namespace mhd {

namespace {

struct CtCol {
  static constexpr int TX = 32, TY = 8, NT = TX * TY;
};

// The coefficients of one face the edge average takes: alpha+ and alpha-
// (EM 0), or the UCT-HLLD weight and diffusion coefficients (EM 1).
template <int EM, class R>
struct FaceCoef {
  R c[EM == 1 ? 3 : 2];
};

// The value at byte offset off (a lane's) of the uniform base b.
template <class T>
__device__ __forceinline__ T ld_as(const T* __restrict__ b, uint32_t off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(b) + off);
}

template <class T>
__device__ __forceinline__ void st_as(T* b, uint32_t off, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(b) + off) = v;
}

template <int EM, class R>
__device__ __forceinline__ FaceCoef<EM, R> face_coef(const R* __restrict__ f, int64_t n,
                                                     uint32_t off) {
  FaceCoef<EM, R> o;
  o.c[0] = ld_as(f + S_AP * n, off);
  o.c[1] = ld_as(f + S_AM * n, off);
  if constexpr (EM == 1) o.c[2] = ld_as(f + S_DR * n, off);
  return o;
}

// Edge EMF from the coefficients of the a-faces (below the edge along B,
// then the cell's own) and b-faces, and the reconstructed values.
template <int LIM, int EM, class R>
__device__ __forceinline__ R emf_from(const FaceCoef<EM, R>& am, const FaceCoef<EM, R>& ac,
                                      const FaceCoef<EM, R>& bm, const FaceCoef<EM, R>& bc,
                                      const R* vbA, const R* bB, const R* vaB, const R* bA) {
  if constexpr (EM == 1)
    return emf_core_hlld<LIM, R>(am.c[0], ac.c[0], am.c[1], ac.c[1], am.c[2], ac.c[2], bm.c[0],
                                 bc.c[0], bm.c[1], bc.c[1], bm.c[2], bc.c[2], vbA, bB, vaB, bA);
  else
    return emf_core<LIM, R>(am.c[0], ac.c[0], am.c[1], ac.c[1], bm.c[0], bc.c[0], bm.c[1],
                            bc.c[1], vbA, bB, vaB, bA);
}

// One plane of the column's EMF inputs in LDS, each over the neighbours that the
// edge values and averages read: cells -2 .. +1 along x (v_x on z- and y-faces,
// b_y), along y (v_y on z- and x-faces, b_x) or both (b_z), the cell below along x
// (coefficients of the y-faces), y (x-faces) or both (z-faces).
template <int EM, class R>
struct CtLds {
  static constexpr int NC = EM == 1 ? 3 : 2, TX = CtCol::TX, TY = CtCol::TY;
  R xz[TY][TX + 3], xy[TY][TX + 3], by[TY][TX + 3];
  R yz[TY + 3][TX], yx[TY + 3][TX], bx[TY + 3][TX];
  R bz[TY + 3][TX + 3];
  R zc[NC][TY + 1][TX + 1], yc[NC][TY][TX + 1], xc[NC][TY + 1][TX];
  R e[2][3][CtCol::NT];  // the EMFs of two planes
};

// A thread's share of the next plane: its cell's values (v_z on the y- and
// x-face and b_y, b_x one plane up) and up to three of the halo.
template <int EM, class R>
struct CtPlane {
  R zyp, zxp, xz, xy, yz, yx;
  double byp, bxp, bz;
  FaceCoef<EM, R> yc, xc, zc;
  double hb;
  R hv, hc;
};

// stage as rk_coef; TWO: one that reads U0. 3: no state. LB != nullptr: L of the
// staggered field into LB[3][n].
template <int LIM, class R, int EM, bool TWO>
__global__ __launch_bounds__(CtCol::NT) __attribute__((amdgpu_waves_per_eu(2)))
void k_ct_march(const double* __restrict__ U, const double* U0, double* out,
                const double* __restrict__ FW, double* __restrict__ LB, Geom g, MarchGrid mg,
                int stage, double dt, const double* __restrict__ dtp) {
  constexpr int TX = CtCol::TX, TY = CtCol::TY, NT = CtCol::NT;
  constexpr int NC = CtLds<EM, R>::NC;
  __shared__ CtLds<EM, R> L;
  R* const lds = &L.xz[0][0];
  const unsigned b = xcd_grouped(blockIdx.x, gridDim.x);
  const int tx = (int)(b % (unsigned)mg.ntx);
  const unsigned r = b / (unsigned)mg.ntx;
  const int ty = (int)(r % (unsigned)mg.nty);
  const int zc = (int)(r / (unsigned)mg.nty);
  // columns of equal width (but for the last)
  const int wx = (g.nx + mg.ntx - 1) / mg.ntx, wy = (g.ny + mg.nty - 1) / mg.nty;
  const int t = (int)threadIdx.x, x = t % TX, y = t / TX;
  const int i0 = tx * wx, j0 = ty * wy;
  const bool owner = x < wx && y < wy && i0 + x < g.nx && j0 + y < g.ny;
  const int k0 = zc * mg.lz;
  const int k1 = min(k0 + mg.lz, g.nz);
  const int64_t n = g.n, nxy = (int64_t)g.nx * g.ny;
  const double h = (stage == 0 || stage == 3) ? 0.0 : uni(dtp ? *dtp : dt);
  const RkCoef rk = rk_coef(stage, h);
  const double idx = uni(1.0 / g.dx), idy = uni(1.0 / g.dy), idz = uni(1.0 / g.dz);
  const R* const fx0 = stored<R>(FW);
  const R* const fy0 = fx0 + (int64_t)NSLOT * n;
  const R* const fz0 = fx0 + (int64_t)2 * NSLOT * n;
  const double* const bx0 = U + F_BX * n;
  const double* const by0 = U + F_BY * n;
  const double* const bz0 = U + F_BZ * n;
  // byte offset in a plane of one field of R (SD times that in one of the
  // state): 32 bits, a plane holds fewer than 2^29 cells
  constexpr uint32_t SR = sizeof(R), SD = 8 / sizeof(R);
  // (a remainder only where the grid is smaller than what its last column reaches)
  const bool wide = (mg.ntx - 1) * wx + TX < 2 * g.nx && (mg.nty - 1) * wy + TY < 2 * g.ny;
  auto cell = [&](int hx, int hy) {
    const int i = i0 + hx, j = j0 + hy;
    return (uint32_t)(wide ? wrap(j, g.ny) * g.nx + wrap(i, g.nx)
                           : wrap_any(j, g.ny) * g.nx + wrap_any(i, g.nx));
  };
  const uint32_t oc = cell(x, y) * SR;
  // The halo: 240 values of the field, 240 velocities, 80 of each coefficient,
  // one of each kind per thread: where from and where to.
  const double* hb;
  const R *hv, *hc;
  int lb, lv, lc;
  {
    // cell e of the three columns beside the tile, or of the three rows
    auto col = [](int e, int& hx, int& hy) {
      hx = (e / TY < 2) ? e / TY - 2 : TX;
      hy = e % TY;
    };
    auto row = [](int e, int& hx, int& hy) {
      hx = e % TX;
      hy = (e / TX < 2) ? e / TX - 2 : TY;
    };
    constexpr int X = 3 * TY, Y = 3 * TX;
    int hx, hy;
    int e = min(t, 2 * (X + Y) - 1);
    // 0: b_y and xz beside the tile, 1: b_z and xy; 2: b_x and yz along it, 3: b_z and yx
    const int kind = e < X ? 0 : e < 2 * X ? 1 : e < 2 * X + Y ? 2 : 3;
    if (kind < 2) col(kind ? e - X : e, hx, hy);
    else row(kind == 2 ? e - 2 * X : e - 2 * X - Y, hx, hy);
    uint32_t c = cell(hx, hy);
    hb = (kind == 0 ? by0 : kind == 2 ? bx0 : bz0) + c;
    hv = (kind == 0 ? fz0 + S_V1 * n : kind == 1 ? fy0 + S_V2 * n
          : kind == 2 ? fz0 + S_V2 * n : fx0 + S_V1 * n) + c;
    lb = (int)((kind == 0 ? &L.by[hy][hx + 2] : kind == 2 ? &L.bx[hy + 2][hx]
                                                          : &L.bz[hy + 2][hx + 2]) - lds);
    lv = (int)((kind == 0 ? &L.xz[hy][hx + 2] : kind == 1 ? &L.xy[hy][hx + 2]
                : kind == 2 ? &L.yz[hy + 2][hx] : &L.yx[hy + 2][hx]) - lds);
    // coefficients: of the z- and y-faces to the left, of the z- and x-faces below
    constexpr int C = 2 * (TX + TY);
    e = min(t, NC * C - 1);
    const int m = e / C;
    e -= m * C;
    const int slot = m == 0 ? S_AP : m == 1 ? S_AM : S_DR;
    const int k = e < TY ? 0 : e < 2 * TY ? 1 : e < 2 * TY + TX ? 2 : 3;
    hx = k < 2 ? -1 : (e - 2 * TY) % TX;
    hy = k < 2 ? e % TY : -1;
    c = cell(hx, hy);
    hc = (k == 1 ? fy0 : k == 3 ? fx0 : fz0) + slot * n + c;
    lc = (int)((k == 1 ? &L.yc[m][hy][0] : k == 3 ? &L.xc[m][0][hx]
                                                  : &L.zc[m][hy + 1][hx + 1]) - lds);
  }
  const bool hasv = t < 6 * (TX + TY), hasc = t < NC * 2 * (TX + TY);
  // planes k-2 .. k+1 of this column: v_z on y-faces and b_y (E_x), v_z on
  // x-faces and b_x (E_y); the coefficients of y- and x-faces on planes k-1, k
  R yv[4], yb[4], xv[4], xb[4];
  FaceCoef<EM, R> yc[2], xc[2];
  double by = 0.0, bx = 0.0;  // b_x, b_y of the own cell, plane k
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int64_t p = wrap(k0 - 2 + s, g.nz) * nxy;
    yv[s] = ld_as(fy0 + S_V1 * n + p, oc);
    xv[s] = ld_as(fx0 + S_V2 * n + p, oc);
    by = ld_as(by0 + p, oc * SD);
    bx = ld_as(bx0 + p, oc * SD);
    yb[s] = (R)by;
    xb[s] = (R)bx;
  }
  {
    const int64_t p = wrap(k0 - 1, g.nz) * nxy;
    yc[0] = face_coef<EM, R>(fy0 + p, n, oc);
    xc[0] = face_coef<EM, R>(fx0 + p, n, oc);
  }
  CtPlane<EM, R> q;
  auto load = [&](int k) {
    const int64_t p = wrap(k, g.nz) * nxy, pp = wrap(k + 1, g.nz) * nxy;
    const R *fx = fx0 + p, *fy = fy0 + p, *fz = fz0 + p;
    const uint32_t c = here(oc);
    q.xz = ld_as(fz + S_V1 * n, c);
    q.yz = ld_as(fz + S_V2 * n, c);
    q.xy = ld_as(fy + S_V2 * n, c);
    q.yx = ld_as(fx + S_V1 * n, c);
    q.zc = face_coef<EM, R>(fz, n, c);
    q.yc = face_coef<EM, R>(fy, n, c);
    q.xc = face_coef<EM, R>(fx, n, c);
    q.bz = ld_as(bz0 + p, c * SD);
    q.hb = hb[p];
    q.hv = hv[p];
    q.hc = hc[p];
    q.zyp = ld_as(fy0 + S_V1 * n + pp, c);
    q.zxp = ld_as(fx0 + S_V2 * n + pp, c);
    q.byp = ld_as(by0 + pp, c * SD);
    q.bxp = ld_as(bx0 + pp, c * SD);
  };
  // of plane k - 1: its EMFs and its field at the own cell
  double exm = 0.0, eym = 0.0, ezm = 0.0, bxm = 0.0, bym = 0.0, bzm = 0.0;
  load(k0);
  for (int k = k0;; ++k) {
    if (k > k0) __syncthreads();  // plane k - 1 has been read
    L.xz[y][x + 2] = q.xz;
    L.xy[y][x + 2] = q.xy;
    L.by[y][x + 2] = (R)by;
    L.yz[y + 2][x] = q.yz;
    L.yx[y + 2][x] = q.yx;
    L.bx[y + 2][x] = (R)bx;
    L.bz[y + 2][x + 2] = (R)q.bz;
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      L.zc[m][y + 1][x + 1] = q.zc.c[m];
      L.yc[m][y][x + 1] = q.yc.c[m];
      L.xc[m][y + 1][x] = q.xc.c[m];
    }
    if (hasv) {
      lds[lb] = (R)q.hb;
      lds[lv] = q.hv;
    }
    if (hasc) lds[lc] = q.hc;
    yc[1] = q.yc;
    xc[1] = q.xc;
    yv[3] = q.zyp;
    xv[3] = q.zxp;
    const double bz = here(q.bz), bxp = here(q.bxp), byp = here(q.byp);
    yb[3] = (R)byp;
    xb[3] = (R)bxp;
    __syncthreads();
    // What the update of plane k - 1 reads, then the next plane's inputs (both by
    // every thread, in no branch, so that the wait for the former counts the
    // latter and leaves them on the way).
    const int64_t p = wrap(k - 1, g.nz) * nxy;
    double u0x = 0.0, u0y = 0.0, u0z = 0.0;
    if constexpr (TWO) {
      const uint32_t c = here(oc) * SD;
      u0x = ld_as(U0 + F_BX * n + p, c);
      u0y = ld_as(U0 + F_BY * n + p, c);
      u0z = ld_as(U0 + F_BZ * n + p, c);
    }
    __builtin_amdgcn_sched_barrier(0);
    load(k + 1);
    __builtin_amdgcn_sched_barrier(0);
    R ex, ey, ez;
    {
      FaceCoef<EM, R> zo, zi, zj, yi, xj;
      R axz[4], axy[4], aby[4], ayz[4], ayx[4], abx[4], azx[4], azy[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        axz[s] = L.xz[y][x + s];
        axy[s] = L.xy[y][x + s];
        aby[s] = L.by[y][x + s];
        ayz[s] = L.yz[y + s][x];
        ayx[s] = L.yx[y + s][x];
        abx[s] = L.bx[y + s][x];
        azx[s] = L.bz[y + 2][x + s];
        azy[s] = L.bz[y + s][x + 2];
      }
#pragma unroll
      for (int m = 0; m < NC; ++m) {
        zo.c[m] = L.zc[m][y + 1][x + 1];
        zi.c[m] = L.zc[m][y + 1][x];
        zj.c[m] = L.zc[m][y][x + 1];
        yi.c[m] = L.yc[m][y][x];
        xj.c[m] = L.xc[m][y][x];
      }
      // E_x: (A, B) = (y, z); a-faces are y-faces, b-faces z-faces
      ex = emf_from<LIM, EM, R>(yc[0], yc[1], zj, zo, ayz, azy, yv, yb);
      // E_y: (A, B) = (z, x); a-faces are z-faces, b-faces x-faces
      ey = emf_from<LIM, EM, R>(zi, zo, xc[0], xc[1], xv, xb, axz, azx);
      // E_z: (A, B) = (x, y); a-faces are x-faces, b-faces y-faces
      ez = emf_from<LIM, EM, R>(xj, xc[1], yi, yc[1], axy, aby, ayx, abx);
    }
    if (k > k0 && owner) {  // plane k - 1
      const R(*e)[NT] = L.e[(k - k0 + 1) & 1];
      const uint32_t c = here(oc) * SD;
      const double L5 = -(((double)e[2][t + TX] - ezm) * idy - ((double)ey - eym) * idz);
      const double L6 = -(((double)ex - exm) * idz - ((double)e[2][t + 1] - ezm) * idx);
      const double L7 = -(((double)e[1][t + 1] - eym) * idx - ((double)e[0][t + TX] - exm) * idy);
      if (stage != 3) {
        st_as(out + F_BX * n + p, c, rk_apply(rk, bxm, u0x, L5));
        st_as(out + F_BY * n + p, c, rk_apply(rk, bym, u0y, L6));
        st_as(out + F_BZ * n + p, c, rk_apply(rk, bzm, u0z, L7));
      }
      if (LB) {
        st_as(LB + p, c, L5);
        st_as(LB + n + p, c, L6);
        st_as(LB + 2 * n + p, c, L7);
      }
    }
    if (k == k1) break;
    {  // (two buffers, two barriers a plane: no reader is left)
      R(*e)[NT] = L.e[(k - k0) & 1];
      e[0][t] = ex;
      e[1][t] = ey;
      e[2][t] = ez;
    }
    exm = (double)ex;
    eym = (double)ey;
    ezm = (double)ez;
    bxm = bx;
    bym = by;
    bzm = bz;
    bx = bxp;
    by = byp;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      yv[s] = yv[s + 1];
      yb[s] = yb[s + 1];
      xv[s] = xv[s + 1];
      xb[s] = xb[s + 1];
    }
    yc[0] = yc[1];
    xc[0] = xc[1];
  }
}

// Columns of at most 31 x 7 cells. Runs: one costs about two planes more, and the
// workgroups take turns on 2 (FP64) or 3 places per CU: the length up to 20 with
// the shortest turns in all (64^3: 4 planes, 32 us, against 36 with 2; 150 x 131 x
// 97: 20, 105 against 116 with 16; 256^3: 20, 788 against 809 with 16).
MarchGrid ct_grid(const Geom& g, int precision) {
  MarchGrid mg;
  mg.ntx = (g.nx + CtCol::TX - 2) / (CtCol::TX - 1);
  mg.nty = (g.ny + CtCol::TY - 2) / (CtCol::TY - 1);
  const int slots = precision == 1 ? 768 : 512;
  const int64_t cols = (int64_t)mg.ntx * mg.nty;
  int64_t best = 0;
  mg.lz = 0;
  for (int most = min(g.nz, 20); most >= 1; --most) {
    const int runs = (g.nz + most - 1) / most, lz = (g.nz + runs - 1) / runs;
    const int64_t t = (cols * runs + slots - 1) / slots * (lz + 2);
    if (mg.lz == 0 || t < best) {
      best = t;
      mg.lz = lz;
    }
  }
  mg.nzc = (g.nz + mg.lz - 1) / mg.lz;
  mg.nblocks = (unsigned)(cols * mg.nzc);
  return mg;
}

template <int LIM, class R, int EM>
void ct_impl(const StageArgs& a) {
  const MarchGrid mg = ct_grid(a.g, a.precision);
  const auto k = (a.stage == 2 || a.stage == 4 || a.stage == 5) ? k_ct_march<LIM, R, EM, true>
                                                                : k_ct_march<LIM, R, EM, false>;
  hipLaunchKernelGGL(k, dim3(mg.nblocks), dim3(CtCol::NT), 0, a.stream, a.U, a.U0, a.out, a.FW,
                     a.keep_rhs ? a.EW : nullptr, a.g, mg, a.stage, a.dt, a.dtp);
}
template <int LIM>
void ct_lim(const StageArgs& a) {
  if (a.precision == 1) {
    if (a.emf == 1) ct_impl<LIM, float, 1>(a);
    else ct_impl<LIM, float, 0>(a);
  } else {
    if (a.emf == 1) ct_impl<LIM, double, 1>(a);
    else ct_impl<LIM, double, 0>(a);
  }
}

}  // namespace

void launch_ct(const StageArgs& a) {
  if (a.limiter == 0) ct_lim<0>(a);
  else ct_lim<1>(a);  // WENO-Z takes van Leer PLM for the edge values
}

}  // namespace mhd
