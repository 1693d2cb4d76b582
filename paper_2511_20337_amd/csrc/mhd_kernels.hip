// HIP kernels of the ideal-MHD step for gfx950, and their launchers.
//
// One stage in 3D with CT is two launches: the z-marching face kernel of
// mhd_faces3d.hpp, which finishes the cell-averaged fields, and that of mhd_ct3d.hpp,
// the upwind CT EMFs on the cells' edges and the update of the staggered field. GLM
// stages are the face kernel alone; WENO-Z ones recover every cell's primitives
// first (k_prim). In 2D a stage is one kernel (mhd_stage2d.hpp), except for the
// adjoint's, which keep their records. The CFL time step is a per-cell minimum
// reduced with wave64 shuffles and a block LDS step into per-block partials (by
// a kernel of the step itself where it recovers every cell's primitives anyway);
// on small grids every workgroup of the first stage reduces these, else one block
// does.
//
// Layout: state and workspace arrays are field-major SoA, x fastest, so a
// wavefront of 64 consecutive cells reads 512 contiguous bytes per field.
#include <mutex>

#include "mhd_ct3d.hpp"
#include "mhd_device.hpp"
#include "mhd_faces3d.hpp"
#include "mhd_grid.hpp"
#include "mhd_kernels.hpp"
#include "mhd_stage2d.hpp"

namespace mhd {

namespace {

// ---------------------------------------------------------------------------
// The adjoint's 2D stages, which keep their records (FP64, the HLL average; the
// steps run k_stage_2d). Faces on tiles of 16 x 16 cells, one per thread.
struct Tile {
  static constexpr int TX = 16, TY = 16;
  static constexpr int NCORE = TX * TY;  // also the workgroup size
  // cross-shaped halo: two cells below and one above the tile along each axis
  static constexpr int HX = 3 * TY, HY = 3 * TX;
  static constexpr int NPRIM = NCORE + HX + HY;
};

// EMF and update on row tiles: a wavefront covers 64 consecutive cells of one
// row (512 contiguous bytes per field).
struct RowTile {
  static constexpr int TX = 64, TY = 4;
  static constexpr int NT = TX * TY;  // workgroup size
};

// Tiles along x (visited fastest) and in all.
struct TileGrid {
  int ntx;
  unsigned ntiles;
};

template <class T>
TileGrid tile_grid(const Geom& g) {
  TileGrid tg;
  tg.ntx = (g.nx + T::TX - 1) / T::TX;
  tg.ntiles = (unsigned)tg.ntx * (unsigned)((g.ny + T::TY - 1) / T::TY);
  return tg;
}

// LDS slot of a tile-relative cell position (at most one coordinate outside).
__device__ __forceinline__ int pslot(int x, int y) {
  using T = Tile;
  if (x < 0 || x >= T::TX) return T::NCORE + (x < 0 ? x + 2 : 2) * T::TY + y;
  if (y < 0 || y >= T::TY) return T::NCORE + T::HX + (y < 0 ? y + 2 : 2) * T::TX + x;
  return y * T::TX + x;
}

// Inverse of pslot for the load loop.
__device__ __forceinline__ void pslot_pos(int e, int& x, int& y) {
  using T = Tile;
  if (e < T::NCORE) {
    x = e % T::TX;
    y = e / T::TX;
  } else if (e < T::NCORE + T::HX) {
    const int s = (e - T::NCORE) / T::TY;
    x = (s == 2) ? T::TX : s - 2;
    y = (e - T::NCORE) % T::TY;
  } else {
    const int s = (e - T::NCORE - T::HX) / T::TX;
    x = (e - T::NCORE - T::HX) % T::TX;
    y = (s == 2) ? T::TY : s - 2;
  }
}

// The lower D-face of the tile cell (x, y) from LDS primitives; its record: the
// fluxes of the cell fields (with B_z), then the EMF inputs, alpha+- and the
// HLL-weighted velocities. The normal-B flux is zero and the edge EMF replaces
// the in-plane B_t flux.
template <int D, int LIM, int RS>
__device__ __forceinline__ void tile_face(const double (*sp)[Tile::NPRIM], double bn,
                                          double* __restrict__ FW, const Geom& g, int x, int y,
                                          int64_t c) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  constexpr int slot[7] = {0, 1 + D, 1 + T1, 1 + T2, 5 + T1, 5 + T2, 4};
  int e[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) e[s] = pslot(x + (D == 0 ? s - 2 : 0), y + (D == 1 ? s - 2 : 0));
  double wl[7], wr[7];
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    const double* P = sp[slot[q]];
    plm_pair<LIM, double>(P[e[0]], P[e[1]], P[e[2]], P[e[3]], wl[q], wr[q]);
  }
  RiemannOut<double> o;
  riemann<RS, double, 0>(g.gamma, wl, wr, bn, o);
  const int64_t n = g.n;
  double* fw = FW + (int64_t)D * NSLOT * n + c;
  fw[S_RHO * n] = o.f[0];
  fw[(S_MX + D) * n] = o.f[1];
  fw[(S_MX + T1) * n] = o.f[2];
  fw[(S_MX + T2) * n] = o.f[3];
  fw[S_EN * n] = o.f[6];
  fw[S_BZ * n] = (D == 0) ? o.f[5] : o.f[4];  // B_z is t2 of x, t1 of y
  fw[S_AP * n] = o.ap;
  fw[S_AM * n] = o.am;
  fw[S_V1 * n] = o.v1;
  fw[S_V2 * n] = o.v2;
}

// Primitives of the tile and its cross halo are recovered once into LDS, then
// each thread solves the lower x- and y-face of its cell.
template <int LIM, int RS>
__global__ __launch_bounds__(Tile::NCORE) void k_faces_tiled(const double* __restrict__ U,
                                                             double* __restrict__ FW, Geom g,
                                                             TileGrid tg, int* __restrict__ flag) {
  using T = Tile;
  __shared__ double sp[8][T::NPRIM];
  const int i0 = (int)(blockIdx.x % (unsigned)tg.ntx) * T::TX;
  const int j0 = (int)(blockIdx.x / (unsigned)tg.ntx) * T::TY;
  const int x = (int)threadIdx.x % T::TX, y = (int)threadIdx.x / T::TX;
  const int i = i0 + x, j = j0 + y;
  // The normal fields of the cell's faces first (any in-bounds cell for a
  // thread outside the grid): loaded after the x-face records, waiting for
  // them would wait for those stores too.
  const int64_t c = lin(g, min(i, g.nx - 1), min(j, g.ny - 1), 0);
  const double bx = U[F_BX * g.n + c], by = U[F_BY * g.n + c];
  bool bad = false;
  for (int e = threadIdx.x; e < T::NPRIM; e += T::NCORE) {
    int ex, ey;
    pslot_pos(e, ex, ey);
    double V[8];
    bad |= !prim_at<2>(U, g, wrap_any(i0 + ex, g.nx), wrap_any(j0 + ey, g.ny), 0, V);
#pragma unroll
    for (int q = 0; q < 8; ++q) sp[q][e] = V[q];
  }
  if (bad) atomicOr(flag, 1);
  __syncthreads();
  if (i < g.nx && j < g.ny) {
    tile_face<0, LIM, RS>(sp, bx, FW, g, x, y, c);
    tile_face<1, LIM, RS>(sp, by, FW, g, x, y, c);
  }
}

// E_z at the lower corner of cell (i, j) from the face records (the upwind
// average with the HLL bounds).
template <int LIM>
__device__ __forceinline__ double emf_z(const double* __restrict__ U,
                                        const double* __restrict__ FW, const Geom& g, int i,
                                        int j) {
  const int64_t n = g.n, c = lin(g, i, j, 0);
  const double* fx = FW;
  const double* fy = FW + (int64_t)NSLOT * n;
  const int64_t jm = shifted<1>(g, i, j, 0, -1);  // x-face below the corner
  const int64_t im = shifted<0>(g, i, j, 0, -1);  // y-face left of the corner
  const int64_t i2 = shifted<0>(g, i, j, 0, -2), i1 = shifted<0>(g, i, j, 0, 1);
  const int64_t j2 = shifted<1>(g, i, j, 0, -2), j1 = shifted<1>(g, i, j, 0, 1);
  const double* vx = fy + S_V2 * n;  // v_x on y-faces
  const double* vy = fx + S_V1 * n;  // v_y on x-faces
  const double* by = U + F_BY * n;
  const double* bx = U + F_BX * n;
  const double wv[4] = {vx[i2], vx[im], vx[c], vx[i1]};
  const double wb[4] = {by[i2], by[im], by[c], by[i1]};
  const double sv[4] = {vy[j2], vy[jm], vy[c], vy[j1]};
  const double sb[4] = {bx[j2], bx[jm], bx[c], bx[j1]};
  return emf_core<LIM, double>(fx[S_AP * n + jm], fx[S_AP * n + c], fx[S_AM * n + jm],
                               fx[S_AM * n + c], fy[S_AP * n + im], fy[S_AP * n + c],
                               fy[S_AM * n + im], fy[S_AM * n + c], wv, wb, sv, sb);
}

template <int LIM>
__global__ __launch_bounds__(RowTile::NT) void k_emf(const double* __restrict__ U,
                                                     const double* __restrict__ FW,
                                                     double* __restrict__ EW, Geom g,
                                                     TileGrid tg) {
  const int i = (int)(blockIdx.x % (unsigned)tg.ntx) * RowTile::TX + (int)threadIdx.x % RowTile::TX;
  const int j = (int)(blockIdx.x / (unsigned)tg.ntx) * RowTile::TY + (int)threadIdx.x / RowTile::TX;
  if (i < g.nx && j < g.ny) EW[2 * g.n + lin(g, i, j, 0)] = emf_z<LIM>(U, FW, g, i, j);
}

// EMF and update in one kernel: each thread forms E_z at the lower corner of its
// cell (any thread past the grid at the periodic image of that corner), threads
// 0..68 also the corners of the row above and of the column to the right, all
// into LDS behind one barrier; then each cell of the grid is updated, and its own
// E_z is stored for the records. Stage 1, or 4 (the second of SSP-RK3).
template <int LIM, int STAGE>
__global__ __launch_bounds__(RowTile::NT) void k_emf_update_2d(const double* __restrict__ U,
                                                               const double* U0, double* out,
                                                               const double* __restrict__ FW,
                                                               double* __restrict__ EW, Geom g,
                                                               TileGrid tg, double dt) {
  constexpr int TX = RowTile::TX, TY = RowTile::TY, SX = TX + 1;
  __shared__ double ezs[(TY + 1) * SX];
  const int i0 = (int)(blockIdx.x % (unsigned)tg.ntx) * TX;
  const int j0 = (int)(blockIdx.x / (unsigned)tg.ntx) * TY;
  const int x = (int)threadIdx.x % TX, y = (int)threadIdx.x / TX;
  const int i = i0 + x, j = j0 + y;
  const bool inside = i < g.nx && j < g.ny;
  const int64_t n = g.n;
  {
    const double ez = emf_z<LIM>(U, FW, g, wrap_any(i, g.nx), wrap_any(j, g.ny));
    ezs[y * SX + x] = ez;
    if (inside) EW[2 * n + lin(g, i, j, 0)] = ez;
  }
  if (threadIdx.x < TX + TY + 1) {
    const int h = (int)threadIdx.x;
    const int hx = (h < TX) ? h : TX, hy = (h < TX) ? TY : h - TX;  // h = TX + TY: the corner
    ezs[hy * SX + hx] = emf_z<LIM>(U, FW, g, wrap_any(i0 + hx, g.nx), wrap_any(j0 + hy, g.ny));
  }
  __syncthreads();
  if (!inside) return;
  const int64_t c = lin(g, i, j, 0);
  const int64_t xp = lin(g, wrap(i + 1, g.nx), j, 0);
  const int64_t yp = lin(g, i, wrap(j + 1, g.ny), 0);
  const double idx = 1.0 / g.dx, idy = 1.0 / g.dy;
  const double* fx = FW;
  const double* fy = fx + (int64_t)NSLOT * n;
  double L[8];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const double acc =
        (fx[q * n + xp] - fx[q * n + c]) * idx + (fy[q * n + yp] - fy[q * n + c]) * idy;
    L[q == 5 ? 7 : q] = -acc;
  }
  const double ezc = ezs[y * SX + x];
  L[5] = -((ezs[(y + 1) * SX + x] - ezc) * idy);
  L[6] = (ezs[y * SX + x + 1] - ezc) * idx;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const double v = U[q * n + c] + dt * L[q];
    out[q * n + c] = (STAGE == 1) ? v : (3.0 * U0[q * n + c] + v) / 4.0;
  }
}

// Primitives (rho, v_x, v_y, v_z, p, B_x, B_y, B_z, psi) of cell c of a GLM
// state; false for an unphysical one.
__device__ __forceinline__ bool glm_prim(const double* __restrict__ U, int64_t n, int64_t c,
                                         double gamma, double* V) {
  RawCell r;  // (the mean of two equal faces is the cell's field, exactly)
#pragma unroll
  for (int q = 0; q < 8; ++q) r.u[q] = U[q * n + c];
  r.bxp = r.u[5];
  r.byp = r.u[6];
  r.bzp = r.u[7];
  V[8] = U[8 * n + c];
  return prim_from_raw<3>(r, gamma, V);
}

// Primitive recovery for the 3D WENO-Z faces (FP64): every cell's primitives, in
// the order of prim_at (GLM: with psi), into PW[8 or 9][n]. cflp != nullptr: also
// the CFL bound of the state, reduced over the workgroup into cflp[blockIdx.x].
template <bool GLM>
__global__ __launch_bounds__(kBlock) void k_prim(const double* __restrict__ U,
                                                 double* __restrict__ PW, Geom g,
                                                 int* __restrict__ flag,
                                                 double* __restrict__ cflp) {
  int i, j, k;
  int64_t c;
  const bool inside = linear_cell(g, i, j, k, c);
  double cmin = __builtin_inf();
  if (inside) {
    double V[9];
    bool ok;
    if constexpr (GLM) ok = glm_prim(U, g.n, c, g.gamma, V);
    else ok = prim_at<3>(U, g, i, j, k, V);
#pragma unroll
    for (int q = 0; q < (GLM ? 9 : 8); ++q) PW[q * g.n + c] = V[q];
    if (!ok) atomicOr(flag, 1);
    if (cflp) cmin = cfl_bound<3>(g, V, cmin);
  }
  if (cflp) workgroup_min_store(cmin, cflp + blockIdx.x);
}

// CFL: per-cell min over directions of dx_d / (|v_d| + c_f,d) (GLM: of the
// cell-centred state); grid-stride, wave64 shuffle + LDS reduction to one
// partial per block.
template <int DIM, bool GLM>
__global__ __launch_bounds__(kBlock) void k_cfl(const double* __restrict__ U, Geom g,
                                                double* __restrict__ partial,
                                                int* __restrict__ flag) {
  double m = __builtin_inf();
  for (int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x; c < g.n;
       c += (int64_t)gridDim.x * kBlock) {
    double V[9];
    bool ok;
    if constexpr (GLM) {
      ok = glm_prim(U, g.n, c, g.gamma, V);
    } else {
      int i, j, k;
      coords(g, c, i, j, k);
      ok = prim_at<DIM>(U, g, i, j, k, V);
    }
    if (!ok) atomicOr(flag, 1);
    m = cfl_bound<DIM>(g, V, m);
  }
  workgroup_min_store(m, partial + blockIdx.x);
}

// One block; eight loads in flight per thread (170 k partials of the 352^3 WENO-Z
// step: 80 -> 36 us).
__global__ __launch_bounds__(1024) void k_cfl_final(const double* __restrict__ partial, int np,
                                                    double cfl, double* __restrict__ dt_out) {
  double m = __builtin_inf();
  int b = threadIdx.x;
  for (; b + 7 * 1024 < np; b += 8 * 1024) {
    double v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = partial[b + s * 1024];
#pragma unroll
    for (int s = 0; s < 8; ++s) m = (v[s] < m) ? v[s] : m;
  }
  for (; b < np; b += 1024) m = (partial[b] < m) ? partial[b] : m;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(m, off, 64);
    m = (o < m) ? o : m;
  }
  __shared__ double red[16];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = red[0];
    for (int w = 1; w < 16; ++w) r = (red[w] < r) ? red[w] : r;
    *dt_out = cfl * r;
  }
}

// The adjoint's 2D stages (stage 1 and 4, or 3: records only), FP64 with the HLL
// average: face records in FW, E_z in EW.
template <int LIM, int RS>
hipError_t records_2d(const StageArgs& a) {
  const TileGrid rg = tile_grid<RowTile>(a.g), tg = tile_grid<Tile>(a.g);
  MHD_TIMED(a, K_FACES,
            hipLaunchKernelGGL((k_faces_tiled<LIM, RS>), dim3(tg.ntiles), dim3(Tile::NCORE), 0,
                               a.stream, a.U, a.FW, a.g, tg, a.flag));
  if (a.stage == 3)
    MHD_TIMED(a, K_EMF,
              hipLaunchKernelGGL((k_emf<LIM>), dim3(rg.ntiles), dim3(RowTile::NT), 0, a.stream,
                                 a.U, a.FW, a.EW, a.g, rg));
  else if (a.stage == 1)
    MHD_TIMED(a, K_UPDATE,
              hipLaunchKernelGGL((k_emf_update_2d<LIM, 1>), dim3(rg.ntiles), dim3(RowTile::NT), 0,
                                 a.stream, a.U, a.U0, a.out, a.FW, a.EW, a.g, rg, a.dt));
  else if (a.stage == 4)
    MHD_TIMED(a, K_UPDATE,
              hipLaunchKernelGGL((k_emf_update_2d<LIM, 4>), dim3(rg.ntiles), dim3(RowTile::NT), 0,
                                 a.stream, a.U, a.U0, a.out, a.FW, a.EW, a.g, rg, a.dt));
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

size_t stage_cfl_blocks(const Geom& g, int limiter, bool glm) {
  const size_t nl = (size_t)((g.n + kBlock - 1) / kBlock);
  return limiter == 2 || faces_by_cells(g, limiter, glm) || nl < kCfl3d ? nl : kCfl3d;
}

namespace {

// A: StageArgs or CflArgs. CFL partials of U, one per block of the grid-stride
// reduction; then dt from partials.
template <class A>
void cfl_pass(const A& a, double* partial, int np, int* flag) {
  const auto k = a.dim == 3 ? (a.glm ? k_cfl<3, true> : k_cfl<3, false>)
                            : (a.glm ? k_cfl<2, true> : k_cfl<2, false>);
  MHD_TIMED(a, K_CFL,
            hipLaunchKernelGGL(k, dim3(np), dim3(kBlock), 0, a.stream, a.U, a.g, partial, flag));
}
template <class A>
void cfl_final(const A& a, const double* partial, int np) {
  MHD_TIMED(a, K_CFL_FINAL,
            hipLaunchKernelGGL(k_cfl_final, dim3(1), dim3(1024), 0, a.stream, partial, np, a.cfl,
                               a.dt_out));
}

// Partials of the grid-stride CFL pass: at most most, as many as blocks of cells.
int cfl_parts(const Geom& g, int most) {
  const int64_t need = (g.n + kBlock - 1) / kBlock;
  return (int)(need < most ? need : most);
}

// 3D stage. WENO-Z: the primitives of every cell first. A time step that is the
// CFL bound of U: from those, or from a pass over U. Then the face kernel, which
// finishes the cell-averaged fields itself, and with CT the EMFs and the update of
// the staggered field.
//
// (With PLM and CT the face kernel once reduced the CFL bound itself, and as its
// state then had to wait for the next kernel, L was written and read back instead
// of U read once more: 256^3 5.18 -> 4.95 ms a step without, 384^3 mixed 12.0 ->
// 10.9.)
hipError_t stage3d(const StageArgs& a) {
  const double* cflp = a.cfl_partial;
  int np = 0;
  const bool cells = faces_by_cells(a.g, a.limiter, a.glm);
  if (a.limiter == 2 || cells) {
    if (!a.PW || (a.limiter == 2 && a.precision == 1)) return hipErrorInvalidValue;
    np = (int)((a.g.n + kBlock - 1) / kBlock);
    MHD_TIMED(a, K_PRIM,
              hipLaunchKernelGGL(a.glm ? k_prim<true> : k_prim<false>, dim3(np), dim3(kBlock), 0,
                                 a.stream, a.U, a.PW, a.g, a.flag, a.cfl_partial));
  } else if (cflp) {
    np = cfl_parts(a.g, kCfl3d);
    cfl_pass(a, a.cfl_partial, np, a.flag);
  }
  if (cflp && (cells || np > (int)kCfl3d ||
               march_grid(a.g, a.limiter).nblocks > kInlineCfl3d)) {
    cfl_final(a, cflp, np);
    cflp = nullptr;
  }
  if (cells) launch_faces_cells(a);
  else MHD_TIMED(a, K_FACES, launch_faces_march(a, cflp, np));
  if (!a.glm && (a.stage != 3 || a.keep_rhs)) MHD_TIMED(a, K_EMF, launch_ct(a));
  return hipGetLastError();
}

// 2D stage (a.records false): one kernel. Where the time step is the CFL
// bound of U, its partials come from the stage that wrote U or a pass over it;
// the stage's workgroups reduce up to kInlineCfl2d of them themselves on grids
// of about as many tiles, else k_cfl_final does it once.
hipError_t stage2d(const StageArgs& a) {
  const double* cflp = a.cfl_prev;
  int np = a.ncfl;
  if (a.cfl_partial && !cflp) {
    np = cfl_parts(a.g, kInlineCfl2d);
    cflp = a.cfl_partial;
    cfl_pass(a, a.cfl_partial, np, a.flag);
  }
  if (cflp && (np > kInlineCfl2d || stage_2d_tiles(a.g, a.limiter, a.emf, a.precision, a.glm) >
                                        2 * kInlineCfl2d)) {
    cfl_final(a, cflp, np);
    cflp = nullptr;
  }
  MHD_TIMED(a, K_FACES, launch_stage_2d(a, cflp, np));
  return hipGetLastError();
}

}  // namespace

hipError_t launch_stage(const StageArgs& a) {
  if (a.dim == 3) return stage3d(a);
  if (!a.records) return stage2d(a);
  if (a.limiter == 0) return a.riemann == 0 ? records_2d<0, 0>(a) : records_2d<0, 1>(a);
  return a.riemann == 0 ? records_2d<1, 0>(a) : records_2d<1, 1>(a);
}

// ---------------------------------------------------------------------------
// Allocation-free CFL time step (mhd_dt_device_noalloc). Its per-block
// partials and the unphysical flag live in this file-scope device array
// instead of the caller's workspace: kNoAllocPartials doubles, then the flag
// (an int) in the next double. Every device holds its own copy at its own
// address, found with hipGetSymbolAddress on the first call made with that
// device current; host code uses only that address, never the array's name.
// Calls that overlap on one device share the array and race.
static __device__ __align__(256) double scratch[kNoAllocPartials + 32];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch[kMaxDevices] = {};

hipError_t scratch_here(double** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[dev] = static_cast<double*>(p);
  }
  *out = g_scratch[dev];
  return hipSuccess;
}

// The flag must start each call at zero: a kernel clears it (no memset, so
// that a captured graph replays the clear correctly).
__global__ void k_flag_clear(int* __restrict__ flag) {
  if (threadIdx.x == 0) *flag = 0;
}

__global__ void k_flag_copy(const int* __restrict__ flag, int32_t* __restrict__ out) {
  if (threadIdx.x == 0) *out = *flag;
}

}  // namespace

hipError_t launch_cfl_noalloc(const CflArgs& a, int32_t* flag_out) {
  if (a.nblocks < 1 || a.nblocks > kNoAllocPartials) return hipErrorInvalidValue;
  double* base = nullptr;
  hipError_t e = scratch_here(&base);
  if (e != hipSuccess) return e;
  int* flag = reinterpret_cast<int*>(base + kNoAllocPartials);
  hipLaunchKernelGGL(k_flag_clear, dim3(1), dim3(64), 0, a.stream, flag);
  cfl_pass(a, base, a.nblocks, flag);
  cfl_final(a, base, a.nblocks);
  if (flag_out) hipLaunchKernelGGL(k_flag_copy, dim3(1), dim3(64), 0, a.stream, flag, flag_out);
  return hipGetLastError();
}

hipError_t launch_cfl(const CflArgs& a) {
  cfl_pass(a, a.partial, a.nblocks, a.flag);
  cfl_final(a, a.partial, a.nblocks);
  return hipGetLastError();
}

}  // namespace mhd
