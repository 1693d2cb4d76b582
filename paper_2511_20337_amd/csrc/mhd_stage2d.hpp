// 2D stage in one kernel (PLM, WENO-Z; CT, GLM cleaning): a workgroup recovers
// the primitives of its tile of W x H cells and the two (WENO-Z: three) cells
// around it, solves every face that the tile's flux differences and corner EMFs
// read, forms E_z at the tile's corners and updates its cells, all through LDS.
//
// What bounds it: on small grids the latency of this chain (the launches it
// replaces cost more), on large ones the instruction count. Measured against
// the two kernels per stage it replaces (tiled faces with 9 stored values each,
// EMF and update): 128^2 30.5 -> 15.2 us a step, KH 512^2 72.8 -> 60 us, 1500 x
// 1001 mixed with UCT-HLLD 341 -> 193 us. Against the three of WENO-Z and of GLM
// (primitives, faces, update): WENO-Z and RK2 29 x 21 43.3 -> 17.3 us a step,
// L(U) at 323 x 312 27.0 -> 24.2 us; WENO-Z, GLM and RK3 56 x 1230 90.6 -> 64.5
// us a step; GLM and RK2 82 x 831 49.7 -> 33.2 us. Choices:
//  - The faces are one list, x-faces then y-faces, dealt to the threads in
//    turn, so that the two extra rows and columns do not leave waves idle; a
//    lane's direction is two LDS offsets and a few selects.
//  - Large grids: 32 x 8 cells, 512 threads: 720 faces are 12 waves' work for 8
//    waves, and two workgroups fit a CU (16 waves, four per SIMD at 128
//    VGPRs; GLM in FP64 with HLLD spills 12 bytes a lane). A step of two launches at
//    512^2: 58.5 us, with 256 threads 63.3, 384: 81.9, 32 x 16 cells and 1024 threads
//    57.7 (1024^2: 203, 214, 298, 214), 8 x 8 cells 74. Small ones: 8 x 8 or 16 x 4
//    cells, 216 or 236 faces for 256 threads, one each: the shortest chain, and four
//    times the workgroups.
//  - The time step of the CFL bound is reduced from its partials by every
//    workgroup itself (a minimum is exact in any order), and between the steps
//    of one run the stage that writes a state leaves its partials, which saves
//    the pass over U (128^2: 17.0 -> 15.2 us a step).
#pragma once
#include <algorithm>

#include "mhd_device.hpp"
#include "mhd_grid.hpp"
#include "mhd_kernels.hpp"

namespace mhd {

namespace {

// S: cells around the tile that a reconstruction reaches; E: faces around it
// that the corner EMFs read (GLM has none).
template <int W_, int H_, int NT_, int S_, int E_>
struct Tile2 {
  static constexpr int W = W_, H = H_, NT = NT_, S = S_, E = E_;
  static constexpr int PW = W + 2 * S, NP = PW * (H + 2 * S);    // cells recovered
  static constexpr int NX = (W + 1) * (H + 2 * E);               // x-faces solved
  static constexpr int NF = NX + (W + 2 * E) * (H + 1);          // and y-faces
  static constexpr int FX = (W + 1) * H, FN = FX + W * (H + 1);  // those with fluxes
  static constexpr int NC = (W + 1) * (H + 1);                   // corners
};

// EM 0, 1: CT with the HLL or the UCT-HLLD average; 2: GLM.
template <class R, class T, int EM>
struct Lds2 {
  static constexpr int NV = EM == 2 ? 9 : 10, NFL = EM == 2 ? 9 : 6;
  R v[NV][T::NP];   // the eight primitives, then b_x and b_y (GLM: psi)
  R fl[NFL][T::FN];  // fluxes of rho, m_x, m_y, m_z, E, B_z (GLM: all nine fields)
  R ed[EM == 2 ? 1 : (EM == 1 ? 4 : 3)][EM == 2 ? 1 : T::NF];  // alpha+- (or om, d^L,
                                                              // d^R), the EMF's velocity
  R ez[EM == 2 ? 1 : T::NC];
  double red[T::NT / 64];
};

// i in [-3, n + W + 2] to its periodic image (n may be smaller than a tile)
__device__ __forceinline__ int wrap_near(int i, int n) {
  if (i < 0) return i + n;
  if (i < n) return i;
  i -= n;
  return (i < n) ? i : i % n;
}

// stage: as rk_coef. cflp != nullptr: dt = cfl times the minimum of the npart
// partials, written to *dt_out by workgroup 0; else *dtp or dt. cfl_next !=
// nullptr (the last stage of a step that another follows; out then is neither
// U nor U0, whose values above the tile are read): also the CFL bound of the
// new state over the tile into its place in cfl_next. tile0: the first workgroup's
// tile.
template <class T, int LIM, int RS, class R, int EM>
__global__ __launch_bounds__(T::NT) __attribute__((amdgpu_waves_per_eu(T::NT == 512 ? 4 : 2)))
void k_stage_2d(const double* __restrict__ U, const double* U0, double* out, Geom g, int ntx,
                unsigned tile0, int stage, double dt, const double* __restrict__ dtp,
                const double* __restrict__ cflp, int npart, double cfl,
                double* __restrict__ dt_out, double* __restrict__ cfl_next,
                int* __restrict__ flag, double dmin, double decay) {
  constexpr int W = T::W, H = T::H, NT = T::NT, PW = T::PW, NP = T::NP, NX = T::NX, NF = T::NF;
  constexpr int S = T::S, E = T::E;
  constexpr bool GLM = EM == 2;
  constexpr int NU = GLM ? 9 : 8, NW = GLM ? 9 : 7;  // fields, reconstructed quantities
  __shared__ Lds2<R, T, EM> L;
  const int t = (int)threadIdx.x;
  const unsigned tile = tile0 + blockIdx.x;
  const int i0 = (int)(tile % (unsigned)ntx) * W, j0 = (int)(tile / (unsigned)ntx) * H;
  const int64_t n = g.n;
  bool bad = false;
  for (int e = t; e < NP; e += NT) {
    const int i = wrap_near(i0 + e % PW - S, g.nx), j = wrap_near(j0 + e / PW - S, g.ny);
    double V[9];
    RawCell raw;
    if constexpr (GLM) {
      const int64_t cc = (int64_t)j * g.nx + i;
#pragma unroll
      for (int q = 0; q < 8; ++q) raw.u[q] = U[q * n + cc];
      raw.bxp = raw.u[5];  // (the mean of two equal faces is the cell's field, exactly)
      raw.byp = raw.u[6];
      raw.bzp = 0.0;
      V[8] = U[8 * n + cc];
    } else {
      raw = load_raw<2>(U, g, i, j, 0);
    }
    bad |= !prim_from_raw<2>(raw, g.gamma, V);
#pragma unroll
    for (int q = 0; q < 8; ++q) L.v[q][e] = (R)V[q];
    if constexpr (GLM) {
      L.v[8][e] = (R)V[8];
    } else {
      L.v[8][e] = (R)raw.u[5];
      L.v[9][e] = (R)raw.u[6];
    }
  }
  if (cflp) {
    double m = __builtin_inf();
    for (int b = t; b < npart; b += NT) m = (cflp[b] < m) ? cflp[b] : m;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(m, off, 64);
      m = (o < m) ? o : m;
    }
    if ((t & 63) == 0) L.red[t >> 6] = m;
  }
  if (bad) atomicOr(flag, 1);
  __syncthreads();
  double h = 0.0;
  if (cflp) {
    double m = L.red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) m = (L.red[w] < m) ? L.red[w] : m;
    h = cfl * m;
    if (tile == 0 && t == 0) *dt_out = h;
  } else if (stage != 0) {
    h = dtp ? *dtp : dt;
  }
  const R ch = GLM ? (R)(cfl * dmin / h) : R(0);  // the largest speed dt allows
  const R* v = &L.v[0][0];
  for (int f = t; f < NF; f += NT) {
    const bool yf = f >= NX;
    // the face's place: column and row of its cell in the list's rectangle
    const int q0 = yf ? f - NX : f, w0 = yf ? W + 2 * E : W + 1;
    const int fr = q0 / w0, fc = q0 - fr * w0;
    // first stencil cell, step
    const int o = yf ? fr * PW + fc + S - E : (fr + S - E) * PW + fc, st = yf ? PW : 1;
    // slots of the x frame, plus 1 at (v_n, v_t1, B_t1, B_n) and minus 2 at
    // (v_t2, B_t2) for a y-face
    constexpr int slot[9] = {0, 1, 2, 3, 6, 7, 4, 5, 8}, kind[9] = {0, 1, 1, 2, 1, 2, 0, 1, 0};
    const int ok[3] = {o, o + (yf ? NP : 0), o - (yf ? 2 * NP : 0)};
    R wl[NW], wr[NW];
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const R* p = v + ok[kind[q]] + slot[q] * NP;
      if constexpr (LIM == 2) {
        const R a[6] = {p[0], p[st], p[2 * st], p[3 * st], p[4 * st], p[5 * st]};
        wl[q] = wenoz_upper(a[0], a[1], a[2], a[3], a[4]);
        wr[q] = wenoz_upper(a[5], a[4], a[3], a[2], a[1]);
      } else {
        plm_pair<LIM, R>(p[0], p[st], p[2 * st], p[3 * st], wl[q], wr[q]);
      }
    }
    RiemannOut<R> r;
    R psi, fpsi;
    face_solve<RS, R, EM>((R)g.gamma, wl, wr, GLM ? R(0) : v[o + S * st + (yf ? 9 : 8) * NP], ch, r,
                          psi, fpsi);
    if constexpr (!GLM) {
      if (EM == 1) {
        L.ed[0][f] = r.om;
        L.ed[1][f] = r.dl;
        L.ed[2][f] = r.dr;
      } else {
        L.ed[0][f] = r.ap;
        L.ed[1][f] = r.am;
      }
      L.ed[EM == 1 ? 3 : 2][f] = yf ? r.v2 : r.v1;  // v_x on y-faces, v_y on x-faces
    }
    const int fi = yf ? T::FX + fr * W + fc - E : (fr - E) * (W + 1) + fc;
    if (yf ? (fc >= E && fc < W + E) : (fr >= E && fr < H + E)) {
      L.fl[0][fi] = r.f[0];
      L.fl[1][fi] = yf ? r.f[3] : r.f[1];
      L.fl[2][fi] = yf ? r.f[1] : r.f[2];
      L.fl[3][fi] = yf ? r.f[2] : r.f[3];
      L.fl[4][fi] = r.f[6];
      if constexpr (GLM) {
        L.fl[5][fi] = yf ? r.f[5] : psi;
        L.fl[6][fi] = yf ? psi : r.f[4];
        L.fl[7][fi] = yf ? r.f[4] : r.f[5];
        L.fl[8][fi] = fpsi;
      } else {
        L.fl[5][fi] = yf ? r.f[4] : r.f[5];
      }
    }
  }
  __syncthreads();
  // own cell (the first W * H threads; past the grid its periodic image, which
  // another tile owns); its state is loaded ahead of the EMFs
  const int x = t % W, y = t / W;
  const bool cell = t < W * H;
  const bool own = cell && i0 + x < g.nx && j0 + y < g.ny;
  const bool used = own || (cell && cfl_next);
  const int64_t c =
      used ? (int64_t)wrap_near(j0 + y, g.ny) * g.nx + wrap_near(i0 + x, g.nx) : 0;
  double u[NU], u0[NU];
#pragma unroll
  for (int q = 0; q < NU; ++q) {
    u[q] = used ? U[q * n + c] : 0.0;
    u0[q] = used ? U0[q * n + c] : 0.0;
  }
  // cfl_next: the faces above the tile, one each for the next H + W threads
  static_assert(T::NT >= W * H + W + H, "a thread for each face above the tile");
  const int ab = t - W * H;  // 0 .. H - 1: b_x at column W; H .. H + W - 1: b_y at row H
  const bool above = !GLM && cfl_next && ab >= 0 && ab < H + W;
  double ua = 0.0, ua0 = 0.0;
  if (above) {
    const int64_t ca = (ab < H) ? (int64_t)wrap_near(j0 + ab, g.ny) * g.nx + wrap_near(i0 + W, g.nx)
                                : (int64_t)wrap_near(j0 + H, g.ny) * g.nx + wrap_near(i0 + ab - H, g.nx);
    const int64_t fo = (ab < H ? F_BX : F_BY) * n + ca;
    ua = U[fo];
    ua0 = U0[fo];
  }
  if constexpr (!GLM) {
  constexpr int EL = LIM == 2 ? 1 : LIM;  // WENO-Z: van Leer PLM at the corners
  for (int e = t; e < T::NC; e += NT) {
    const int cj = e / (W + 1), ci = e - cj * (W + 1);
    const int xf = (cj + E) * (W + 1) + ci;         // the x-face above the corner
    const int yf = NX + cj * (W + 2 * E) + ci + E;      // the y-face to its right
    constexpr int VS = EM == 1 ? 3 : 2;
    R wv[4], wb[4], sv[4], sb[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      wv[s] = L.ed[VS][yf - 2 + s];
      wb[s] = L.v[9][(cj + S) * PW + ci + S - 2 + s];
      sv[s] = L.ed[VS][xf + (s - 2) * (W + 1)];
      sb[s] = L.v[8][(cj + S - 2 + s) * PW + ci + S];
    }
    const int xm = xf - (W + 1), ym = yf - 1;
    if constexpr (EM == 1)
      L.ez[e] = emf_core_hlld<EL, R>(L.ed[0][xm], L.ed[0][xf], L.ed[1][xm], L.ed[1][xf],
                                      L.ed[2][xm], L.ed[2][xf], L.ed[0][ym], L.ed[0][yf],
                                      L.ed[1][ym], L.ed[1][yf], L.ed[2][ym], L.ed[2][yf], wv, wb,
                                      sv, sb);
    else
      L.ez[e] = emf_core<EL, R>(L.ed[0][xm], L.ed[0][xf], L.ed[1][xm], L.ed[1][xf], L.ed[0][ym],
                                 L.ed[0][yf], L.ed[1][ym], L.ed[1][yf], wv, wb, sv, sb);
  }
  __syncthreads();
  }
  const RkCoef rk = rk_coef(stage, h);
  const double idx = 1.0 / g.dx, idy = 1.0 / g.dy;
  double v1[NU];
  if (used) {
    const int fx = y * (W + 1) + x, fy = T::FX + y * W + x, ec = y * (W + 1) + x;
    double Lq[NU];
#pragma unroll
    for (int q = 0; q < (GLM ? 9 : 6); ++q)
      Lq[!GLM && q == 5 ? 7 : q] = -(((double)L.fl[q][fx + 1] - (double)L.fl[q][fx]) * idx +
                                     ((double)L.fl[q][fy + W] - (double)L.fl[q][fy]) * idy);
    if constexpr (!GLM) {
      const double e0 = (double)L.ez[ec];
      Lq[5] = -(((double)L.ez[ec + W + 1] - e0) * idy);
      Lq[6] = ((double)L.ez[ec + 1] - e0) * idx;
    }
#pragma unroll
    for (int q = 0; q < NU; ++q) v1[q] = rk_apply(rk, u[q], u0[q], Lq[q]);
    if (GLM) v1[NU - 1] *= decay;
    if (own) {
#pragma unroll
      for (int q = 0; q < NU; ++q) out[q * n + c] = v1[q];
    }
  }
  if (!cfl_next) return;
  // the new staggered field, in the place of the primitives
  static_assert(sizeof(double) * (T::FX + W * (H + 1)) <= sizeof(R) * 8 * NP, "it fits there");
  double* const nbx = reinterpret_cast<double*>(&L.v[0][0]);
  double* const nby = nbx + T::FX;
  if (used) {
    nbx[y * (W + 1) + x] = v1[5];
    nby[y * W + x] = v1[6];
  }
  if (above) {
    if constexpr (GLM) {
    } else if (ab < H) {
      const int ec = ab * (W + 1) + W;
      nbx[ec] = rk_apply(rk, ua, ua0, -(((double)L.ez[ec + W + 1] - (double)L.ez[ec]) * idy));
    } else {
      const int ec = H * (W + 1) + ab - H;
      nby[H * W + ab - H] =
          rk_apply(rk, ua, ua0, ((double)L.ez[ec + 1] - (double)L.ez[ec]) * idx);
    }
  }
  __syncthreads();
  double m = __builtin_inf();
  if (own) {
    RawCell raw;
#pragma unroll
    for (int q = 0; q < 8; ++q) raw.u[q] = v1[q];
    raw.bxp = GLM ? v1[5] : nbx[y * (W + 1) + x + 1];
    raw.byp = GLM ? v1[6] : nby[(y + 1) * W + x];
    raw.bzp = 0.0;
    double V[8];
    prim_from_raw<2>(raw, g.gamma, V);  // (an unphysical cell is the next stage's to report)
    m = cfl_bound<2>(g, V, m);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(m, off, 64);
    m = (o < m) ? o : m;
  }
  if ((t & 63) == 0) L.red[t >> 6] = m;
  __syncthreads();
  if (t == 0) {
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) m = (L.red[w] < m) ? L.red[w] : m;
    cfl_next[tile] = m;
  }
}

// A launch has fewer than 2^32 threads; a narrow grid of many rows takes several.
constexpr unsigned kTilesPerLaunch = 1u << 22;

template <class T, int LIM, int RS, class R, int EM>
void stage_2d(const StageArgs& a, const double* cflp, int npart) {
  const int ntx = (a.g.nx + T::W - 1) / T::W, nty = (a.g.ny + T::H - 1) / T::H;
  const unsigned tiles = (unsigned)ntx * (unsigned)nty;
  for (unsigned t0 = 0; t0 < tiles; t0 += kTilesPerLaunch)
    hipLaunchKernelGGL((k_stage_2d<T, LIM, RS, R, EM>),
                       dim3(std::min(tiles - t0, kTilesPerLaunch)), dim3(T::NT), 0, a.stream, a.U,
                       a.U0 ? a.U0 : a.U, a.out, a.g, ntx, t0, a.stage, a.dt, a.dtp, cflp, npart,
                       a.cfl, a.dt_out, a.cfl_next, a.flag, a.glm_dmin,
                       (a.stage == 2 || a.stage == 5) ? a.glm_decay : 1.0);
}

// Widths of the large tiles: what two workgroups of a CU have LDS for (in FP64
// the UCT-HLLD average keeps four values a face, and WENO-Z recovers three
// cells around).
constexpr int large_w(int limiter, int emf, int precision) {
  return emf == 2 ? 32 : limiter == 2 ? 24 : (emf == 1 && precision == 0) ? 28 : 32;
}
// The tile of a grid: a large one, or a small one of 64 cells, square or (where that
// takes fewer by a tenth: few or ragged rows) flat. Grids of at most kSmallTiles2d
// large tiles take small ones, and so does a grid that they cover in less: a large
// tile's cell costs 0.8 of a small one's (WENO-Z 0.9, mixed precision 0.6). A step in us,
// large / square / flat: GLM 4 x 40000 220 / 71 / -, WENO-Z 25 x 6400 115 / 87 / -, 160000 x
// 4 423 / 451 / 239, 37647 x 17 303 / 342 / 277, KH 512^2 60 / 76 / -. (Narrow tiles of 4 x
// 16 take 1.45 times as long as square ones, their rows being 32 bytes.)
constexpr int kLargeH = 8;
struct TileShape {
  int w, h;
};
TileShape tile_shape(const Geom& g, int limiter, int large, bool mixed) {
  auto tiles = [&](int w, int h) {
    return (int64_t)((g.nx + w - 1) / w) * ((g.ny + h - 1) / h);
  };
  TileShape t = {8, 8};
  if (10 * tiles(16, 4) <= 9 * tiles(8, 8)) t = {16, 4};
  const double cell = limiter == 2 ? 0.9 : mixed ? 0.6 : 0.8;
  if (tiles(32, 8) > kSmallTiles2d &&
      cell * (large * kLargeH) * (double)tiles(large, kLargeH) <=
          (double)(t.w * t.h) * (double)tiles(t.w, t.h))
    t = {large, kLargeH};
  return t;
}

template <int LIM, int RS, class R, int EM>
void stage_2d_tile(const StageArgs& a, const double* cflp, int npart) {
  constexpr int S = LIM == 2 ? 3 : 2, E = EM == 2 ? 0 : 2;
  constexpr int large = large_w(LIM, EM, sizeof(R) == 4);
  const TileShape t = tile_shape(a.g, LIM, large, sizeof(R) == 4);
  if (t.w == large) stage_2d<Tile2<large, kLargeH, 512, S, E>, LIM, RS, R, EM>(a, cflp, npart);
  else if (t.w == 16) stage_2d<Tile2<16, 4, 256, S, E>, LIM, RS, R, EM>(a, cflp, npart);
  else stage_2d<Tile2<8, 8, 256, S, E>, LIM, RS, R, EM>(a, cflp, npart);
}
template <int LIM, int RS, class R>
void stage_2d_emf(const StageArgs& a, const double* cflp, int npart) {
  if (a.glm) stage_2d_tile<LIM, RS, R, 2>(a, cflp, npart);
  else if (a.emf == 1) stage_2d_tile<LIM, RS, R, 1>(a, cflp, npart);
  else stage_2d_tile<LIM, RS, R, 0>(a, cflp, npart);
}
template <int RS>
void stage_2d_lim(const StageArgs& a, const double* cflp, int npart) {
  const bool mixed = a.precision == 1;
  if (a.limiter == 2) {
    stage_2d_emf<2, RS, double>(a, cflp, npart);
  } else if (a.limiter == 1) {
    if (mixed) stage_2d_emf<1, RS, float>(a, cflp, npart);
    else stage_2d_emf<1, RS, double>(a, cflp, npart);
  } else {
    if (mixed) stage_2d_emf<0, RS, float>(a, cflp, npart);
    else stage_2d_emf<0, RS, double>(a, cflp, npart);
  }
}

}  // namespace

int stage_2d_tiles(const Geom& g, int limiter, int emf, int precision, bool glm) {
  const TileShape t =
      tile_shape(g, limiter, large_w(limiter, glm ? 2 : emf, precision), precision == 1);
  return ((g.nx + t.w - 1) / t.w) * ((g.ny + t.h - 1) / t.h);
}

void launch_stage_2d(const StageArgs& a, const double* cflp, int npart) {
  if (a.riemann == 0) stage_2d_lim<0>(a, cflp, npart);
  else stage_2d_lim<1>(a, cflp, npart);
}

}  // namespace mhd
