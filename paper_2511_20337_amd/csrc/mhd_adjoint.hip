// Adjoint (vector-Jacobian product) of one SSP-RK2 or SSP-RK3 step, FP64,
// gather form.
//
// The RK2 step is Phi(Un) = (Un + S(S(Un)))/2 with S(U) = U + dt L(U). Reverse:
//   G2 = Ubar1/2;        U1bar = G2 + dt J_L(U1)^T G2;
//   Ubar0 = Ubar1/2 + U1bar + dt J_L(Un)^T U1bar;
//   dtbar = <G2, L(U1)> + <U1bar, L(Un)>.
// The RK3 step takes the same per-stage adjoint three times (adjoint_rk3).
// J_L^T G is assembled from the local Jacobians of each piece of L, every
// output written by exactly one thread (no atomics, deterministic):
//   k_adj_edges — the EMF cotangent from -curl E, times the partial
//                 derivatives of the upwind EMF average w.r.t. its twelve
//                 inputs (per edge, stored);
//   k_adj_faces — per face: flux cotangents from the divergence, cotangents
//                 of alpha+-, the weighted velocities and b gathered from the
//                 edges that used them (through the adjoint of their
//                 reconstruction), then the Riemann solver's vector-Jacobian
//                 product: one hand-written reverse sweep (HLL over the values
//                 the solver recorded, HLLD over values formed again);
//   k_adj_cells — per cell: adjoint of PLM (gathering the face-state
//                 cotangents of the faces each cell feeds) and of primitive
//                 recovery;
//   k_adj_final — staggered-field cotangents, the RK combination and the
//                 dtbar reduction.
// At every non-smooth point the derivative of the branch taken by the
// forward step is used (limiter at extrema, min/max, Riemann region).
#include "mhd_adjoint.hpp"
#include "mhd_grid.hpp"
#include "mhd_kernels.hpp"

namespace mhd {

namespace {

// ---------------------------------------------------------------------------
// Hand-written reverse sweeps of the Riemann solvers. The forward values that
// decide a branch come from the forward solvers' own functions, so every branch
// (wave-speed min/max, HLL/HLLD region, degenerate star state, sign of the normal
// field) is the one the forward kernels take; the derivative of each branch is then
// propagated backwards once for all fifteen inputs. At a square root of zero
// the derivative is taken as zero.
//
// BT: whether the cotangents of the two B_t fluxes (fb[4], fb[5]) can be
// nonzero: in 3D neither, in 2D that of B_z (t2 of x-faces, t1 of y-faces).

// phys(): cotangents of u[7], f[7] and pt -> added to wb[7] and bnb. Those of f
// and u are al and be times the flux cotangents fbar (u[6], the energy: ub6
// more), so that no array of them is held.
template <bool B4, bool B5>
__device__ __forceinline__ void phys_vjp(double igm1, const double* w, double bn,
                                         const double* fbar, double al, double be, double ub6,
                                         double ptb, double* wb, double& bnb) {
  double fb[7], ub[7];
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    fb[q] = al * fbar[q];
    ub[q] = be * fbar[q];
  }
  ub[6] += ub6;
  const double rho = w[0], vn = w[1], v1 = w[2], v2 = w[3], b1 = w[4], b2 = w[5], p = w[6];
  const double bb = bn * bn + b1 * b1 + b2 * b2;
  const double pt = p + 0.5 * bb;
  const double v2s = vn * vn + v1 * v1 + v2 * v2;
  const double en = p * igm1 + 0.5 * rho * v2s + 0.5 * bb;
  const double mn = rho * vn;
  const double vb = vn * bn + v1 * b1 + v2 * b2;
  double mnb = fb[0] + fb[1] * vn + fb[2] * v1 + fb[3] * v2 + ub[1];
  double vnb = fb[1] * mn + fb[6] * (en + pt);
  double v1b = fb[2] * mn + ub[2] * rho;
  double v2b = fb[3] * mn + ub[3] * rho;
  double b1b = -fb[2] * bn;
  double b2b = -fb[3] * bn;
  double bnl = -2.0 * bn * fb[1] - fb[2] * b1 - fb[3] * b2 - fb[6] * vb;
  if (B4) {
    vnb += fb[4] * b1;
    v1b -= fb[4] * bn;
    b1b += fb[4] * vn + ub[4];
    bnl -= fb[4] * v1;
  }
  if (B5) {
    vnb += fb[5] * b2;
    v2b -= fb[5] * bn;
    b2b += fb[5] * vn + ub[5];
    bnl -= fb[5] * v2;
  }
  const double ptt = ptb + fb[1] + fb[6] * vn;
  const double enb = ub[6] + fb[6] * vn;
  const double vbb = -fb[6] * bn;
  vnb += vbb * bn;
  bnl += vbb * vn;
  v1b += vbb * b1;
  b1b += vbb * v1;
  v2b += vbb * b2;
  b2b += vbb * v2;
  const double rhob = ub[0] + ub[2] * v1 + ub[3] * v2 + mnb * vn + enb * 0.5 * v2s;
  vnb += mnb * rho;
  const double v2sb = enb * 0.5 * rho;
  const double bbb = 0.5 * (enb + ptt);
  const double pb = enb * igm1 + ptt;
  vnb += 2.0 * vn * v2sb;
  v1b += 2.0 * v1 * v2sb;
  v2b += 2.0 * v2 * v2sb;
  bnl += 2.0 * bn * bbb;
  b1b += 2.0 * b1 * bbb;
  b2b += 2.0 * b2 * bbb;
  wb[0] += rhob; wb[1] += vnb; wb[2] += v1b; wb[3] += v2b; wb[4] += b1b; wb[5] += b2b;
  wb[6] += pb;
  bnb += bnl;
}

// cfast(): cotangent of c_f -> added to rho, p (wb[0], wb[6]), b_t (wb[4], wb[5]), bn.
// The branch values are recomputed with cfast's own expressions.
__device__ __forceinline__ void cfast_vjp(double g, const double* w, double bn, double cfb,
                                          double* wb, double& bnb) {
  const double rho = w[0], p = w[6], b1 = w[4], b2 = w[5];
  const double gp = g * p;
  const double bn2 = bn * bn;
  const double bb = fma_r(b2, b2, fma_r(b1, b1, bn2));
  const double a = gp + bb;
  const double x = fma_r(a, a, -(4.0 * gp) * bn2);
  const double disc = max_r(0.0, x);
  const double sd = sqrt_r(disc);
  const double q = div_r(a + sd, 2.0 * rho);
  const double cf = sqrt_r(q);
  // reciprocals from the refined estimate (a few ulps from the quotients);
  // the selects drop the non-finite values at cf = 0, sd = 0
  const double qb = cf > 0.0 ? cfb * 0.5 * rcp_r(cf) : 0.0;
  const double irho = rcp_r(rho);
  const double i2r = 0.5 * irho;
  double ab = qb * i2r;
  const double sdb = qb * i2r;
  const double rhob = -qb * q * irho;
  const double discb = sd > 0.0 ? sdb * 0.5 * rcp_r(sd) : 0.0;
  const double xb = (x > 0.0) ? discb : 0.0;
  ab += 2.0 * a * xb;
  const double gpb = -4.0 * bn2 * xb + ab;
  const double bn2b = -4.0 * gp * xb + ab;
  wb[0] += rhob;
  wb[6] += g * gpb;
  wb[4] += 2.0 * b1 * ab;
  wb[5] += 2.0 * b2 * ab;
  bnb += 2.0 * bn * bn2b;
}

// HLL: the forward values recorded by riemann_core.
template <bool B4, bool B5>
__device__ __forceinline__ void hll_vjp(double g, const double* wl, const double* wr, double bn,
                                        const double* fbar, double apbar, double ambar,
                                        double v1bar, double v2bar, double* wlb, double* wrb,
                                        double& bnb) {
  RiemannTape t;
  RiemannOut<double> o;
  riemann_core<double, RiemannTape>(g, wl, wr, bn, o, t);
  const double igm1 = rcp_r(g - 1.0);
#pragma unroll
  for (int q = 0; q < 7; ++q) { wlb[q] = 0.0; wrb[q] = 0.0; }
  bnb = 0.0;
  double all = 0.0, bel = 0.0, alr = 0.0, ber = 0.0;  // of phys_vjp, left and right
  double slb = 0.0, srb = 0.0;
  // HLL-weighted velocities v = (ap wl + am wr) / (ap + am)
  const double n1b = v1bar * t.isum, n2b = v2bar * t.isum;
  const double sumb = -(v1bar * t.v1 + v2bar * t.v2) * t.isum;
  const double apb = apbar + n1b * wl[2] + n2b * wl[3] + sumb;
  const double amb = ambar + n1b * wr[2] + n2b * wr[3] + sumb;
  wlb[2] += n1b * t.ap;
  wrb[2] += n1b * t.am;
  wlb[3] += n2b * t.ap;
  wrb[3] += n2b * t.am;
  if (t.region == 0) {
    all = 1.0;
  } else if (t.region == 1) {
    alr = 1.0;
  } else {
    // HLL fan: f = (sl sr (ur - ul) + sr fl - sl fr) / (sr - sl)
    double db = 0.0;
#pragma unroll
    for (int q = 0; q < 7; ++q) {
      if ((q == 4 && !B4) || (q == 5 && !B5)) continue;
      const double nb = fbar[q] * t.idn;
      db -= nb * o.f[q];
      const double du = t.ur[q] - t.ul[q];
      slb += nb * (t.sr * du - t.fr[q]);
      srb += nb * (t.sl * du + t.fl[q]);
    }
    all = t.idn * t.sr;
    alr = -t.idn * t.sl;
    ber = t.idn * t.sl * t.sr;
    bel = -ber;
    srb += db;
    slb -= db;
  }
  // alpha+- = max(0, S_R), max(0, -S_L)
  if (t.sr > 0.0) srb += apb;
  if (-t.sl > 0.0) slb -= amb;
  // S_L = min(u_L, u_R) - c, S_R = max(u_L, u_R) + c, c = max(c_L, c_R);
  // the selected argument takes the cotangent (the first one on ties)
  if (wr[1] < wl[1]) wrb[1] += slb; else wlb[1] += slb;
  if (wr[1] > wl[1]) wrb[1] += srb; else wlb[1] += srb;
  const double cmb = srb - slb;
  {
    // one evaluation on the side whose fast speed was taken, by selects
    const bool rs = t.cr > t.cl;
    double wc[7], wcb[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 7; ++q) wc[q] = rs ? wr[q] : wl[q];
    cfast_vjp(g, wc, bn, cmb, wcb, bnb);
    constexpr int touched[4] = {0, 4, 5, 6};  // rho, B_t1, B_t2, p
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = touched[e];
      wrb[q] += rs ? wcb[q] : 0.0;
      wlb[q] += rs ? 0.0 : wcb[q];
    }
  }
  phys_vjp<B4, B5>(igm1, wl, bn, fbar, all, bel, 0.0, 0.0, wlb, bnb);
  phys_vjp<B4, B5>(igm1, wr, bn, fbar, alr, ber, 0.0, 0.0, wrb, bnb);
}

// Reverse of one side's tangential star state (hlld_flux: eta, zeta and what
// they multiply): the cotangents vsb, wsb, b1sb, b2sb of v*_t, B*_t and rsb of
// rho* of the side with state w, front S, mass flux m = d rho, ism = 1/(S - S_M).
// The cotangent of ism that the energy adds comes in as esism = esbar E* .
struct StarSide {
  double S, d, m, ism, rs, iden2, eta, zeta;
  bool deg;
};
__device__ __forceinline__ void star_vjp(const StarSide& t, const double* w, double bn, double sm,
                                         double vsb, double wsb, double b1sb, double b2sb,
                                         double rsb, double esism, double* wb, double& mb,
                                         double& db, double& Sb, double& smb, double& bnb,
                                         double& bn2b) {
  wb[2] += vsb;
  wb[3] += wsb;
  wb[4] += b1sb * t.zeta - vsb * t.eta;
  wb[5] += b2sb * t.zeta - wsb * t.eta;
  // (degenerate: eta = 0 and zeta = 1 are constants)
  const double etab = t.deg ? 0.0 : -(vsb * w[4] + wsb * w[5]);
  const double zetab = t.deg ? 0.0 : b1sb * w[4] + b2sb * w[5];
  const double i2 = t.deg ? 0.0 : t.iden2;
  const double e = etab * i2, z = zetab * i2;
  const double denb = -(etab * t.eta + zetab * t.zeta) * i2;
  bnb += e * (sm - w[1]);
  wb[1] -= e * bn;
  mb += z * t.d + denb * (t.S - sm) + rsb * t.ism;
  db += z * t.m;
  bn2b -= z + denb;
  const double it = -(esism + rsb * t.rs) * t.ism;
  Sb += denb * t.m + it;
  smb += e * bn - denb * t.m - it;
}

// HLLD. As in hlld_flux the side a of the contact that the face lies on is
// selected first; the solver is symmetric under the exchange of the sides, with
// tau = 1 (a left) or -1 in the places of its signs, so one sweep in (a, o =
// the other side) serves both, and the cotangents are dealt to left and right
// at the end (4750 instructions for the three faces of a cell in 3D, against
// 7900 and 440 registers with a tape of both sides).
template <bool B4, bool B5>
__device__ __forceinline__ void hlld_vjp(double g, const double* wl, const double* wr, double bn,
                                         const double* fbar, double apbar, double ambar,
                                         double v1bar, double v2bar, double* wlb, double* wrb,
                                         double& bnb) {
  // forward (hlld_fan, hlld_star, hlld_front: as the flux forms them)
  const double igm1 = rcp_r(g - 1.0);
  const double bn2 = bn * bn;
  const HlldFan<double> fn = hlld_fan<double>(g, wl, wr, bn, bn2);
  const double ptl = fn.ptl, ptr = fn.ptr, c2l = fn.c2l, c2r = fn.c2r;
  const double sl = fn.sl, sr = fn.sr, sm = fn.sm, pts = fn.pts, iden = fn.iden;
  const bool fan = fn.fan, rt = fn.rt;
  const bool lo_o = rt ? !(wr[1] < wl[1]) : (wr[1] < wl[1]);  // min(u) is the other side's
  const bool hi_o = rt ? !(wr[1] > wl[1]) : (wr[1] > wl[1]);
  const bool c_o = rt ? !(c2r > c2l) : (c2r > c2l);           // and the fast speed
  const double tau = rt ? -1.0 : 1.0;
  double w[7], wo[7], wb[7], wob[7];
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    w[q] = rt ? wr[q] : wl[q];
    wo[q] = rt ? wl[q] : wr[q];
    wb[q] = 0.0;
    wob[q] = 0.0;
  }
  bnb = 0.0;
  const double Sa = rt ? sr : sl, So = rt ? sl : sr;
  const double pta = rt ? ptr : ptl, pto = rt ? ptl : ptr;
  double Sab = 0.0, Sob = 0.0, ptab = 0.0;
  // HLL-weighted velocities v = (A w_a + O w_o) / (A + O), A and O the alphas
  // that weigh the sides: A = max(0, tau S_o), O = max(0, -tau S_a)
  {
    const double A = max0_r(tau * So), O = max0_r(-tau * Sa);
    const double isum = rcp_r(A + O);
    const double n1b = v1bar * isum, n2b = v2bar * isum;
    const double sumb = -(n1b * (A * w[2] + O * wo[2]) + n2b * (A * w[3] + O * wo[3])) * isum;
    const double Ab = (rt ? ambar : apbar) + n1b * w[2] + n2b * w[3] + sumb;
    const double Ob = (rt ? apbar : ambar) + n1b * wo[2] + n2b * wo[3] + sumb;
    wb[2] = n1b * A;
    wob[2] = n1b * O;
    wb[3] = n2b * A;
    wob[3] = n2b * O;
    Sob = (A > 0.0) ? tau * Ab : 0.0;
    Sab = (O > 0.0) ? -tau * Ob : 0.0;
  }
  double be = 0.0, ub6 = 0.0;  // of phys_vjp
  if (fan) {
    const double en = fma_r(0.5, fma_r(w[5], w[5], fma_r(w[4], w[4], bn2)),
                            fma_r(0.5 * w[0], fma_r(w[3], w[3], fma_r(w[2], w[2], w[1] * w[1])),
                                  w[6] * igm1));
    StarSide a;
    a.S = Sa;
    a.d = Sa - w[1];
    a.m = a.d * w[0];
    a.ism = rcp_r(Sa - sm);
    a.rs = a.m * a.ism;
    const double sq = sqrt_r(a.rs);
    const double abn = abs_r(bn);
    const double sa = hlld_front(sm, abn, sq, rt);
    auto star = [&](StarSide& t, double un) {
      const HlldStar<double> o = hlld_star(t.m, t.d, t.S, un, sm, bn, bn2);
      t.deg = o.deg;
      t.iden2 = o.iden2;
      t.eta = o.eta;
      t.zeta = o.zeta;
    };
    star(a, w[1]);
    const double vs = fma_r(-w[4], a.eta, w[2]), ws = fma_r(-w[5], a.eta, w[3]);
    const double b1s = w[4] * a.zeta, b2s = w[5] * a.zeta;
    const double vb = fma_r(w[3], w[5], fma_r(w[2], w[4], w[1] * bn));
    const double vbs = fma_r(ws, b2s, fma_r(vs, b1s, sm * bn));
    const double es = fma_r(bn, vb - vbs, fma_r(pts, sm, fma_r(a.d, en, -pta * w[1]))) * a.ism;
    const double d_o = So - wo[1], m_o = d_o * wo[0];
    // F*_a = F_a + S_a (U*_a - U_a)
    const double us[7] = {a.rs, a.rs * sm, a.rs * vs, a.rs * ws, b1s, b2s, es};
    const double uu[7] = {w[0], w[0] * w[1], w[0] * w[2], w[0] * w[3], w[4], w[5], en};
#pragma unroll
    for (int q = 0; q < 7; ++q)
      if (!((q == 4 && !B4) || (q == 5 && !B5))) Sab += fbar[q] * (us[q] - uu[q]);
    be = -Sa;
    double Su = Sa;  // the cotangent of U*_a is Su fbar
    double vsb = 0.0, wsb = 0.0, b1sb = 0.0, b2sb = 0.0, rsb = 0.0, esb = 0.0, smb = 0.0;
    double mab = 0.0, dab = 0.0, mob = 0.0, dob = 0.0, bn2b = 0.0;
    if ((sa >= 0.0) == rt) {
      // between the Alfven fronts: F**_a = F*_a + S*_a (U**_a - U*_a)
      StarSide o;
      o.S = So;
      o.d = d_o;
      o.m = m_o;
      o.ism = rcp_r(So - sm);
      o.rs = m_o * o.ism;
      const double sqo = sqrt_r(o.rs);
      star(o, wo[1]);
      const double vso = fma_r(-wo[4], o.eta, wo[2]), wso = fma_r(-wo[5], o.eta, wo[3]);
      const double b1so = wo[4] * o.zeta, b2so = wo[5] * o.zeta;
      const double st = tau * ((bn > 0.0) ? 1.0 : ((bn < 0.0) ? -1.0 : 0.0));
      const double isq = rcp_r(sq + sqo);
      const double q2 = st * sq * sqo;
      const double vss = (sq * vs + sqo * vso + st * (b1so - b1s)) * isq;
      const double wss = (sq * ws + sqo * wso + st * (b2so - b2s)) * isq;
      const double b1ss = (sq * b1so + sqo * b1s + q2 * (vso - vs)) * isq;
      const double b2ss = (sq * b2so + sqo * b2s + q2 * (wso - ws)) * isq;
      const double T = vs * b1s + ws * b2s - (vss * b1ss + wss * b2ss);
      const double ess = es - st * sq * T;
      const double uss[7] = {a.rs, a.rs * sm, a.rs * vss, a.rs * wss, b1ss, b2ss, ess};
      double sab = 0.0;
#pragma unroll
      for (int q = 0; q < 7; ++q)
        if (!((q == 4 && !B4) || (q == 5 && !B5))) sab += fbar[q] * (uss[q] - us[q]);
      Su -= sa;
      auto ussb = [&](int q) { return sa * fbar[q]; };  // cotangent of U**_a
      rsb += ussb(0) + ussb(1) * sm + ussb(2) * vss + ussb(3) * wss;
      smb += ussb(1) * a.rs + sab;
      esb += ussb(6);
      const double Tb = -st * sq * ussb(6);
      double sqb = -st * T * ussb(6);
      vsb += Tb * b1s;
      b1sb += Tb * vs;
      wsb += Tb * b2s;
      b2sb += Tb * ws;
      const double nvb = (ussb(2) * a.rs - Tb * b1ss) * isq, nwb = (ussb(3) * a.rs - Tb * b2ss) * isq;
      const double nb1b = ((B4 ? ussb(4) : 0.0) - Tb * vss) * isq;
      const double nb2b = ((B5 ? ussb(5) : 0.0) - Tb * wss) * isq;
      const double sumb = -(nvb * vss + nwb * wss + nb1b * b1ss + nb2b * b2ss);
      const double qb = nb1b * (vso - vs) + nb2b * (wso - ws);
      sqb += nvb * vs + nwb * ws + nb1b * b1so + nb2b * b2so + sumb + qb * st * sqo;
      const double sqob = nvb * vso + nwb * wso + nb1b * b1s + nb2b * b2s + sumb + qb * st * sq;
      vsb += nvb * sq - nb1b * q2;
      wsb += nwb * sq - nb2b * q2;
      b1sb += nb1b * sqo - nvb * st;
      b2sb += nb2b * sqo - nwb * st;
      // the Alfven front S*_a = S_M - tau |bn| / sqrt(rho*_a)
      const double isa = rcp_r(sq);
      bnb -= tau * sab * isa * (bn < 0.0 ? -1.0 : 1.0);
      sqb += tau * sab * abn * isa * isa;
      rsb += sq > 0.0 ? sqb * 0.5 * isa : 0.0;
      const double rsob = sqo > 0.0 ? sqob * 0.5 * rcp_r(sqo) : 0.0;
      star_vjp(o, wo, bn, sm, nvb * sqo + nb1b * q2, nwb * sqo + nb2b * q2, nb1b * sq + nvb * st,
               nb2b * sq + nwb * st, rsob, 0.0, wob, mob, dob, Sob, smb, bnb, bn2b);
    }
    // U*_a = (rho*, rho* S_M, rho* v*, rho* w*, B*_t1, B*_t2, E*)
    rsb += Su * (fbar[0] + fbar[1] * sm + fbar[2] * vs + fbar[3] * ws);
    smb += Su * fbar[1] * a.rs;
    vsb += Su * fbar[2] * a.rs;
    wsb += Su * fbar[3] * a.rs;
    if (B4) b1sb += Su * fbar[4];
    if (B5) b2sb += Su * fbar[5];
    esb += Su * fbar[6];
    // E* = (d E - pt u + pts S_M + bn (v.B - v*.B*)) / (S - S_M)
    const double neb = esb * a.ism;
    dab += neb * en;
    ub6 = neb * a.d;
    ptab -= neb * w[1];
    wb[1] -= neb * pta;
    const double ptsb = neb * sm;
    smb += neb * pts;
    const double vbb = neb * bn;
    bnb += neb * (vb - vbs) + vbb * (w[1] - sm);
    smb -= vbb * bn;
    vsb -= vbb * b1s;
    b1sb -= vbb * vs;
    wsb -= vbb * b2s;
    b2sb -= vbb * ws;
    wb[1] += vbb * bn;
    wb[2] += vbb * w[4];
    wb[4] += vbb * w[2];
    wb[3] += vbb * w[5];
    wb[5] += vbb * w[3];
    star_vjp(a, w, bn, sm, vsb, wsb, b1sb, b2sb, rsb, esb * es, wb, mab, dab, Sab, smb, bnb, bn2b);
    bnb += 2.0 * bn * bn2b;
    // S_M = (m_o u_o - m_a u_a + pt_a - pt_o) / (m_o - m_a) and the star total
    // pressure (m_a m_o (u_o - u_a) + m_o pt_a - m_a pt_o) / (m_o - m_a); iden
    // is 1/(m_R - m_L)
    const double id = tau * iden;
    const double Nb = smb * id, Pb = ptsb * id, Dt = -(smb * sm + ptsb * pts) * id;
    const double du = wo[1] - w[1], mm = a.m * m_o;
    mob += Nb * wo[1] + Pb * (a.m * du + pta) + Dt;
    mab += Pb * (m_o * du - pto) - Nb * w[1] - Dt;
    wob[1] += Nb * m_o + Pb * mm;
    wb[1] -= Nb * a.m + Pb * mm;
    ptab += Nb + Pb * m_o;
    const double ptob = -Nb - Pb * a.m;
    // m = d rho, d = S - u
    dob += mob * wo[0];
    wob[0] += mob * d_o;
    dab += mab * w[0];
    wb[0] += mab * a.d;
    Sob += dob;
    wob[1] -= dob;
    Sab += dab;
    wb[1] -= dab;
    // the other side's total pressure
    wob[6] += ptob;
    wob[4] += ptob * wo[4];
    wob[5] += ptob * wo[5];
    bnb += ptob * bn;
  }
  // S_L = min(u_L, u_R) - c, S_R = max(u_L, u_R) + c, c = max(c_L, c_R); the
  // selected argument takes the cotangent (the first one on ties)
  const double slb = rt ? Sob : Sab, srb = rt ? Sab : Sob;
  const double uob = (lo_o ? slb : 0.0) + (hi_o ? srb : 0.0);
  wob[1] += uob;
  wb[1] += slb + srb - uob;
  {
    double wc[7], wcb[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    constexpr int touched[4] = {0, 4, 5, 6};  // rho, B_t1, B_t2, p
#pragma unroll
    for (int e = 0; e < 4; ++e) wc[touched[e]] = c_o ? wo[touched[e]] : w[touched[e]];
    cfast_vjp(g, wc, bn, srb - slb, wcb, bnb);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = touched[e];
      wob[q] += c_o ? wcb[q] : 0.0;
      wb[q] += c_o ? 0.0 : wcb[q];
    }
  }
  phys_vjp<B4, B5>(igm1, w, bn, fbar, 1.0, be, ub6, ptab, wb, bnb);
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    wlb[q] = rt ? wob[q] : wb[q];
    wrb[q] = rt ? wb[q] : wob[q];
  }
}

template <int RS, bool B4, bool B5>
__device__ __forceinline__ void riemann_vjp(double g, const double* wl, const double* wr, double bn,
                                            const double* fbar, double apbar, double ambar,
                                            double v1bar, double v2bar, double* wlb, double* wrb,
                                            double& bnb) {
  if constexpr (RS == 0)
    hlld_vjp<B4, B5>(g, wl, wr, bn, fbar, apbar, ambar, v1bar, v2bar, wlb, wrb, bnb);
  else
    hll_vjp<B4, B5>(g, wl, wr, bn, fbar, apbar, ambar, v1bar, v2bar, wlb, wrb, bnb);
}

// Edge-partial slots: d E / d input times Ebar.
enum : int { E_APA = 0, E_AMA, E_VW, E_BW, E_VE, E_BE, E_APB, E_AMB, E_VS, E_BS, E_VN, E_BN, NE };

struct Bufs {
  double* EB;    // 3 components x NE x n
  double* WB;    // 3 directions x 14 x n: wL-bar (7), wR-bar (7)
  double* BF;    // 3 x n: staggered-field cotangent gathered at each face
  double* BC;    // 3 x n: cell-centred field cotangent
  double* T;     // 8 x n: J^T G of the cell-averaged fields
  double* A;     // 8 x n: cotangent of the stage-1 state
  double* PW;    // 8 x n: FP64 primitives of the state the stage adjoint linearises at
  double* FWn;   // dim x NSLOT x n: face records at U_n (kept from the stage-1 forward)
  double* EWn;   // 3 x n: edge EMFs at U_n
  // SSP-RK3 only (nullptr otherwise):
  double* FW1;   // dim x NSLOT x n: face records at U1 (kept from the stage-2 forward)
  double* EW1;   // 3 x n: edge EMFs at U1
  double* A1;    // 8 x n: cotangent of the stage-1 state
  double* part;  // (2 or 3) x nblocks: dtbar partial sums, one set per stage
};

// Byte offset within one field of the cell shifted by s (|s| <= 2) along D. 32
// bits (the launcher checks): a load then takes the field's base from scalar
// registers and the offset from one vector register, where 64-bit indices cost
// an address addition per load.
template <int D>
__device__ __forceinline__ uint32_t shift_off(const Geom& g, int i, int j, int k, int s) {
  const int ii = D == 0 ? wrap(i + s, g.nx) : i, jj = D == 1 ? wrap(j + s, g.ny) : j;
  const int kk = D == 2 ? wrap(k + s, g.nz) : k;
  return (((uint32_t)kk * (uint32_t)g.ny + (uint32_t)jj) * (uint32_t)g.nx + (uint32_t)ii) * 8u;
}
__device__ __forceinline__ void st_at(double* b, uint32_t off, double v) {
  *reinterpret_cast<double*>(reinterpret_cast<char*>(b) + off) = v;
}

template <int D>
__device__ __forceinline__ double delta(const Geom& g) {
  return D == 0 ? g.dx : (D == 1 ? g.dy : g.dz);
}

// ---------------------------------------------------------------------------
template <int C, int LIM>
__device__ __forceinline__ void edge_partials(const double* __restrict__ U,
                                              const double* __restrict__ FW,
                                              const double* __restrict__ G, double s,
                                              const Geom& g, int i, int j, int k, uint32_t c,
                                              double* __restrict__ EB) {
  constexpr int A = (C + 1) % 3, B = (C + 2) % 3;
  const int64_t n = g.n;
  const double* fa = FW + (int64_t)A * NSLOT * n;
  const double* fb = FW + (int64_t)B * NSLOT * n;
  const uint32_t cmb = shift_off<B>(g, i, j, k, -1);
  const uint32_t cma = shift_off<A>(g, i, j, k, -1);
  // Ebar = sum over the four faces whose -curl E uses this edge
  const double* GA = G + (F_BX + A) * n;
  const double* GB = G + (F_BX + B) * n;
  const double eb = s * ((ld_at(GA, c) - ld_at(GA, cmb)) / delta<B>(g) - (ld_at(GB, c) - ld_at(GB, cma)) / delta<A>(g));
  const double apa = max_r(ld_at(fa + S_AP * n, cmb), ld_at(fa + S_AP * n, c));
  const double ama = max_r(ld_at(fa + S_AM * n, cmb), ld_at(fa + S_AM * n, c));
  const double apb = max_r(ld_at(fb + S_AP * n, cma), ld_at(fb + S_AP * n, c));
  const double amb = max_r(ld_at(fb + S_AM * n, cma), ld_at(fb + S_AM * n, c));
  const uint32_t a2 = shift_off<A>(g, i, j, k, -2), a1 = shift_off<A>(g, i, j, k, 1);
  const uint32_t b2 = shift_off<B>(g, i, j, k, -2), b1 = shift_off<B>(g, i, j, k, 1);
  const double* vbA = fb + S_V2 * n;
  const double* bB = U + (F_BX + B) * n;
  const double* vaB = fa + S_V1 * n;
  const double* bA = U + (F_BX + A) * n;
  double vW, vE, bW, bE, vS, vN, bS, bN;
  edge_pair<LIM, double>(ld_at(vbA, a2), ld_at(vbA, cma), ld_at(vbA, c), ld_at(vbA, a1), vW, vE);
  edge_pair<LIM, double>(ld_at(bB, a2), ld_at(bB, cma), ld_at(bB, c), ld_at(bB, a1), bW, bE);
  edge_pair<LIM, double>(ld_at(vaB, b2), ld_at(vaB, cmb), ld_at(vaB, c), ld_at(vaB, b1), vS, vN);
  edge_pair<LIM, double>(ld_at(bA, b2), ld_at(bA, cmb), ld_at(bA, c), ld_at(bA, b1), bS, bN);
  // E = tb - ta
  const double isa = 1.0 / (apa + ama), isb = 1.0 / (apb + amb);
  const double ta = (apa * vW * bW + ama * vE * bE - apa * ama * (bE - bW)) * isa;
  const double tb = (apb * vS * bS + amb * vN * bN - apb * amb * (bN - bS)) * isb;
  double* e = EB + (int64_t)C * NE * n;
  st_at(e + E_VW * n, c, -eb * apa * bW * isa);
  st_at(e + E_BW * n, c, -eb * apa * (vW + ama) * isa);
  st_at(e + E_VE * n, c, -eb * ama * bE * isa);
  st_at(e + E_BE * n, c, -eb * ama * (vE - apa) * isa);
  st_at(e + E_APA * n, c, -eb * (vW * bW - ama * (bE - bW) - ta) * isa);
  st_at(e + E_AMA * n, c, -eb * (vE * bE - apa * (bE - bW) - ta) * isa);
  st_at(e + E_VS * n, c, eb * apb * bS * isb);
  st_at(e + E_BS * n, c, eb * apb * (vS + amb) * isb);
  st_at(e + E_VN * n, c, eb * amb * bN * isb);
  st_at(e + E_BN * n, c, eb * amb * (vN - apb) * isb);
  st_at(e + E_APB * n, c, eb * (vS * bS - amb * (bN - bS) - tb) * isb);
  st_at(e + E_AMB * n, c, eb * (vN * bN - apb * (bN - bS) - tb) * isb);
}

// Workgroup order of the 3D gather kernels: logical index t (consecutive 64 go
// to one XCD, xcd_grouped) -> workgroup of kBlock consecutive cells. With P
// workgroups to a plane (about), the order runs through bricks of 8 planes x 8
// workgroups, so that the 64 workgroups an XCD works on together reach each
// other's planes above and below through its L2. A permutation of 0 .. nb-1;
// the remainder past whole blocks of 8 planes keeps its order.
__device__ __forceinline__ unsigned brick_order(unsigned t, unsigned nb, unsigned P) {
  const unsigned slab = 8u * P;  // workgroups of 8 planes
  const unsigned s = t / slab;
  if ((s + 1u) * slab > nb) return t;
  const unsigned r = t - s * slab;
  const unsigned col = r / 64u;           // brick: 8 workgroups wide, the last one narrower
  const unsigned w = min(8u, P - col * 8u);
  const unsigned q = r - col * 64u;
  const unsigned z = q / w;
  return s * slab + z * P + col * 8u + (q - z * w);
}
template <int DIM>
__device__ __forceinline__ int64_t adj_cell(const Geom& g) {
  const unsigned t = xcd_grouped(blockIdx.x, gridDim.x);
  if (DIM == 2) return (int64_t)t * kBlock + threadIdx.x;
  const unsigned P = (unsigned)max(1, (int)(((int64_t)g.nx * g.ny) / kBlock));
  return (int64_t)brick_order(t, gridDim.x, P) * kBlock + threadIdx.x;
}

template <int DIM, int LIM>
__global__ __launch_bounds__(kBlock) void k_adj_edges(const double* __restrict__ U,
                                                      const double* __restrict__ FW,
                                                      const double* __restrict__ G, double s,
                                                      Geom g, double* __restrict__ EB) {
  // XCD-grouped workgroup order: the rows above and below, which the stencil
  // reads, mostly come through the same L2 (KH 512^2 adjoint 2878 -> 3041
  // steps/s, blast 256^3 30.5 -> 31.1, for edges, faces and cells together)
  const int64_t c = adj_cell<DIM>(g);
  if (c >= g.n) return;
  int i, j, k;
  coords(g, c, i, j, k);
  const uint32_t o = (uint32_t)c * 8u;
  if (DIM == 3) {
    edge_partials<0, LIM>(U, FW, G, s, g, i, j, k, o, EB);
    edge_partials<1, LIM>(U, FW, G, s, g, i, j, k, o, EB);
  }
  edge_partials<2, LIM>(U, FW, G, s, g, i, j, k, o, EB);
}

// ---------------------------------------------------------------------------
// Cotangents a face receives from the edges of component C that use it.
// ROLE 0: the face is an a-face of C (normal A = D), its v_B (slot V1) and
// b_D are reconstructed along B; ROLE 1: a b-face (normal B = D), its v_A
// (slot V2) and b_D along A. Split into the loads (edge_load) and the
// arithmetic (edge_apply), so that a face's loads all go out before any of
// its arithmetic waits for one.
struct EdgeIn {
  double apm, ap0, app, amm, am0, amp;  // alpha+- of the faces c-e, c, c+e
  double ea0, eap, em0, emp;            // alpha cotangents of the edges at c, c+e
  double xv[5], xb[5];                  // v and b on the faces c-2e .. c+2e
  double vp[3], vm[3], bp[3], bm[3];    // cotangents of their edge values
};

template <int C, int ROLE>
__device__ __forceinline__ void edge_load(const double* __restrict__ U,
                                          const double* __restrict__ FW,
                                          const double* __restrict__ EB, const Geom& g, int i,
                                          int j, int k, uint32_t c, EdgeIn& in) {
  constexpr int A = (C + 1) % 3, B = (C + 2) % 3;
  constexpr int D = ROLE == 0 ? A : B;      // this face's normal
  constexpr int E = ROLE == 0 ? B : A;      // reconstruction / neighbour direction
  constexpr int sap = ROLE == 0 ? E_APA : E_APB, sam = ROLE == 0 ? E_AMA : E_AMB;
  constexpr int svlo = ROLE == 0 ? E_VS : E_VW, svhi = ROLE == 0 ? E_VN : E_VE;
  constexpr int sblo = ROLE == 0 ? E_BS : E_BW, sbhi = ROLE == 0 ? E_BN : E_BE;
  const int64_t n = g.n;
  const double* f = FW + (int64_t)D * NSLOT * n;
  const double* e = EB + (int64_t)C * NE * n;
  const uint32_t cm1 = shift_off<E>(g, i, j, k, -1), cp1 = shift_off<E>(g, i, j, k, 1);
  const uint32_t cm2 = shift_off<E>(g, i, j, k, -2), cp2 = shift_off<E>(g, i, j, k, 2);
  const double* ap = f + S_AP * n;
  const double* am = f + S_AM * n;
  in.apm = ld_at(ap, cm1); in.ap0 = ld_at(ap, c); in.app = ld_at(ap, cp1);
  in.amm = ld_at(am, cm1); in.am0 = ld_at(am, c); in.amp = ld_at(am, cp1);
  in.ea0 = ld_at(e + sap * n, c); in.eap = ld_at(e + sap * n, cp1);
  in.em0 = ld_at(e + sam * n, c); in.emp = ld_at(e + sam * n, cp1);
  const double* v = f + (ROLE == 0 ? S_V1 : S_V2) * n;
  const double* b = U + (F_BX + D) * n;
  const uint32_t c5[5] = {cm2, cm1, c, cp1, cp2};
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    in.xv[s] = ld_at(v, c5[s]);
    in.xb[s] = ld_at(b, c5[s]);
  }
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    in.vp[s] = ld_at(e + svlo * n, c5[s + 2]);
    in.vm[s] = ld_at(e + svhi * n, c5[s + 1]);
    in.bp[s] = ld_at(e + sblo * n, c5[s + 2]);
    in.bm[s] = ld_at(e + sbhi * n, c5[s + 1]);
  }
}

template <int LIM>
__device__ __forceinline__ void edge_apply(EdgeIn& in, double& apbar, double& ambar,
                                           double& vbar, double& bbar) {
  // the empty asm keeps the compiler from sinking the four alpha cotangent
  // loads into the branches that add them (one round trip each)
  asm volatile("" : "+v"(in.ea0), "+v"(in.eap), "+v"(in.em0), "+v"(in.emp));
  // alpha: the edge at c takes max(face c-e, face c); the edge at c+e takes
  // max(face c, face c+e); the first argument wins ties.
  apbar = (in.ap0 > in.apm) ? apbar + in.ea0 : apbar;
  apbar = !(in.app > in.ap0) ? apbar + in.eap : apbar;
  ambar = (in.am0 > in.amm) ? ambar + in.em0 : ambar;
  ambar = !(in.amp > in.am0) ? ambar + in.emp : ambar;
  // reconstructed values: upper extrapolation of face p feeds the edge at
  // p+e (as its lower value), the lower extrapolation feeds the edge at p
  vbar += plm_adjoint<LIM>(in.xv, in.vp, in.vm);
  bbar += plm_adjoint<LIM>(in.xb, in.bp, in.bm);
}

// Reconstructed face-frame states of the lower D-face of cell (i,j,k) as
// the forward kernels form them, from the recovered primitives PW of the four cells
// c-2..c+1 along D (the values primitive recovery gives, computed once per
// cell by k_adj_prim): pw_load gathers the 28 values, pw_states reconstructs.
template <int D>
__device__ __forceinline__ void pw_load(const double* __restrict__ PW, const Geom& g, int i,
                                        int j, int k, double (&v)[7][4]) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  constexpr int slot[7] = {0, 1 + D, 1 + T1, 1 + T2, 5 + T1, 5 + T2, 4};
  const int64_t n = g.n;
  uint32_t cs[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) cs[s] = shift_off<D>(g, i, j, k, s - 2);
#pragma unroll
  for (int q = 0; q < 7; ++q)
#pragma unroll
    for (int s = 0; s < 4; ++s) v[q][s] = ld_at(PW + (int64_t)slot[q] * n, cs[s]);
}
template <int LIM>
__device__ __forceinline__ void pw_states(const double (&v)[7][4], double* wl, double* wr) {
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    const double a = v[q][0], b = v[q][1], c = v[q][2], e = v[q][3];
    plm_pair<LIM, double>(a, b, c, e, wl[q], wr[q]);
  }
}

// FP64 primitives of every cell of the stage's state, once, for the face and
// cell kernels of the stage adjoint (which read each cell's from up to
// thirteen stencils).
template <int DIM>
__global__ __launch_bounds__(kBlock) void k_adj_prim(const double* __restrict__ U,
                                                     double* __restrict__ PW, Geom g) {
  const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (c >= g.n) return;
  int i, j, k;
  coords(g, c, i, j, k);
  double V[8];
  prim_at<DIM>(U, g, i, j, k, V);
#pragma unroll
  for (int q = 0; q < 8; ++q) PW[q * g.n + c] = V[q];
}

template <int DIM, int D, int LIM, int RS>
__device__ __forceinline__ void face_adjoint(const double* __restrict__ U,
                                             const double* __restrict__ FW,
                                             const double* __restrict__ G, double s,
                                             const double* __restrict__ EB, const Geom& g, int i,
                                             int j, int k, uint32_t c, const Bufs& bf) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  constexpr int C1 = (D + 2) % 3;  // this face is an a-face of C1
  constexpr int C2 = (D + 1) % 3;  // and a b-face of C2
  constexpr bool E1 = (DIM == 3 || C1 == 2), E2 = (DIM == 3 || C2 == 2);
  const int64_t n = g.n;
  const uint32_t cm = shift_off<D>(g, i, j, k, -1);
  const double idl = s / delta<D>(g);
  // Gather: the values of the edges, then (2D: together with) the others, each
  // set issued before any of it is used. One set for a face of the 3D grid
  // would be 103 values, over what two waves per SIMD have registers for.
  double apbar = 0.0, ambar = 0.0, v1bar = 0.0, v2bar = 0.0, bbar = 0.0;
  EdgeIn e1, e2;
  if (E1) edge_load<C1, 0>(U, FW, EB, g, i, j, k, c, e1);
  if (E2) edge_load<C2, 1>(U, FW, EB, g, i, j, k, c, e2);
  if (DIM == 3) {
    __builtin_amdgcn_sched_barrier(0);
    if (E1) edge_apply<LIM>(e1, apbar, ambar, v1bar, bbar);
    if (E2) edge_apply<LIM>(e2, apbar, ambar, v2bar, bbar);
    __builtin_amdgcn_sched_barrier(0);
  }
  constexpr int NG = (DIM == 2) ? 6 : 5;
  constexpr int gq[6] = {0, F_MX + D, F_MX + T1, F_MX + T2, F_EN, F_BZ};
  double gc[NG], gm[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    gc[q] = ld_at(G + gq[q] * n, c);
    gm[q] = ld_at(G + gq[q] * n, cm);
  }
  double pv[7][4];
  pw_load<D>(bf.PW, g, i, j, k, pv);
  const double bn = ld_at(U + (F_BX + D) * n, c);
  __builtin_amdgcn_sched_barrier(0);
  if (DIM == 2) {
    if (E1) edge_apply<LIM>(e1, apbar, ambar, v1bar, bbar);
    if (E2) edge_apply<LIM>(e2, apbar, ambar, v2bar, bbar);
  }
  // flux cotangents (face frame: rho, m_n, m_t1, m_t2, B_t1, B_t2, E)
  double fb[7];
  fb[0] = (gc[0] - gm[0]) * idl;
  fb[1] = (gc[1] - gm[1]) * idl;
  fb[2] = (gc[2] - gm[2]) * idl;
  fb[3] = (gc[3] - gm[3]) * idl;
  fb[4] = 0.0;
  fb[5] = 0.0;
  fb[6] = (gc[4] - gm[4]) * idl;
  if (DIM == 2) {
    const double bz = (gc[NG - 1] - gm[NG - 1]) * idl;
    if (D == 0) fb[5] = bz; else fb[4] = bz;   // B_z is t2 of x-faces, t1 of y-faces
  }
  // Riemann vector-Jacobian product: one reverse sweep
  double wl[7], wr[7];
  pw_states<LIM>(pv, wl, wr);
  double* wb = bf.WB + (int64_t)D * 14 * n;
  double wlb[7], wrb[7], bnbar;
  riemann_vjp<RS, DIM == 2 && D == 1, DIM == 2 && D == 0>(
      g.gamma, wl, wr, bn, fb, apbar, ambar, v1bar, v2bar, wlb, wrb, bnbar);
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    st_at(wb + (int64_t)q * n, c, wlb[q]);
    st_at(wb + (int64_t)(7 + q) * n, c, wrb[q]);
  }
  st_at(bf.BF + (int64_t)D * n, c, bnbar + bbar);
  __builtin_amdgcn_sched_barrier(0);  // the next face's gather stays behind this sweep
}

// What bounds it: HBM (112 values per cell at the least) and the latency of its
// gathers. Two waves per SIMD, without spills (but 20 bytes a lane for HLL in 3D): the
// sweep in one copy for both sides, the gather in two sets, and nothing derived from
// the cell's place shared between the faces (here()). 192^3 3.12 -> 2.13 ms, KH 512^2 60 -> 41 us;
// capped at two waves with 170 bytes of spills 2.72 ms, one wave 2.55 ms.
template <int DIM, int LIM, int RS>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
void k_adj_faces(const double* __restrict__ U,
                                                      const double* __restrict__ FW,
                                                      const double* __restrict__ G, double s,
                                                      Geom g, Bufs bf) {
  const int64_t c = adj_cell<DIM>(g);
  if (c >= g.n) return;
  int i, j, k;
  coords(g, c, i, j, k);
  const uint32_t o = (uint32_t)c * 8u;
  face_adjoint<DIM, 0, LIM, RS>(U, FW, G, s, bf.EB, g, here(i), here(j), here(k), here(o), bf);
  face_adjoint<DIM, 1, LIM, RS>(U, FW, G, s, bf.EB, g, here(i), here(j), here(k), here(o), bf);
  if (DIM == 3)
    face_adjoint<DIM, 2, LIM, RS>(U, FW, G, s, bf.EB, g, here(i), here(j), here(k), here(o), bf);
}

// ---------------------------------------------------------------------------
template <int DIM, int D, int LIM>
__device__ __forceinline__ void plm_cell_adjoint(const double* __restrict__ PW,
                                                 const double* __restrict__ WB, const Geom& g,
                                                 int i, int j, int k, double* vbar) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  constexpr int slot[7] = {0, 1 + D, 1 + T1, 1 + T2, 5 + T1, 5 + T2, 4};
  const int64_t n = g.n;
  uint32_t cs[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) cs[s] = shift_off<D>(g, i, j, k, s - 2);
  double V[5][8];
#pragma unroll
  for (int s = 0; s < 5; ++s)
#pragma unroll
    for (int q = 0; q < 7; ++q) V[s][slot[q]] = ld_at(PW + (int64_t)slot[q] * n, cs[s]);
  // faces p (lower face of cell p) for p = c-1 .. c+2 along D
  uint32_t fidx[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) fidx[s] = shift_off<D>(g, i, j, k, s - 1);
  const double* w = WB + (int64_t)D * 14 * n;
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    const int sl = slot[q];
    const double x[5] = {V[0][sl], V[1][sl], V[2][sl], V[3][sl], V[4][sl]};
    // upper extrapolation of cell p = left state of face p+1;
    // lower extrapolation of cell p = right state of face p. (All 77 values of
    // a direction ahead of a scheduling barrier: three waves per SIMD instead
    // of six, 1.30 ms against 1.12 at 192^3.)
    const double xp[3] = {ld_at(w + q * n, fidx[1]), ld_at(w + q * n, fidx[2]),
                          ld_at(w + q * n, fidx[3])};
    const double xm[3] = {ld_at(w + (7 + q) * n, fidx[0]), ld_at(w + (7 + q) * n, fidx[1]),
                          ld_at(w + (7 + q) * n, fidx[2])};
    vbar[sl] += plm_adjoint<LIM>(x, xp, xm);
  }
}

template <int DIM, int LIM>
__global__ __launch_bounds__(kBlock) void k_adj_cells(const double* __restrict__ U, Geom g,
                                                      Bufs bf) {
  const int64_t c = adj_cell<DIM>(g);
  if (c >= g.n) return;
  int i, j, k;
  coords(g, c, i, j, k);
  const int64_t n = g.n;
  double vb[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  plm_cell_adjoint<DIM, 0, LIM>(bf.PW, bf.WB, g, i, j, k, vb);
  plm_cell_adjoint<DIM, 1, LIM>(bf.PW, bf.WB, g, i, j, k, vb);
  if (DIM == 3) plm_cell_adjoint<DIM, 2, LIM>(bf.PW, bf.WB, g, i, j, k, vb);
  // primitive recovery: v = m/rho, p = (gamma-1)(E - |m|^2/(2 rho) - |Bc|^2/2)
  double V[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) V[q] = bf.PW[q * n + c];
  const double gm1 = g.gamma - 1.0;
  const double pb = vb[4] * gm1;
  const double irho = 1.0 / V[0];
  const double v2 = V[1] * V[1] + V[2] * V[2] + V[3] * V[3];
  double trho = vb[0] + 0.5 * pb * v2;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    trho -= vb[1 + d] * V[1 + d] * irho;
    bf.T[(F_MX + d) * n + c] = vb[1 + d] * irho - pb * V[1 + d];
  }
  bf.T[c] = trho;
  bf.T[F_EN * n + c] = pb;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double bcb = vb[5 + d] - pb * V[5 + d];
    if (DIM == 2 && d == 2) bf.T[F_BZ * n + c] = bcb;  // cell-centred B_z
    else bf.BC[(int64_t)d * n + c] = bcb;
  }
}

// L(U) of cell (i,j,k) from the forward records, as the update kernel forms it.
template <int DIM>
__device__ __forceinline__ void stage_rhs(const double* __restrict__ FW,
                                          const double* __restrict__ EW, const Geom& g, int i,
                                          int j, int k, int64_t c, double* L) {
  const int64_t n = g.n;
  const int64_t xp = lin(g, wrap(i + 1, g.nx), j, k);
  const int64_t yp = lin(g, i, wrap(j + 1, g.ny), k);
  const double idx = 1.0 / g.dx, idy = 1.0 / g.dy;
  if constexpr (DIM == 3) {  // the cell fields' L as the face kernel left it
#pragma unroll
    for (int q = 0; q < 5; ++q) L[q] = FW[q * n + c];
  } else {
    const double* fx = FW;
    const double* fy = FW + (int64_t)NSLOT * n;
#pragma unroll
    for (int q = 0; q < 6; ++q)
      L[q == 5 ? 7 : q] = -((fx[q * n + xp] - fx[q * n + c]) * idx +
                            (fy[q * n + yp] - fy[q * n + c]) * idy);
  }
  if (DIM == 3) {  // and the field's as the CT kernel left it
#pragma unroll
    for (int d = 0; d < 3; ++d) L[5 + d] = EW[d * n + c];
  } else {
    const double* ez = EW + 2 * n;
    L[5] = -((ez[yp] - ez[c]) * idy);
    L[6] = (ez[xp] - ez[c]) * idx;
  }
}

// ---------------------------------------------------------------------------
// out = cd * Dir + s G + dt J^T (s G); DT: also the per-block partial of
// <s G, L(U)> (L(U) from the forward records), which only dt-bar needs.
template <int DIM, bool DT>
__global__ __launch_bounds__(kBlock) void k_adj_final(const double* __restrict__ G, double s,
                                                      const double* __restrict__ Dir, double cd,
                                                      const double* __restrict__ FW,
                                                      const double* __restrict__ EW, Geom g,
                                                      double dt, Bufs bf, double* out,
                                                      double* __restrict__ part) {
  const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double dot = 0.0;
  if (c < g.n) {
    int i, j, k;
    coords(g, c, i, j, k);
    const int64_t n = g.n;
    double jt[8];
#pragma unroll
    for (int q = 0; q < 5; ++q) jt[q] = bf.T[q * n + c];
    const int64_t xm = lin(g, wrap(i - 1, g.nx), j, k);
    const int64_t ym = lin(g, i, wrap(j - 1, g.ny), k);
    jt[5] = 0.5 * (bf.BC[c] + bf.BC[xm]) + bf.BF[c];
    jt[6] = 0.5 * (bf.BC[n + c] + bf.BC[n + ym]) + bf.BF[n + c];
    if (DIM == 3) {
      const int64_t zm = lin(g, i, j, wrap(k - 1, g.nz));
      jt[7] = 0.5 * (bf.BC[2 * n + c] + bf.BC[2 * n + zm]) + bf.BF[2 * n + c];
    } else {
      jt[7] = bf.T[F_BZ * n + c];
    }
    double L[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (DT) stage_rhs<DIM>(FW, EW, g, i, j, k, c, L);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double sg = s * G[q * n + c];
      double v = sg + dt * jt[q];
      if (Dir) v += cd * Dir[q * n + c];
      out[q * n + c] = v;
      if constexpr (DT) dot += sg * L[q];
    }
  }
  if constexpr (!DT) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off, 64);
  __shared__ double red[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = dot;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) r += red[w];
    part[blockIdx.x] = r;
  }
}

__global__ __launch_bounds__(1024) void k_sum_final(const double* __restrict__ part, int np,
                                                    double* __restrict__ out) {
  double acc = 0.0;
  for (int b = threadIdx.x; b < np; b += 1024) acc += part[b];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  __shared__ double red[16];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < 16; ++w) r += red[w];
    *out = r;
  }
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

Bufs carve(double* scratch, int dim, int64_t n, int integrator) {
  Bufs b;
  double* p = scratch;
  b.EB = p; p += 3 * NE * n;
  b.WB = p; p += 3 * 14 * n;
  b.BF = p; p += 3 * n;
  b.BC = p; p += 3 * n;
  b.T = p; p += 8 * n;
  b.A = p; p += 8 * n;
  b.PW = p; p += 8 * n;
  b.FWn = p; p += (int64_t)dim * NSLOT * n;
  b.EWn = p; p += 3 * n;
  b.FW1 = b.EW1 = b.A1 = nullptr;
  if (integrator == 1) {
    b.FW1 = p; p += (int64_t)dim * NSLOT * n;
    b.EW1 = p; p += 3 * n;
    b.A1 = p; p += 8 * n;
  }
  b.part = p;
  return b;
}

// J^T of one stage, combined: out = cd Dir + s G + dt J_L(U)^T (s G); the
// forward records FW/EW must hold the face/edge data at U.
template <int DIM, int LIM, int RS>
hipError_t stage_adjoint(const AdjointArgs& a, const Bufs& bf, const double* U, const double* FW,
                         const double* EW, const double* G, double s, const double* Dir,
                         double cd, double* out, double* part) {
  const unsigned nb = blocks_for(a.g.n);
  hipLaunchKernelGGL((k_adj_prim<DIM>), dim3(nb), dim3(kBlock), 0, a.stream, U, bf.PW, a.g);
  hipLaunchKernelGGL((k_adj_edges<DIM, LIM>), dim3(nb), dim3(kBlock), 0, a.stream, U, FW, G, s,
                     a.g, bf.EB);
  hipLaunchKernelGGL((k_adj_faces<DIM, LIM, RS>), dim3(nb), dim3(kBlock), 0, a.stream, U, FW, G,
                     s, a.g, bf);
  hipLaunchKernelGGL((k_adj_cells<DIM, LIM>), dim3(nb), dim3(kBlock), 0, a.stream, U, a.g, bf);
  if (a.want_dtbar)
    hipLaunchKernelGGL((k_adj_final<DIM, true>), dim3(nb), dim3(kBlock), 0, a.stream, G, s, Dir,
                       cd, FW, EW, a.g, a.dt, bf, out, part);
  else
    hipLaunchKernelGGL((k_adj_final<DIM, false>), dim3(nb), dim3(kBlock), 0, a.stream, G, s, Dir,
                       cd, FW, EW, a.g, a.dt, bf, out, part);
  return hipGetLastError();
}

// Elementwise out = a x + b y (n doubles).
__global__ __launch_bounds__(kBlock) void k_axpby(const double* __restrict__ x, double a,
                                                  const double* __restrict__ y, double b,
                                                  double* __restrict__ out, int64_t n) {
  const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (c < n) out[c] = a * x[c] + b * y[c];
}

// Adjoint of one SSP-RK3 step (Eq. (RK3)): U1 = Un + dt L(Un),
// U2 = 3/4 Un + 1/4 (U1 + dt L(U1)), U3 = 1/3 Un + 2/3 (U2 + dt L(U2)).
// With G = Ubar of U3, in reverse:
//   A2 = 2/3 (G + dt J(U2)^T G)        (cotangent of U2)
//   A1 = 1/4 (A2 + dt J(U1)^T A2)      (cotangent of U1)
//   Ubar_n = 3/4 A2 + 1/3 G + A1 + dt J(Un)^T A1,
// and dtbar = sum over the stages of (s G_stage) . L(U_stage). The forward
// pass keeps the face/edge records at Un and U1 and recomputes those at U2;
// the direct term 3/4 A2 + 1/3 G goes to the space of U2, which nothing reads
// after the last stage's adjoint.
template <int DIM, int LIM, int RS>
hipError_t adjoint_rk3(const AdjointArgs& a, const Bufs& bf, StageArgs f) {
  const int64_t n = a.g.n;
  const unsigned nb = blocks_for(n);
  if (!a.U2 || !bf.FW1) return hipErrorInvalidValue;
  f.stage = 1;  // U1 = Un + dt L(Un), records at Un kept
  f.U = a.Un;
  f.U0 = nullptr;
  f.out = a.U1;
  f.FW = bf.FWn;
  f.EW = bf.EWn;
  hipError_t e = launch_stage(f);
  if (e != hipSuccess) return e;
  f.stage = 4;  // U2 = (3 Un + (U1 + dt L(U1))) / 4, records at U1 kept
  f.U = a.U1;
  f.U0 = a.Un;
  f.out = a.U2;
  f.FW = bf.FW1;
  f.EW = bf.EW1;
  e = launch_stage(f);
  if (e != hipSuccess) return e;
  f.stage = 3;  // records at U2
  f.U = a.U2;
  f.U0 = nullptr;
  f.FW = a.FW;
  f.EW = a.EW;
  e = launch_stage(f);
  if (e != hipSuccess) return e;
  e = stage_adjoint<DIM, LIM, RS>(a, bf, a.U2, a.FW, a.EW, a.Ubar1, 2.0 / 3.0, nullptr, 0.0, bf.A,
                                  bf.part);
  if (e != hipSuccess) return e;
  const unsigned n8 = (unsigned)((8 * n + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_axpby, dim3(n8), dim3(kBlock), 0, a.stream, bf.A, 0.75, a.Ubar1,
                     1.0 / 3.0, a.U2, 8 * n);
  e = stage_adjoint<DIM, LIM, RS>(a, bf, a.U1, bf.FW1, bf.EW1, bf.A, 0.25, nullptr, 0.0, bf.A1,
                                  bf.part + nb);
  if (e != hipSuccess) return e;
  e = stage_adjoint<DIM, LIM, RS>(a, bf, a.Un, bf.FWn, bf.EWn, bf.A1, 1.0, a.U2, 1.0, a.Ubar0,
                                  bf.part + 2 * nb);
  if (e != hipSuccess) return e;
  if (a.want_dtbar)
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(1024), 0, a.stream, bf.part, (int)(3 * nb),
                       a.dtbar_dev);
  return hipGetLastError();
}

template <int DIM, int LIM, int RS>
hipError_t adjoint_impl(const AdjointArgs& a) {
  const int64_t n = a.g.n;
  const Bufs bf = carve(a.scratch, a.dim, n, a.integrator);
  const unsigned nb = blocks_for(n);
  StageArgs f{};
  f.dim = a.dim;
  f.limiter = a.limiter;
  f.riemann = a.riemann;
  f.precision = 0;
  f.g = a.g;
  f.FW = a.FW;
  f.EW = a.EW;
  f.dt = a.dt;
  f.dtp = nullptr;
  f.records = a.dim == 2;
  f.keep_rhs = a.dim == 3 && a.want_dtbar;  // L(U) for dt-bar
  f.flag = a.flag;
  f.stream = a.stream;
  f.timer = nullptr;
  if (a.integrator == 1) return adjoint_rk3<DIM, LIM, RS>(a, bf, f);
  // forward stage 1: U1 = Un + dt L(Un); its face/edge records at Un are
  // kept (FWn, EWn) for the stage-1 adjoint
  f.stage = 1;
  f.U = a.Un;
  f.U0 = nullptr;
  f.out = a.U1;
  f.FW = bf.FWn;
  f.EW = bf.EWn;
  hipError_t e = launch_stage(f);
  if (e != hipSuccess) return e;
  // records at U1, then the stage-2 adjoint: A = G2 + dt J(U1)^T G2, G2 = Ubar1/2
  f.stage = 3;
  f.U = a.U1;
  f.FW = a.FW;
  f.EW = a.EW;
  e = launch_stage(f);
  if (e != hipSuccess) return e;
  e = stage_adjoint<DIM, LIM, RS>(a, bf, a.U1, a.FW, a.EW, a.Ubar1, 0.5, nullptr, 0.0, bf.A,
                                  bf.part);
  if (e != hipSuccess) return e;
  // the stage-1 adjoint at Un: Ubar0 = Ubar1/2 + A + dt J(Un)^T A
  e = stage_adjoint<DIM, LIM, RS>(a, bf, a.Un, bf.FWn, bf.EWn, bf.A, 1.0, a.Ubar1, 0.5, a.Ubar0,
                                  bf.part + nb);
  if (e != hipSuccess) return e;
  if (a.want_dtbar)
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(1024), 0, a.stream, bf.part, (int)(2 * nb),
                       a.dtbar_dev);
  return hipGetLastError();
}

template <int DIM>
hipError_t adjoint_dim(const AdjointArgs& a) {
  if (a.limiter == 0)
    return a.riemann == 0 ? adjoint_impl<DIM, 0, 0>(a) : adjoint_impl<DIM, 0, 1>(a);
  return a.riemann == 0 ? adjoint_impl<DIM, 1, 0>(a) : adjoint_impl<DIM, 1, 1>(a);
}

}  // namespace

size_t adjoint_workspace_bytes(int dim, size_t ncell, int integrator) {
  const size_t nb = (ncell + kBlock - 1) / kBlock;
  size_t per_cell = 3 * NE + 3 * 14 + 3 + 3 + 8 + 8 + 8 + (size_t)dim * NSLOT + 3;
  if (integrator == 1) per_cell += (size_t)dim * NSLOT + 3 + 8;  // FW1, EW1, A1
  return sizeof(double) * (per_cell * ncell + (integrator == 1 ? 3 : 2) * nb) + 256;
}

hipError_t launch_adjoint_step(const AdjointArgs& a) {
  // 32-bit byte offsets within a field (the workspace of such a grid would be
  // over 680 GB)
  if (a.g.n >= (int64_t)1 << 29) return hipErrorNotSupported;
  return (a.dim == 3) ? adjoint_dim<3>(a) : adjoint_dim<2>(a);
}

}  // namespace mhd
