// residual.hip -- right-hand side of the first split sweep (paper eq. (spl1)):
//   R = -(Uk - Un) - tau * F_h(Ubar),  Ubar = (Uk + Un)/2,
// F_h(V) = (D + D_M)(V) V + G is the full discrete operator of the
// non-conservative system (nonconservmass)-(nonconservener) in spherical
// components (Appendix B): advection with curvature terms, pressure gradient,
// compressibility terms, viscosity, viscous heating, heat conduction,
// Coriolis and gravity.
//
// Viscosity: -(mu/rho) (Lap u + grad div u / 3) = -(mu/rho) V with
// V = (4/3) grad(div u) - curl(curl u) on the MAC complex: the divergence at
// cell centres, the vorticity at cell edges (circulation round the dual face
// over its area), its curl at a face (circulation round the face over the
// face area).  Then div(curl) vanishes identically and a discretely
// solenoidal velocity field keeps a solenoidal viscous update.  A radial
// circulation r_a u_a - r_b u_b over centres r_a = r_f + dr/2, r_b = r_f - dr/2
// is formed as r_f (u_a - u_b) + dr (u_a + u_b) / 2 (the same value, without
// the cancellation of two products of size r).  The phi rows next to a pole
// keep the component form (the edge vorticity on the polar axis is one value
// for the whole ring).
//
// A thread owns the centre (i,j,k) and the three faces with the same indices of
// the extended index space (nr+1) x (nt+1) x npf.  Inside a step the midpoint is
// resident (written by the previous iteration's phi sweep, or U^n itself at the
// first); the C-ABI call forms it from Un and Uk and writes it.  The launches,
// by size:
//   * large grids: the interior's r planes walked through a window in LDS, the
//     shell in the same launch or one of its own (k_residual_march, _march_mid
//     with k_residual_mid_shell for the C-ABI call, _marchB for a batch);
//   * smaller ones: interior and shell in one launch (k_residual_one; a batch
//     k_residual_in and k_residual; the C-ABI call k_residual_mid, or k_midpoint
//     and then k_residual_one);
//   * what these launches' dimensions or 32-bit indices do not hold: every point
//     by the general rules (k_residual).
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "dsw_common.hpp"
#include "dsw_internal.hpp"
#include "kargs.hpp"
#include "rows_fast.hpp"

namespace dsw {

template <class S>
__device__ __forceinline__ double F_p_T(const Geo &g, const Mat &m, const S &s, int i, int j, int k, double *FT) {
  Cent c;
  centre(g, m, s, i, j, k, c);
  const double ir = g.irc[i], is = g.isc[j];
  const double hr = 0.5 * g.idr, ht = 0.5 * ir * g.idt, hp = 0.5 * ir * is * g.idp;
  double dpr = gC(g, s, F_P, i + 1, j, k) - gC(g, s, F_P, i - 1, j, k);
  // perturbation form: the reference column's gradient joins the r difference
  if constexpr (S::PERT) dpr += s.pref[min(i + 1, g.nr - 1)] - s.pref[max(i - 1, 0)];
  const double advp = c.ur * dpr * hr +
                      c.ut * (gC(g, s, F_P, i, j + 1, k) - gC(g, s, F_P, i, j - 1, k)) * ht +
                      c.uf * (gC(g, s, F_P, i, j, k + 1) - gC(g, s, F_P, i, j, k - 1)) * hp;
  const double Tim = gC(g, s, F_T, i - 1, j, k), Tip = gC(g, s, F_T, i + 1, j, k);
  const double Tjm = gC(g, s, F_T, i, j - 1, k), Tjp = gC(g, s, F_T, i, j + 1, k);
  const double Tkm = gC(g, s, F_T, i, j, k - 1), Tkp = gC(g, s, F_T, i, j, k + 1);
  const double advT = c.ur * (Tip - Tim) * hr + c.ut * (Tjp - Tjm) * ht + c.uf * (Tkp - Tkm) * hp;
  const double T0 = c.T, ir2 = ir * ir;
  const double lap =
      (g.rf[i + 1] * g.rf[i + 1] * (Tip - T0) - g.rf[i] * g.rf[i] * (T0 - Tim)) * (ir2 * g.idr * g.idr) +
      (g.sf[j + 1] * (Tjp - T0) - g.sf[j] * (T0 - Tjm)) * (ir2 * is * g.idt * g.idt) +
      (Tkp - 2.0 * T0 + Tkm) * (ir2 * is * is * g.idp * g.idp);
  const double phi = m.mu * (2.0 * (c.Grr * c.Grr + c.Gtt * c.Gtt + c.Gff * c.Gff) + c.Srt * c.Srt +
                             c.Srf * c.Srf + c.Stf * c.Stf - (2.0 / 3.0) * c.tr * c.div);
  *FT = advT + (m.gam - 1.0) * c.T * c.div - c.chi * phi - c.chi * m.kap * lap;
  return advp + m.gam * c.P * c.div - (m.gam - 1.0) * phi - (m.gam - 1.0) * m.kap * lap;
}

template <class S>
__device__ __forceinline__ double F_ur(const Geo &g, const Mat &m, const S &s, int f, int j, int k) {
  const double irF = g.irf[f], is = g.isc[j];
  const double irho = irho_mean(g, m, s, f - 1, j, k, f, j, k);
  const double nu = m.mu * irho;
  const double un = gR(g, s, f, j, k);
  const double ua = 0.25 * (gT(g, s, f - 1, j, k) + gT(g, s, f - 1, j + 1, k) + gT(g, s, f, j, k) +
                            gT(g, s, f, j + 1, k));
  const double ub = 0.25 * (gF(g, s, f - 1, j, k) + gF(g, s, f - 1, j, k + 1) + gF(g, s, f, j, k) +
                            gF(g, s, f, j, k + 1));
  const double xp = gR(g, s, f + 1, j, k), xm = gR(g, s, f - 1, j, k);
  const double yp = gR(g, s, f, j + 1, k), ym = gR(g, s, f, j - 1, k);
  const double zp = gR(g, s, f, j, k + 1), zm = gR(g, s, f, j, k - 1);
  double N = (gC(g, s, F_P, f, j, k) - gC(g, s, F_P, f - 1, j, k)) * (irho * g.idr);
  N += un * (xp - xm) * (0.5 * g.idr) + ua * (yp - ym) * (0.5 * irF * g.idt) +
       ub * (zp - zm) * (0.5 * irF * is * g.idp) - (ua * ua + ub * ub) * irF;
  const double gd = (divc(g, s, f, j, k) - divc(g, s, f - 1, j, k)) * g.idr;
  // vorticity: omega_phi at the edges (f, j) and (f, j + 1), omega_theta at
  // the edges (f, k) and (f, k + 1); C = (curl omega)_r
  const double T00 = gT(g, s, f - 1, j, k), T01 = gT(g, s, f - 1, j + 1, k);
  const double T10 = gT(g, s, f, j, k), T11 = gT(g, s, f, j + 1, k);
  const double F00 = gF(g, s, f - 1, j, k), F01 = gF(g, s, f - 1, j, k + 1);
  const double F10 = gF(g, s, f, j, k), F11 = gF(g, s, f, j, k + 1);
  const double wp0 = (T10 - T00) * g.idr + 0.5 * (T10 + T00) * irF - (un - ym) * (irF * g.idt);
  const double wp1 = (T11 - T01) * g.idr + 0.5 * (T11 + T01) * irF - (yp - un) * (irF * g.idt);
  const double wt0 = (un - zm) * (irF * is * g.idp) - (F10 - F00) * g.idr - 0.5 * (F10 + F00) * irF;
  const double wt1 = (zp - un) * (irF * is * g.idp) - (F11 - F01) * g.idr - 0.5 * (F11 + F01) * irF;
  const double C = ((g.sf[j + 1] * wp1 - g.sf[j] * wp0) * g.idt - (wt1 - wt0) * g.idp) * (irF * is);
  const double vis = gd - C;  // nu (vis + gd / 3) = nu ((4/3) gd - C)
  N += -2.0 * m.omega * g.sc[j] * ub;
  if constexpr (S::PERT) {
    // perturbation form: the gradient of p' above, and gravity less the
    // reference column's balanced gradient, g (rho_f - rhobar_f) / rho_f,
    // with rho - rhobar = (p' Tbar - (pbar + pi_inf)(T - Tbar)) / (R T Tbar)
    const double Ta = gC(g, s, F_T, f - 1, j, k), Tb = gC(g, s, F_T, f, j, k);
    const double ta = s.tref[f - 1], tb = s.tref[f];
    const double da = (gC(g, s, F_P, f - 1, j, k) * ta - (s.pref[f - 1] + m.pinf) * (Ta - ta)) * rcp_nr(m.Rg * Ta * ta);
    const double db = (gC(g, s, F_P, f, j, k) * tb - (s.pref[f] + m.pinf) * (Tb - tb)) * rcp_nr(m.Rg * Tb * tb);
    return N - nu * vis - nu * (1.0 / 3.0) * gd + m.g_r * (0.5 * (da + db)) * irho;
  } else {
    return N - nu * vis - nu * (1.0 / 3.0) * gd + m.g_r;
  }
}

template <class S>
__device__ __forceinline__ double F_ut(const Geo &g, const Mat &m, const S &s, int i, int f, int k) {
  const double ir = g.irc[i], isF = g.isf[f], ctF = g.ctf[f];
  const int j0 = f - 1, j1 = f;
  const double irho = irho_mean(g, m, s, i, j0, k, i, j1, k);
  const double nu = m.mu * irho;
  const double un = gT(g, s, i, f, k);
  const double ua = 0.25 * (gR(g, s, i, j0, k) + gR(g, s, i, j1, k) + gR(g, s, i + 1, j0, k) +
                            gR(g, s, i + 1, j1, k));
  const double ub = 0.25 * (gF(g, s, i, j0, k) + gF(g, s, i, j0, k + 1) + gF(g, s, i, j1, k) +
                            gF(g, s, i, j1, k + 1));
  const double xp = gT(g, s, i + 1, f, k), xm = gT(g, s, i - 1, f, k);
  const double yp = gT(g, s, i, f + 1, k), ym = gT(g, s, i, f - 1, k);
  const double zp = gT(g, s, i, f, k + 1), zm = gT(g, s, i, f, k - 1);
  double N = (gC(g, s, F_P, i, j1, k) - gC(g, s, F_P, i, j0, k)) * (irho * ir * g.idt);
  N += ua * (xp - xm) * (0.5 * g.idr) + un * (yp - ym) * (0.5 * ir * g.idt) +
       ub * (zp - zm) * (0.5 * ir * isF * g.idp) + (un * ua - ub * ub * ctF) * ir;
  const double gd = (divc(g, s, i, j1, k) - divc(g, s, i, j0, k)) * (ir * g.idt);
  // vorticity: omega_r at the edges (f, k) and (f, k + 1), omega_phi at the
  // edges (i, f) and (i + 1, f); C = (curl omega)_theta
  const double R00 = gR(g, s, i, j0, k), R01 = gR(g, s, i, j1, k);
  const double R10 = gR(g, s, i + 1, j0, k), R11 = gR(g, s, i + 1, j1, k);
  const double F00 = gF(g, s, i, j0, k), F01 = gF(g, s, i, j0, k + 1);
  const double F10 = gF(g, s, i, j1, k), F11 = gF(g, s, i, j1, k + 1);
  const double wr0 = ((g.sc[j1] * F10 - g.sc[j0] * F00) * g.idt - (un - zm) * g.idp) * (ir * isF);
  const double wr1 = ((g.sc[j1] * F11 - g.sc[j0] * F01) * g.idt - (zp - un) * g.idp) * (ir * isF);
  const double ira = g.irf[i], irb = g.irf[i + 1];
  const double wp0 = (un - xm) * g.idr + 0.5 * (un + xm) * ira - (R01 - R00) * (ira * g.idt);
  const double wp1 = (xp - un) * g.idr + 0.5 * (xp + un) * irb - (R11 - R10) * (irb * g.idt);
  const double C = (wr1 - wr0) * (ir * isF * g.idp) - (g.rf[i + 1] * wp1 - g.rf[i] * wp0) * (ir * g.idr);
  const double vis = gd - C;
  N += -2.0 * m.omega * g.cf[f] * ub;
  return N - nu * vis - nu * (1.0 / 3.0) * gd;
}

template <class S>
__device__ __forceinline__ double F_uf(const Geo &g, const Mat &m, const S &s, int i, int j, int f) {
  const double ir = g.irc[i], is = g.isc[j], ct = g.ctc[j], ir2 = ir * ir;
  // (a window holds the ghost columns at their own places)
  const bool wrap = !S::WIN && g.periodic;
  const int k0 = wrap ? wrapk(g, f - 1) : f - 1, k1 = wrap ? wrapk(g, f) : f;
  const double irho = irho_mean(g, m, s, i, j, k0, i, j, k1);
  const double nu = m.mu * irho;
  const double un = gF(g, s, i, j, f);
  const double ua = 0.25 * (gR(g, s, i, j, k0) + gR(g, s, i, j, k1) + gR(g, s, i + 1, j, k0) +
                            gR(g, s, i + 1, j, k1));
  const double ub = 0.25 * (gT(g, s, i, j, k0) + gT(g, s, i, j, k1) + gT(g, s, i, j + 1, k0) +
                            gT(g, s, i, j + 1, k1));
  const double xp = gF(g, s, i + 1, j, f), xm = gF(g, s, i - 1, j, f);
  const double yp = gF(g, s, i, j + 1, f), ym = gF(g, s, i, j - 1, f);
  const double zp = gF(g, s, i, j, f + 1), zm = gF(g, s, i, j, f - 1);
  double N = (gC(g, s, F_P, i, j, k1) - gC(g, s, F_P, i, j, k0)) * (irho * ir * is * g.idp);
  N += ua * (xp - xm) * (0.5 * g.idr) + ub * (yp - ym) * (0.5 * ir * g.idt) +
       un * (zp - zm) * (0.5 * ir * is * g.idp) + un * (ua + ub * ct) * ir;
  const double gd = (divc(g, s, i, j, k1) - divc(g, s, i, j, k0)) * (ir * is * g.idp);
  const double R00 = gR(g, s, i, j, k0), R01 = gR(g, s, i, j, k1);
  const double R10 = gR(g, s, i + 1, j, k0), R11 = gR(g, s, i + 1, j, k1);
  const double T00 = gT(g, s, i, j, k0), T01 = gT(g, s, i, j, k1);
  const double T10 = gT(g, s, i, j + 1, k0), T11 = gT(g, s, i, j + 1, k1);
  double vis;
  if (!S::INTERIOR && ((j == 0 && g.pole_lo) || (j == g.nt - 1 && g.pole_hi))) {
    // next to a pole: component form, scalar Laplacians and curvature terms
    vis = (g.rf[i + 1] * g.rf[i + 1] * (xp - un) - g.rf[i] * g.rf[i] * (un - xm)) * (ir2 * g.idr * g.idr) +
          (g.sf[j + 1] * (yp - un) - g.sf[j] * (un - ym)) * (ir2 * is * g.idt * g.idt) +
          (zp - 2.0 * un + zm) * (ir2 * is * is * g.idp * g.idp);
    const double dphr = 0.5 * ((R01 - R00) + (R11 - R10)) * g.idp;
    const double dpht = 0.5 * ((T01 - T00) + (T11 - T10)) * g.idp;
    vis += -un * ir2 * is * is + 2.0 * ir2 * is * dphr + 2.0 * ct * ir2 * is * dpht;
  } else {
    // vorticity: omega_theta at the edges (i, f) and (i + 1, f), omega_r at
    // the edges (j, f) and (j + 1, f); C = (curl omega)_phi
    const double ira = g.irf[i], irb = g.irf[i + 1];
    const double wt0 = (R01 - R00) * (ira * is * g.idp) - (un - xm) * g.idr - 0.5 * (un + xm) * ira;
    const double wt1 = (R11 - R10) * (irb * is * g.idp) - (xp - un) * g.idr - 0.5 * (xp + un) * irb;
    const double wr0 = ((g.scx[j + 1] * un - g.scx[j] * ym) * g.idt - (T01 - T00) * g.idp) * (ir * g.isf[j]);
    const double wr1 = ((g.scx[j + 2] * yp - g.scx[j + 1] * un) * g.idt - (T11 - T10) * g.idp) * (ir * g.isf[j + 1]);
    const double C = (g.rf[i + 1] * wt1 - g.rf[i] * wt0) * (ir * g.idr) - (wr1 - wr0) * (ir * g.idt);
    vis = gd - C;
  }
  N += 2.0 * m.omega * (g.cc[j] * ub + g.sc[j] * ua);
  return N - nu * vis - nu * (1.0 / 3.0) * gd;
}

// F_h at an unknown, less the source term of a forced state (manufactured
// solutions: the residual takes -(F_h - S))
template <class S>
__device__ __forceinline__ double forced(const S &s, int fid, long x, double F) {
  if constexpr (S::WALL) return s.f[fid] ? F - s.f[fid][x] : F;
  else return F;
}

// residual at the centre (i,j,k) and the three faces with the same indices;
// PART 0 .. 3: the centre or the r, theta or phi face alone
template <class S, bool WRITE_UB, int PART = -1>
__device__ __forceinline__ void residual_point(const Geo &g, const Mat &m, const S &s, const Diff &dU,
                                               double tau, const Fields &R, const Fields &Ub,
                                               int *status, int i, int j, int k) {
  if (k >= g.npf) return;
  const bool kc = k < g.np;
  double chk = 0.0; // the sum of this point's residuals: non-finite iff one of them is
  if ((PART < 0 || PART == 0) && i < g.nr && j < g.nt && kc) { // cell centre
    const long x = idx_c(g, i, j, k);
    const double ubp = s.ld(F_P, x), ubT = s.ld(F_T, x);
    if (WRITE_UB) { Ub.p[x] = ubp; Ub.T[x] = ubT; }
    // finite and non-positive; a NaN or an infinity shows as a non-finite
    // residual below
    double pfull = ubp;
    if constexpr (S::PERT) pfull += s.pref[i];
    if (ubT <= 0.0 || pfull + m.pinf <= 0.0) status[ST_NONPHYS] = 1; // plain vector store
    double FT;
    const double Fp = F_p_T(g, m, s, i, j, k, &FT);
    const double rp = -dU.at(F_P, x) - tau * forced(s, F_P, x, Fp);
    const double rT = -dU.at(F_T, x) - tau * forced(s, F_T, x, FT);
    R.p[x] = rp;
    R.T[x] = rT;
    chk = rp + rT;
  }
  if ((PART < 0 || PART == 1) && j < g.nt && kc) { // r face i
    const long x = idx_r(g, i, j, k);
    if (WRITE_UB) Ub.ur[x] = s.ld(F_UR, x);
    const double r = (i >= 1 && i < g.nr) ? -dU.at(F_UR, x) - tau * forced(s, F_UR, x, F_ur(g, m, s, i, j, k)) : 0.0;
    R.ur[x] = r;
    chk += r;
  }
  if ((PART < 0 || PART == 2) && i < g.nr && kc) { // theta face j
    const long x = idx_t(g, i, j, k);
    if (WRITE_UB) Ub.ut[x] = s.ld(F_UT, x);
    const double r = (j >= 1 && j < g.nt) ? -dU.at(F_UT, x) - tau * forced(s, F_UT, x, F_ut(g, m, s, i, j, k)) : 0.0;
    R.ut[x] = r;
    chk += r;
  }
  if ((PART < 0 || PART == 3) && i < g.nr && j < g.nt) { // phi face k
    const long x = idx_f(g, i, j, k);
    if (WRITE_UB) Ub.uf[x] = s.ld(F_UF, x);
    const bool interior = g.periodic || (k >= 1 && k < g.np);
    const double r = interior ? -dU.at(F_UF, x) - tau * forced(s, F_UF, x, F_uf(g, m, s, i, j, k)) : 0.0;
    R.uf[x] = r;
    chk += r;
  }
  if (!isfinite(chk)) status[ST_DIVERGED] = 1; // plain vector store
}

// The interior (1 <= i <= nr-2, 1 <= j <= nt-2, every phi index) is the points
// whose stencils lie inside the arrays in r and theta: its sources apply the
// phi ghost rules without branches, with 32-bit indices.  The shell around it
// takes the ghost rules at every load.  One grid runs both in one launch, a
// batch in two; grids beyond 32-bit indices take the general rules everywhere.
__host__ __device__ inline bool res_interior_ok(const Geo &g) {
  return (long)(g.nr + 1) * (g.nt + 1) * g.npf < 0x7fffffffL;
}
__host__ __device__ inline int res_nk(const Geo &g, int bs) { return (g.npf + bs - 1) / bs; }
__host__ __device__ inline unsigned res_interior_blocks(const Geo &g, int bs) {
  if (!res_interior_ok(g) || g.nr < 3 || g.nt < 3) return 0;
  return (unsigned)res_nk(g, bs) * (unsigned)(g.nt - 2) * (unsigned)(g.nr - 2);
}

// The (i, j) pairs of the shell, or of every point: the shell around the interior, i in {0, nr-1, nr} for every j, then j in
// {0, nt-1, nt} for 1 <= i <= nr-2; else every pair.  Workgroups per pair:
// the phi blocks, res_parts for each.
__host__ __device__ inline unsigned res_shell_pairs(const Geo &g) {
  return 3u * (unsigned)(g.nt + 1) + 3u * (unsigned)(g.nr - 2);
}
__host__ __device__ inline unsigned res_pairs(const Geo &g, bool shell) {
  return shell ? res_shell_pairs(g) : (unsigned)(g.nt + 1) * (unsigned)(g.nr + 1);
}
// Workgroups that share a point of the general launch: one per kind of row
// where that still leaves wave slots free, else one.  The four rows of a point
// one after the other are four memory latencies: 13 us for the shell of
// 32 x 32 x 16 cells against 6.5 split, 135 x 45 x 15 forced 26 against 13,
// 128 x 64 x 32 12.9 against 8.5; but on the 360 x 180 x 40 and 512 x 256 x 128
// spheres (3942 and 9192 workgroups) 25 and 46 us against 31 and 61 split.
__host__ __device__ inline unsigned res_parts(const Geo &g, int bs, bool shell) {
  return (unsigned)res_nk(g, bs) * res_pairs(g, shell) * (unsigned)(bs / 64) <= 2048u ? 4u : 1u;
}
__host__ __device__ inline unsigned res_general_blocks(const Geo &g, int bs, bool shell) {
  return res_parts(g, bs, shell) * (unsigned)res_nk(g, bs) * res_pairs(g, shell);
}

// the pair of workgroup pair number rest of the general launch
__device__ __forceinline__ void res_pair(const Geo &g, unsigned rest, bool shell, int &i, int &j) {
  const unsigned na = 3u * (unsigned)(g.nt + 1);
  if (!shell) {
    j = (int)(rest % (unsigned)(g.nt + 1));
    i = (int)(rest / (unsigned)(g.nt + 1));
  } else if (rest < na) {
    const unsigned ia = rest / (unsigned)(g.nt + 1);
    j = (int)(rest % (unsigned)(g.nt + 1));
    i = ia == 0 ? 0 : (ia == 1 ? g.nr - 1 : g.nr);
  } else {
    const unsigned r2 = rest - na, jb = r2 % 3u;
    i = 1 + (int)(r2 / 3u);
    j = jb == 0 ? 0 : (jb == 1 ? g.nt - 1 : g.nt);
  }
}

// W: a forced pass (wall velocities and source term); PT: the
// perturbation-pressure form
template <bool W = false, bool PT = false>
__device__ __forceinline__ void residual_body(const PassArgs &a, unsigned w4, bool shell) {
  const Geo &g = a.g;
  const int bs = (int)blockDim.x;
  const unsigned nkb = (unsigned)res_nk(g, bs), parts = res_parts(g, bs, shell);
  const unsigned w = parts == 4 ? w4 >> 2 : w4, part = parts == 4 ? w4 & 3u : 4u;
  const unsigned kb = w % nkb, rest = w / nkb;
  int i, j;
  res_pair(g, rest, shell, i, j);
  decltype(auto) s = SrcSel<W, PT>::get(a);
  using S = std::decay_t<decltype(s)>;
  const int k = (int)(kb * blockDim.x + threadIdx.x);
  if (part == 0) residual_point<S, false, 0>(g, a.m, s, a.d, a.tau, a.R, Fields{}, a.status, i, j, k);
  else if (part == 1) residual_point<S, false, 1>(g, a.m, s, a.d, a.tau, a.R, Fields{}, a.status, i, j, k);
  else if (part == 2) residual_point<S, false, 2>(g, a.m, s, a.d, a.tau, a.R, Fields{}, a.status, i, j, k);
  else if (part == 3) residual_point<S, false, 3>(g, a.m, s, a.d, a.tau, a.R, Fields{}, a.status, i, j, k);
  else residual_point<S, false>(g, a.m, s, a.d, a.tau, a.R, Fields{}, a.status, i, j, k);
}

// residual_point for the interior launch (1 <= i <= nr-2, 1 <= j <= nt-2,
// so that every r and theta row exists): every row is evaluated before any
// is stored, and none under a branch except the phi face of a bounded line,
// so that the loads of all four rows can be in flight together (a store of R
// between two rows would hold the next row's loads back until the previous
// row's arithmetic is done, since R may alias the state).  On a bounded phi
// line the lane k = np has no centre: its centre rows are evaluated at
// np - 1 and not stored.  Measured on the 512 x 256 x 128 sphere: 1.40 ->
// 1.00 ms per residual, at 2 waves per SIMD (227 VGPRs) against 4 for the
// row-by-row form; results bitwise unchanged.  Capping the registers for 3
// or 4 waves spills and is slower.
template <class S>
__device__ __forceinline__ void residual_point_in(const Geo &g, const Mat &m, const S &s, const Diff &dU,
                                                  double tau, const Fields &R, int *status, int i, int j,
                                                  int k) {
  if (k >= g.npf) return;
  const bool kc = S::PERIODIC || k < g.np;
  const int kk = S::PERIODIC ? k : min(k, g.np - 1);
  const long xc = idx_c(g, i, j, kk), xr = idx_r(g, i, j, kk), xt = idx_t(g, i, j, kk);
  const double ubp = s.ld(F_P, xc), ubT = s.ld(F_T, xc);
  double pfull = ubp;
  if constexpr (S::PERT) pfull += s.pref[i];
  const bool nonphys = ubT <= 0.0 || pfull + m.pinf <= 0.0;
  double FT;
  const double Fp = F_p_T(g, m, s, i, j, kk, &FT);
  const double rp = -dU.at(F_P, xc) - tau * forced(s, F_P, xc, Fp);
  const double rT = -dU.at(F_T, xc) - tau * forced(s, F_T, xc, FT);
  const double rr = -dU.at(F_UR, xr) - tau * forced(s, F_UR, xr, F_ur(g, m, s, i, j, kk));
  const double rt = -dU.at(F_UT, xt) - tau * forced(s, F_UT, xt, F_ut(g, m, s, i, j, kk));
  const long xf = idx_f(g, i, j, k);
  double rf = 0.0;
  if (S::PERIODIC || (k >= 1 && k < g.np))
    rf = -dU.at(F_UF, xf) - tau * forced(s, F_UF, xf, F_uf(g, m, s, i, j, k));
  if (kc) {
    R.p[xc] = rp;
    R.T[xc] = rT;
    R.ur[xr] = rr;
    R.ut[xt] = rt;
  }
  R.uf[xf] = rf;
  double chk = rf;  // the sum of this point's residuals: non-finite iff one of them is
  if (kc) chk += rp + rT + rr + rt;
  if (kc && nonphys) status[ST_NONPHYS] = 1;  // plain vector store
  if (!isfinite(chk)) status[ST_DIVERGED] = 1;  // plain vector store
}

// the arguments of a pass from its PassArgs at kp
template <class S>
__device__ __forceinline__ void res_source(KPtr kp, S &s) {
#pragma unroll
  for (int f = 0; f < 5; f++) s.a[f] = karr(kp, offsetof(PassArgs, u) + 8 * f);
  if constexpr (S::WALL) {
    s.w = kwall(kp, offsetof(PassArgs, wall));
    const double **const pw[4] = {&s.w.ur_p1, &s.w.ur_p2, &s.w.ut_p1, &s.w.ut_p2};
    const double *const any[2] = {ktab(kp, offsetof(PassArgs, u) + 8 * F_UR), ktab(kp, offsetof(PassArgs, u) + 8 * F_UT)};
#pragma unroll
    for (int q = 0; q < 4; q++) {
      s.has[q] = *pw[q] != nullptr;
      *pw[q] = s.has[q] ? *pw[q] : any[q / 2];
    }
    const Fields q = kfields(kp, offsetof(PassArgs, fsrc));
    s.f[F_P] = q.p; s.f[F_UR] = q.ur; s.f[F_UT] = q.ut; s.f[F_UF] = q.uf; s.f[F_T] = q.T;
  }
  if constexpr (S::PERT) {
    s.pref = ktab(kp, offsetof(PassArgs, pref));
    s.tref = ktab(kp, offsetof(PassArgs, tref));
  }
}
__device__ __forceinline__ Diff res_diff(KPtr kp) {
  Diff d;
#pragma unroll
  for (int f = 0; f < 5; f++) {
    d.k[f] = karr(kp, offsetof(PassArgs, d) + offsetof(Diff, k) + 8 * f);
    d.n[f] = karr(kp, offsetof(PassArgs, d) + offsetof(Diff, n) + 8 * f);
  }
  d.same = karg<int>(kp, offsetof(PassArgs, d) + offsetof(Diff, same));
  return d;
}
__device__ __forceinline__ int *res_status(KPtr kp) {
  return (int *)karg<DSW_AS1 int *>(kp, offsetof(PassArgs, status));
}

template <class SI>
__device__ __forceinline__ void residual_at_in(KPtr kp, unsigned kb, int j, int i) {
  const Geo g = kgeo(kp, offsetof(PassArgs, g));
  SI s;
  res_source(kp, s);
  residual_point_in<SI>(g, kmat(kp, offsetof(PassArgs, m)), s, res_diff(kp), karg<double>(kp, offsetof(PassArgs, tau)),
                        kfields(kp, offsetof(PassArgs, R)), res_status(kp), i, j,
                        (int)(kb * blockDim.x + threadIdx.x));
}

template <bool B>
__global__ void __launch_bounds__(256) DSW_OCC(DSW_WAVES_RES) k_residual(PassArgs a, Batch bt, bool shell) {
  if constexpr (B) {
    const int mb = batch_member(bt, blockIdx.x);
    const PassArgs &am = batch_args(bt, mb);
    residual_body(am, blockIdx.x - bt.woff[mb], res_interior_blocks(am.g, (int)blockDim.x) > 0);
  } else {
    residual_body(a, blockIdx.x, shell);
  }
}

// One row (part 0 .. 3: the centre, the r, theta, phi face) of the shell's
// points k of pair number q.
template <bool W, bool PT>
__device__ __forceinline__ void residual_shell(KPtr kp, unsigned q, int part, int k) {
  using S = std::conditional_t<W, SrcShellW, std::conditional_t<PT, SrcPert<SrcShell>, SrcShell>>;
  const Geo g = kgeo(kp, offsetof(PassArgs, g));
  const Mat m = kmat(kp, offsetof(PassArgs, m));
  S s;
  s.g = g;
  res_source(kp, s);
  const Diff d = res_diff(kp);
  const double tau = karg<double>(kp, offsetof(PassArgs, tau));
  const Fields R = kfields(kp, offsetof(PassArgs, R));
  int *status = res_status(kp);
  int i, j;
  res_pair(g, q, true, i, j);
  if (part == 0) residual_point<S, false, 0>(g, m, s, d, tau, R, Fields{}, status, i, j, k);
  else if (part == 1) residual_point<S, false, 1>(g, m, s, d, tau, R, Fields{}, status, i, j, k);
  else if (part == 2) residual_point<S, false, 2>(g, m, s, d, tau, R, Fields{}, status, i, j, k);
  else residual_point<S, false, 3>(g, m, s, d, tau, R, Fields{}, status, i, j, k);
}

// One grid in one launch (P: periodic): a three-dimensional grid of workgroups
// (phi block, j - 1, i - 1) for the interior, so that their indices need no
// integer division (on this GPU a division of even uniform integers runs on
// the vector unit), and behind its last plane the shell's, one per phi block,
// pair and kind of row.  The two are independent, and on a small grid either
// alone is a chain of latencies in a nearly empty chip: 32 x 32 x 16 cells
// 6.4 and 6.3 us in two launches, 6.6 in one.
template <class SI, bool W, bool PT>
__device__ __forceinline__ void residual_both(KPtr kp) {
  const int nt = karg<int>(kp, offsetof(PassArgs, g) + offsetof(Geo, nt));
  const int nr = karg<int>(kp, offsetof(PassArgs, g) + offsetof(Geo, nr));
  if ((int)blockIdx.z < nr - 2) {
    residual_at_in<SI>(kp, blockIdx.x, 1 + (int)blockIdx.y, 1 + (int)blockIdx.z);
  } else {
    const unsigned w = ((blockIdx.z - (unsigned)(nr - 2)) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const unsigned nkb = gridDim.x, q = w / (4u * nkb), r = w - q * (4u * nkb);
    if (q < 3u * (unsigned)(nt + 1) + 3u * (unsigned)(nr - 2))  // res_shell_pairs
      residual_shell<W, PT>(kp, q, (int)(r & 3u), (int)((r >> 2) * blockDim.x + threadIdx.x));
  }
}
// (the argument is read through the argument block)
template <bool P>
__global__ void __launch_bounds__(256) k_residual_one(PassArgs) {
  residual_both<SrcOneT<true, P>, false, false>((KPtr)__builtin_amdgcn_kernarg_segment_ptr());
}
template <bool P>
__global__ void __launch_bounds__(256) k_residual_one_forced(PassArgs) {
  residual_both<SrcInW<P>, true, false>((KPtr)__builtin_amdgcn_kernarg_segment_ptr());
}
template <bool P>
__global__ void __launch_bounds__(256) k_residual_one_pert(PassArgs) {
  residual_both<SrcPert<SrcOneT<true, P>>, false, true>((KPtr)__builtin_amdgcn_kernarg_segment_ptr());
}
// grids beyond the interior launch's 32-bit indices: every point by the general rules
__global__ void __launch_bounds__(256) k_residual_forced(PassArgs a, bool shell) {
  residual_body<true>(a, blockIdx.x, shell);
}
__global__ void __launch_bounds__(256) k_residual_pert(PassArgs a, bool shell) {
  residual_body<false, true>(a, blockIdx.x, shell);
}

static dim3 one_grid(const Geo &g, unsigned threads) {
  const unsigned nk = (unsigned)res_nk(g, (int)threads), gy = (unsigned)(g.nt - 2);
  const unsigned nsh = 4u * nk * res_shell_pairs(g);
  return dim3(nk, gy, (unsigned)(g.nr - 2) + (nsh + nk * gy - 1) / (nk * gy));
}
// what a launch's y and z dimensions hold; else every point goes by the
// general rules (as on grids beyond the interior's 32-bit indices)
static bool one_fits(const Geo &g, unsigned threads) {
  if (!res_interior_blocks(g, (int)threads)) return false;
  const dim3 d = one_grid(g, threads);
  return d.y <= 65535u && d.z <= 65535u;
}

static void march_one(bool periodic, bool pert, bool forced, const PassArgs &a, hipStream_t st);

void launch_residual_forced(const PassArgs &a, unsigned threads, hipStream_t st) {
  const dim3 bl(threads);
  if (residual_marches(a.g)) march_one(a.g.periodic != 0, false, true, a, st);
  else if (!one_fits(a.g, threads))
    hipLaunchKernelGGL(k_residual_forced, dim3(res_general_blocks(a.g, (int)threads, false)), bl, 0, st, a, false);
  else if (a.g.periodic) hipLaunchKernelGGL(k_residual_one_forced<true>, one_grid(a.g, threads), bl, 0, st, a);
  else hipLaunchKernelGGL(k_residual_one_forced<false>, one_grid(a.g, threads), bl, 0, st, a);
}

void launch_residual_pert(const PassArgs &a, unsigned threads, hipStream_t st) {
  const dim3 bl(threads);
  if (residual_marches(a.g)) march_one(a.g.periodic != 0, true, false, a, st);
  else if (!one_fits(a.g, threads))
    hipLaunchKernelGGL(k_residual_pert, dim3(res_general_blocks(a.g, (int)threads, false)), bl, 0, st, a, false);
  else if (a.g.periodic) hipLaunchKernelGGL(k_residual_one_pert<true>, one_grid(a.g, threads), bl, 0, st, a);
  else hipLaunchKernelGGL(k_residual_one_pert<false>, one_grid(a.g, threads), bl, 0, st, a);
}

// the interior of a batch of grids (P: periodic)
template <bool P>
__global__ void __launch_bounds__(256) k_residual_in(Batch bt) {
  const int mb = batch_member(bt, blockIdx.x);
  KPtr kp = (KPtr)(bt.tab + mb);
  const int nt = karg<int>(kp, offsetof(PassArgs, g) + offsetof(Geo, nt));
  const int npf = karg<int>(kp, offsetof(PassArgs, g) + offsetof(Geo, npf)), bs = (int)blockDim.x;
  // phi block fastest, then j, then i
  const unsigned w = blockIdx.x - bt.woff[mb], nk = (unsigned)((npf + bs - 1) / bs), r = w / nk;
  residual_at_in<SrcOneT<true, P>>(kp, w - r * nk, 1 + (int)(r % (unsigned)(nt - 2)), 1 + (int)(r / (unsigned)(nt - 2)));
}

// The interior of a large grid: a workgroup owns 64 (phi) x 4 (theta) points
// and walks a segment of r planes.  The window of the state that its stencils
// read, three planes of 6 x 66 per field, stands in LDS, ghost columns
// included; the plane after next is loaded to registers before a plane's rows
// are evaluated and written to the fourth slot after them, so its latency
// passes under the arithmetic.  Bound by HBM: 16 to 25 fields' worth of traffic
// (the state, the two iterates of the difference, the result) at 5 TB/s.
constexpr int RM_J = 4, RM_W = 66, RM_FS = (RM_J + 2) * RM_W, RM_PL = 5 * RM_FS;

// the window around (i, j, k): w0, w1, w2 the entries (j - 1, k - 1) of field
// 0 in planes i - 1, i, i + 1
template <bool P>
struct SrcWin {
  const double *w0, *w1, *w2;
  int i, j, k;
  static constexpr bool INTERIOR = true;
  static constexpr bool PERIODIC = P;
  static constexpr bool WALL = false;
  static constexpr bool PERT = false;
  static constexpr bool WIN = true;
  using Row = int;
  __device__ __forceinline__ double at(int f, int i_, int j_, int k_) const {
    const double *w = i_ - i < 0 ? w0 : (i_ - i == 0 ? w1 : w2);
    return w[f * RM_FS + (j_ - j + 1) * RM_W + (k_ - k + 1)];
  }
  __device__ __forceinline__ double ld(int, long) const { return 0.0; }      // never called
  __device__ __forceinline__ double ldk(int, int, int) const { return 0.0; } // never called
};

// kp: the PassArgs of the grid; (bx, by, bz): phi block, theta tile, r segment.
// MID: the state is the midpoint of the difference's two iterates (a.d), formed
// as its planes are loaded and written to a.o.ub as well.  W: a forced pass; the
// ghost columns take the phi walls' velocities, the residual the source.
template <bool P, bool PT, bool MID, bool W = false>
__device__ __forceinline__ void residual_march(KPtr kp, double *lds, int bx, int by, int bz, int seg) {
  using SI = std::conditional_t<PT, SrcPert<SrcWin<P>>, SrcWin<P>>;
  constexpr unsigned GEO = offsetof(PassArgs, g);
  const int tid = threadIdx.y * 64 + threadIdx.x;
  const int k0 = bx * 64, j0 = 1 + by * RM_J;
  const int k = k0 + threadIdx.x, j = __builtin_amdgcn_readfirstlane(j0 + (int)threadIdx.y);
  const int ib = 1 + bz * seg, ie = min(karg<int>(kp, GEO + offsetof(Geo, nr)) - 1, ib + seg);
  // the two window entries this thread stages: byte offsets within a plane of
  // the centres (and r faces), theta faces, phi faces
  unsigned oc[2], ot[2], of[2];
  bool flip[2], hi[2], on;
  unsigned ow[2], owt[2]; // W: index of the entry's row in a plane of the walls' values
  {
    const Geo g = kgeo(kp, GEO);
    on = j < g.nt - 1 && k < g.np;
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int e = min(tid + 256 * q, RM_FS - 1), jj = e / RM_W, kr = k0 - 1 + e - jj * RM_W;
      const int jc = min(j0 - 1 + jj, g.nt - 1), jt = min(j0 - 1 + jj, g.nt);
      const int kc = P ? min(wrapk(g, kr), g.np - 1) : clampi(kr, 0, g.np - 1);
      const int kf = P ? kc : clampi(kr, 0, g.np);
      oc[q] = (unsigned)(jc * g.np + kc) * 8u;
      ot[q] = (unsigned)(jt * g.np + kc) * 8u;
      of[q] = (unsigned)(jc * g.npf + kf) * 8u;
      flip[q] = !P && kc != kr; // no slip at a phi wall
      hi[q] = kr > 0;
      ow[q] = (unsigned)jc * 8u;
      owt[q] = (unsigned)jt * 8u;
    }
  }
  const bool two = tid + 256 < RM_FS;
  double st[2][5], sn[2][5], wr[2], wt[2];
  const auto stage = [&](int p) {
    KPtr q = kp;
    asm volatile("" : "+s"(q), "+s"(p));
    const int nt = karg<int>(q, GEO + offsetof(Geo, nt)), np = karg<int>(q, GEO + offsetof(Geo, np));
    const int npf = karg<int>(q, GEO + offsetof(Geo, npf));
    const long pc = (long)p * nt * np;
    const long pt = (long)p * (nt + 1) * np, pf = (long)p * nt * npf;
#pragma unroll
    for (int f = 0; f < 5; f++) {
      const long x = f == F_UT ? pt : (f == F_UF ? pf : pc);
      const unsigned *o = f == F_UT ? ot : (f == F_UF ? of : oc);
      if constexpr (MID) {
        const double *bk = karr(q, offsetof(PassArgs, d) + offsetof(Diff, k) + 8 * f) + x;
        const double *bn = karr(q, offsetof(PassArgs, d) + offsetof(Diff, n) + 8 * f) + x;
#pragma unroll
        for (int e = 0; e < 2; e++) {
          st[e][f] = ldo(bk, o[e]);
          sn[e][f] = ldo(bn, o[e]);
        }
      } else {
        const double *bu = karr(q, offsetof(PassArgs, u) + 8 * f) + x;
#pragma unroll
        for (int e = 0; e < 2; e++) st[e][f] = ldo(bu, o[e]);
      }
    }
    if constexpr (W && !P) {
      // an absent wall is zero; its pointer stands for an array at least as long
      constexpr unsigned w = offsetof(PassArgs, wall);
      const auto at = [&](unsigned off, int any) {
        const double *x = karr(q, w + off);
        return x ? x : (const double *)karr(q, offsetof(PassArgs, u) + 8 * any);
      };
      const bool has[4] = {karr(q, w + offsetof(Wall, ur_p1)) != nullptr, karr(q, w + offsetof(Wall, ur_p2)) != nullptr,
                           karr(q, w + offsetof(Wall, ut_p1)) != nullptr, karr(q, w + offsetof(Wall, ut_p2)) != nullptr};
      const double *r1 = at(offsetof(Wall, ur_p1), F_UR) + (long)p * nt, *r2 = at(offsetof(Wall, ur_p2), F_UR) + (long)p * nt;
      const double *t1 = at(offsetof(Wall, ut_p1), F_UT) + (long)p * (nt + 1);
      const double *t2 = at(offsetof(Wall, ut_p2), F_UT) + (long)p * (nt + 1);
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const double a1 = ldo(r1, ow[e]), a2 = ldo(r2, ow[e]), b1 = ldo(t1, owt[e]), b2 = ldo(t2, owt[e]);
        wr[e] = hi[e] ? (has[1] ? a2 : 0.0) : (has[0] ? a1 : 0.0);
        wt[e] = hi[e] ? (has[3] ? b2 : 0.0) : (has[2] ? b1 : 0.0);
      }
    }
  };
  const auto commit = [&](int slot) {
#pragma unroll
    for (int q = 0; q < 2; q++) {
      if (q == 1 && !two) continue;
      double *w = lds + slot + tid + 256 * q;
#pragma unroll
      for (int f = 0; f < 5; f++) {
        const double v = MID ? 0.5 * (st[q][f] + sn[q][f]) : st[q][f];
        const double gh = W && !P ? 2.0 * (f == F_UR ? wr[q] : wt[q]) - v : -v;
        w[f * RM_FS] = (f == F_UR || f == F_UT) && flip[q] ? gh : v;
      }
    }
  };
#pragma nounroll
  for (int q = 0; q < 3; q++) {
    stage(ib - 1 + q);
    commit(q * RM_PL);
  }
  __syncthreads();
  int s0 = 0, s1 = RM_PL, s2 = 2 * RM_PL, s3 = 3 * RM_PL;
  const int lane = threadIdx.y * RM_W + threadIdx.x;
  // a lane or wave beyond the grid repeats the last point and stores nothing
  const int jw = min(j, karg<int>(kp, GEO + offsetof(Geo, nt)) - 2);
  const unsigned o = (unsigned)min(k, karg<int>(kp, GEO + offsetof(Geo, np)) - 1) * 8u;
#pragma nounroll
  for (int ii = ib; ii < ie; ii++) {
    KPtr p = kp;
    int i = ii;
    asm volatile("" : "+s"(p), "+s"(i));
    const Geo g = kgeo(p, GEO);
    const long rc = ((long)i * g.nt + jw) * g.np, rt_ = ((long)i * (g.nt + 1) + jw) * g.np;
    const long rf_ = ((long)i * g.nt + jw) * g.npf;
    // loads in the order in which they are waited for: the rows' own
    // differences, then the plane after next
    double dk[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, dn[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (MID || !karg<int>(p, offsetof(PassArgs, d) + offsetof(Diff, same))) {
#pragma unroll
      for (int f = 0; f < 5; f++) {
        const long row = f == F_UT ? rt_ : (f == F_UF ? rf_ : rc);
        dk[f] = ldo(karr(p, offsetof(PassArgs, d) + offsetof(Diff, k) + 8 * f) + row, o);
        dn[f] = ldo(karr(p, offsetof(PassArgs, d) + offsetof(Diff, n) + 8 * f) + row, o);
      }
    }
    stage(min(ii + 2, ie));
    asm volatile("" ::: "memory"); // the loads stay ahead of the arithmetic
    const Mat m = kmat(p, offsetof(PassArgs, m));
    const double tau = karg<double>(p, offsetof(PassArgs, tau));
    SI s;
    s.w0 = lds + s0 + lane;
    s.w1 = lds + s1 + lane;
    s.w2 = lds + s2 + lane;
    s.i = i; s.j = jw; s.k = k;
    if constexpr (PT) {
      s.pref = ktab(p, offsetof(PassArgs, pref));
      s.tref = ktab(p, offsetof(PassArgs, tref));
    }
    double pfull = s.at(F_P, i, jw, k);
    if constexpr (PT) pfull += s.pref[i];
    const bool nonphys = s.at(F_T, i, jw, k) <= 0.0 || pfull + m.pinf <= 0.0;
    double FT;
    double Fp = F_p_T(g, m, s, i, jw, k, &FT);
    double Fr = F_ur(g, m, s, i, jw, k);
    double Ft = F_ut(g, m, s, i, jw, k);
    double Ff = F_uf(g, m, s, i, jw, k);
    if constexpr (W) {
      const Fields q = kfields(p, offsetof(PassArgs, fsrc));
      if (q.p) Fp -= ldo(q.p + rc, o);
      if (q.T) FT -= ldo(q.T + rc, o);
      if (q.ur) Fr -= ldo(q.ur + rc, o);
      if (q.ut) Ft -= ldo(q.ut + rt_, o);
      if (q.uf) Ff -= ldo(q.uf + rf_, o);
    }
    double rp = -(dk[F_P] - dn[F_P]) - tau * Fp;
    double rT = -(dk[F_T] - dn[F_T]) - tau * FT;
    double rr = -(dk[F_UR] - dn[F_UR]) - tau * Fr;
    double rt = -(dk[F_UT] - dn[F_UT]) - tau * Ft;
    double rf = -(dk[F_UF] - dn[F_UF]) - tau * Ff;
    if (!P && k == 0) rf = 0.0;
    const double ubn = MID && !P ? s.at(F_UF, i, jw, k + 1) : 0.0;
    // and the window is written after it, ahead of the stores (whose end the
    // next wait for a load would else wait for)
    asm volatile("" : "+v"(rp), "+v"(rT), "+v"(rr), "+v"(rt), "+v"(rf) : : "memory");
    commit(s3);
    asm volatile("" ::: "memory");
    if (on) {
      const Fields R = kfields(p, offsetof(PassArgs, R));
      sto(R.p + rc, o, rp);
      sto(R.T + rc, o, rT);
      sto(R.ur + rc, o, rr);
      sto(R.ut + rt_, o, rt);
      sto(R.uf + rf_, o, rf);
      if (!P && k == g.np - 1) sto(R.uf + rf_, o + 8u, 0.0);
      if constexpr (MID) {
        const Fields Ub = kfields(p, offsetof(PassArgs, o) + offsetof(Out, ub));
        sto(Ub.p + rc, o, 0.5 * (dk[F_P] + dn[F_P]));
        sto(Ub.T + rc, o, 0.5 * (dk[F_T] + dn[F_T]));
        sto(Ub.ur + rc, o, 0.5 * (dk[F_UR] + dn[F_UR]));
        sto(Ub.ut + rt_, o, 0.5 * (dk[F_UT] + dn[F_UT]));
        sto(Ub.uf + rf_, o, 0.5 * (dk[F_UF] + dn[F_UF]));
        if (!P && k == g.np - 1) sto(Ub.uf + rf_, o + 8u, ubn);
      }
      int *status = (int *)karg<DSW_AS1 int *>(p, offsetof(PassArgs, status));
      if (nonphys) status[ST_NONPHYS] = 1;  // plain vector stores
      // the sum of this point's residuals: non-finite iff one of them is
      if (!isfinite(rf + (rp + rT + rr + rt))) status[ST_DIVERGED] = 1;
    }
    __syncthreads();
    const int t = s0;
    s0 = s1; s1 = s2; s2 = s3; s3 = t;
  }
}

// r planes per segment: a segment loads two planes more than it evaluates, but
// too few leave CUs idle.  Measured with 8, 16, 32 planes: 512 x 256 x 128
// sphere 527, 506, 500 us per residual, 200 x 200 x 100 sector 171, 161, 162;
// with 8, 16 planes 360 x 180 x 40 102, 107; with 2, 4 planes 128 x 64 x 32
// 14.5, 17.5, 150 x 101 x 37 35, 34, 180 x 90 x 24 37, 35.
__host__ __device__ inline unsigned march_tiles(const Geo &g) {
  return (unsigned)((g.np + 63) / 64) * (unsigned)((g.nt - 2 + RM_J - 1) / RM_J);
}
__host__ __device__ inline unsigned march_wgs(const Geo &g, int seg) {
  return march_tiles(g) * (unsigned)((g.nr - 2 + seg - 1) / seg);
}
__host__ __device__ inline int march_seg(const Geo &g) {
  int seg = 16;
  while (seg > 4 && march_wgs(g, seg) < 1024u) seg /= 2;
  return march_wgs(g, seg) < 384u ? 2 : seg;
}

// One grid: the shell's workgroups (64 phi indices of a pair, a wave per kind
// of row) behind the last segment.
template <bool P, bool PT, bool W = false>
__global__ void __launch_bounds__(256) DSW_OCC(2) k_residual_march(PassArgs, int seg, int segs) {
  __shared__ double lds[4 * RM_PL];
  KPtr kp = (KPtr)__builtin_amdgcn_kernarg_segment_ptr();
  if ((int)blockIdx.z < segs) {
    residual_march<P, PT, false, W>(kp, lds, blockIdx.x, blockIdx.y, blockIdx.z, seg);
  } else {
    const unsigned w = ((blockIdx.z - (unsigned)segs) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const int npf = karg<int>(kp, offsetof(PassArgs, g) + offsetof(Geo, npf));
    const unsigned nkb = (unsigned)(npf + 63) / 64u, q = w / nkb;
    const unsigned pairs = 3u * (unsigned)(karg<int>(kp, offsetof(PassArgs, g) + offsetof(Geo, nt)) + 1) +
                           3u * (unsigned)(karg<int>(kp, offsetof(PassArgs, g) + offsetof(Geo, nr)) - 2);
    if (q < pairs)
      residual_shell<W, PT>(kp, q, __builtin_amdgcn_readfirstlane((int)threadIdx.y),
                                (int)((w - q * nkb) * 64u + threadIdx.x));
  }
}
// the public form: the midpoint formed on the way; the shell's points by a
// launch that forms it at every load
template <bool P>
__global__ void __launch_bounds__(256) DSW_OCC(2) k_residual_march_mid(PassArgs, int seg) {
  __shared__ double lds[4 * RM_PL];
  residual_march<P, false, true>((KPtr)__builtin_amdgcn_kernarg_segment_ptr(), lds, blockIdx.x, blockIdx.y, blockIdx.z,
                                 seg);
}
__global__ void __launch_bounds__(64) k_residual_mid_shell(Geo g, Mat m, SrcMid s, Diff dU, double tau, Fields R,
                                                           Fields Ub, int *status) {
  const unsigned nk = (unsigned)(g.npf + 63) / 64u, q = blockIdx.x / nk;
  int i, j;
  res_pair(g, q, true, i, j);
  residual_point<SrcMid, true>(g, m, s, dU, tau, R, Ub, status, i, j, (int)((blockIdx.x - q * nk) * 64u + threadIdx.x));
}
// a batch of grids: workgroups in one dimension, phi block fastest, then theta
template <bool P>
__global__ void __launch_bounds__(256) DSW_OCC(2) k_residual_marchB(Batch bt) {
  __shared__ double lds[4 * RM_PL];
  const int mb = batch_member(bt, blockIdx.x);
  KPtr kp = (KPtr)(bt.tab + mb);
  const Geo g = kgeo(kp, offsetof(PassArgs, g));
  const int w = (int)(blockIdx.x - bt.woff[mb]), nk = (g.np + 63) / 64, nj = (g.nt - 2 + RM_J - 1) / RM_J;
  const int r = w / nk;
  residual_march<P, false, false>(kp, lds, w - r * nk, r % nj, r / nj, march_seg(g));
}

// Workgroups of the shell up to which it joins the interior's launch, where
// its latency is hidden but only two workgroups of it fit a CU: the
// 360 x 180 x 40 sphere (3942) 102 + 25 us in two launches, 113 in one; the
// 512 x 256 x 128 sphere (9192) and the 1024 x 512 x 64 sector (29325) are 1
// and 2 % slower a step in one.
constexpr unsigned RM_SHELL = 4096;
static unsigned march_shell(const Geo &g) {
  const unsigned n = (unsigned)((g.npf + 63) / 64) * res_shell_pairs(g);
  return n <= RM_SHELL ? n : 0u;
}
static dim3 march_grid(const Geo &g, int seg) {
  const unsigned nk = (unsigned)((g.np + 63) / 64), nj = (unsigned)((g.nt - 2 + RM_J - 1) / RM_J);
  const unsigned nsh = march_shell(g);
  return dim3(nk, nj, (unsigned)((g.nr - 2 + seg - 1) / seg) + (nsh + nk * nj - 1) / (nk * nj));
}

// Where it is taken: from 450 workgroups of two planes.  Below that the window
// is a latency more than it saves: one launch with every load up front against
// the window 6.3 against 10.1 us on 32 x 32 x 16 cells (56 workgroups), but
// 17.4 against 14.5 on 128 x 64 x 32 (480), 40 against 34 on 150 x 101 x 37,
// 162 against 102 on 360 x 180 x 40, 262 against 161 on 200 x 200 x 100, 900
// against 506 on 512 x 256 x 128 (the perturbation form of 100 m columns on
// 200 x 200 x 200: 620 against 329; forced steps of two iterations 731 against
// 672 us on 256 x 128 x 32, 2.46 against 2.23 ms on 240 x 256 x 64).
bool residual_marches(const Geo &g) {
  if (!off32_ok(g) || g.nr < 3 || g.nt < 3 || march_wgs(g, 2) < 450u) return false;
  const dim3 d = march_grid(g, march_seg(g));
  return d.y <= 65535u && d.z <= 65535u;
}
unsigned residual_march_blocks(const Geo &g) { return march_wgs(g, march_seg(g)); }

static void march_one(bool periodic, bool pert, bool forced, const PassArgs &a, hipStream_t st) {
  const int seg = march_seg(a.g), segs = (a.g.nr - 2 + seg - 1) / seg;
  const dim3 gr = march_grid(a.g, seg), bl(64, RM_J);
  if (periodic) {
    if (forced) hipLaunchKernelGGL((k_residual_march<true, false, true>), gr, bl, 0, st, a, seg, segs);
    else if (pert) hipLaunchKernelGGL((k_residual_march<true, true>), gr, bl, 0, st, a, seg, segs);
    else hipLaunchKernelGGL((k_residual_march<true, false>), gr, bl, 0, st, a, seg, segs);
  } else {
    if (forced) hipLaunchKernelGGL((k_residual_march<false, false, true>), gr, bl, 0, st, a, seg, segs);
    else if (pert) hipLaunchKernelGGL((k_residual_march<false, true>), gr, bl, 0, st, a, seg, segs);
    else hipLaunchKernelGGL((k_residual_march<false, false>), gr, bl, 0, st, a, seg, segs);
  }
  if (march_shell(a.g)) return;
  const dim3 sb(64), sg(res_general_blocks(a.g, 64, true));
  const Batch none{nullptr, nullptr, 0};
  if (forced) hipLaunchKernelGGL(k_residual_forced, sg, sb, 0, st, a, true);
  else if (pert) hipLaunchKernelGGL(k_residual_pert, sg, sb, 0, st, a, true);
  else hipLaunchKernelGGL(k_residual<false>, sg, sb, 0, st, a, none, true);
}

void launch_residual_march(bool periodic, const PassArgs &a, const Batch &b, unsigned blocks, hipStream_t st) {
  if (!b.tab) march_one(periodic, false, false, a, st);
  else if (periodic) hipLaunchKernelGGL(k_residual_marchB<true>, dim3(blocks), dim3(64, RM_J), 0, st, b);
  else hipLaunchKernelGGL(k_residual_marchB<false>, dim3(blocks), dim3(64, RM_J), 0, st, b);
}

// public form on a small grid: the midpoint formed on the fly from Un and Uk
// and written out, every point in one launch
__global__ void __launch_bounds__(256) k_residual_mid(Geo g, Mat m, SrcMid s, Diff dU, double tau,
                                                      Fields R, Fields Ub, int *status) {
  residual_point<SrcMid, true>(g, m, s, dU, tau, R, Ub, status, blockIdx.z, blockIdx.y,
                               blockIdx.x * blockDim.x + threadIdx.x);
}

// Ub = (Un + Uk) / 2 over the five arrays: two values per thread, one 16-byte
// load from each where the arrays allow it (callers' arrays may start at any
// multiple of 8 bytes)
struct MidArrays {
  const double *n[5], *k[5];
  double *u[5];
  long pairs[6], cnt[5];  // prefix sums of the pairs, array lengths
};
__global__ void __launch_bounds__(256) k_midpoint(MidArrays a) {
  long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= a.pairs[5]) return;
  int f = 0;
  while (t >= a.pairs[f + 1]) f++;
  const long x = 2 * (t - a.pairs[f]);
  const double *n = a.n[f] + x, *k = a.k[f] + x;
  double *u = a.u[f] + x;
  const bool two = x + 1 < a.cnt[f];
  if (two && (((uintptr_t)a.n[f] | (uintptr_t)a.k[f] | (uintptr_t)a.u[f]) & 15u) == 0) {
    const double2 vn = *(const double2 *)n, vk = *(const double2 *)k;
    *(double2 *)u = double2{0.5 * (vk.x + vn.x), 0.5 * (vk.y + vn.y)};
  } else {
    u[0] = 0.5 * (k[0] + n[0]);
    if (two) u[1] = 0.5 * (k[1] + n[1]);
  }
}

unsigned residual_interior_blocks(const Geo &g, int bs) { return res_interior_blocks(g, bs); }
unsigned residual_general_blocks(const Geo &g, int bs) { return res_general_blocks(g, bs, res_interior_blocks(g, bs) > 0); }

static void set5(const double **dst, const Fields &f) {
  dst[F_P] = f.p; dst[F_UR] = f.ur; dst[F_UT] = f.ut; dst[F_UF] = f.uf; dst[F_T] = f.T;
}

// The public residual of a grid whose interior is walked forms the midpoint as
// the planes are loaded: 1024 x 512 x 64 sector 1.79 ms, against 1.97 with a
// pass that writes the midpoint first and 5.83 with it formed at every load.
// Of other grids, those of at least this many interior workgroups of 64 points
// (the largest below the walk, and those beyond its 32-bit offsets) write the
// midpoint first and read it back: 256 x 128 x 64 sector 0.364 -> 0.198 ms; on
// 32 x 32 x 16 the one launch wins (15 against 23 us).  A grid whose interior
// outgrows 32-bit indices has no such workgroups and forms it at every load.
constexpr unsigned RES_MID_SPLIT = 3000;

void launch_residual(const Geo &g, const Mat &m, const Fields &Un, const Fields &Uk, double tau,
                     const Fields &R, const Fields &Ub, const long *cnt, int *status, hipStream_t st) {
  const unsigned th = 64;
  PassArgs a;
  std::memset(&a, 0, sizeof(a));
  a.g = g;
  a.m = m;
  set5(a.u.a, Ub);
  set5(a.d.n, Un);
  set5(a.d.k, Uk);
  a.tau = tau;
  a.R = R;
  a.o.ub = Ub;
  a.status = status;
  SrcMid s;
  set5(s.n, Un);
  set5(s.k, Uk);
  if (residual_marches(g)) {
    const int seg = march_seg(g);
    const dim3 gr((unsigned)((g.np + 63) / 64), (unsigned)((g.nt - 2 + RM_J - 1) / RM_J),
                  (unsigned)((g.nr - 2 + seg - 1) / seg)), bl(64, RM_J);
    if (g.periodic) hipLaunchKernelGGL(k_residual_march_mid<true>, gr, bl, 0, st, a, seg);
    else hipLaunchKernelGGL(k_residual_march_mid<false>, gr, bl, 0, st, a, seg);
    const unsigned nsh = (unsigned)((g.npf + 63) / 64) * res_shell_pairs(g);
    hipLaunchKernelGGL(k_residual_mid_shell, dim3(nsh), dim3(64), 0, st, g, m, s, a.d, tau, R, Ub, status);
    return;
  }
  if (res_interior_blocks(g, (int)th) < RES_MID_SPLIT) {
    const dim3 grid((unsigned)res_nk(g, (int)th), g.nt + 1, g.nr + 1);
    hipLaunchKernelGGL(k_residual_mid, grid, dim3(th), 0, st, g, m, s, a.d, tau, R, Ub, status);
    return;
  }
  MidArrays w;
  set5(w.n, Un);
  set5(w.k, Uk);
  const double *u[5];
  set5(u, Ub);
  w.pairs[0] = 0;
  for (int f = 0; f < 5; f++) {
    w.u[f] = const_cast<double *>(u[f]);
    w.cnt[f] = cnt[f];
    w.pairs[f + 1] = w.pairs[f] + (cnt[f] + 1) / 2;
  }
  hipLaunchKernelGGL(k_midpoint, dim3((unsigned)((w.pairs[5] + 255) / 256)), dim3(256), 0, st, w);
  const Batch none{nullptr, nullptr, 0};
  launch_residual_in_pass(g.periodic != 0, a, none, 0, th, st);
}

void launch_residual_pass(const PassArgs &a, const Batch &b, unsigned blocks, unsigned threads,
                          hipStream_t st) {
  if (b.tab) hipLaunchKernelGGL(k_residual<true>, dim3(blocks), dim3(threads), 0, st, a, b, true);
  else hipLaunchKernelGGL(k_residual<false>, dim3(blocks), dim3(threads), 0, st, a, b, false);
}

// one grid: the shell as well
void launch_residual_in_pass(bool periodic, const PassArgs &a, const Batch &b, unsigned blocks,
                             unsigned threads, hipStream_t st) {
  const dim3 bl(threads);
  if (b.tab) {
    if (periodic) hipLaunchKernelGGL(k_residual_in<true>, dim3(blocks), bl, 0, st, b);
    else hipLaunchKernelGGL(k_residual_in<false>, dim3(blocks), bl, 0, st, b);
  } else if (!one_fits(a.g, threads)) {
    launch_residual_pass(a, b, res_general_blocks(a.g, (int)threads, false), threads, st);
  } else {
    if (periodic) hipLaunchKernelGGL(k_residual_one<true>, one_grid(a.g, threads), bl, 0, st, a);
    else hipLaunchKernelGGL(k_residual_one<false>, one_grid(a.g, threads), bl, 0, st, a);
  }
}

// Courant numbers of a state for the step tau (for a time-step controller):
// at every centre, with the centre-averaged velocity and the spacings
// h_r = dr, h_t = r dtheta, h_f = r sin(theta) dphi, the advective number
// tau (|u_r| / h_r + |u_theta| / h_t + |u_phi| / h_f) and the acoustic one
// tau c max(1/h_r, 1/h_t, 1/h_f), c = sqrt(gamma R T); their maxima over the
// grid.  Non-negative doubles order as their bit patterns, so the maxima are
// unsigned 64-bit atomic maxima (vector atomics) into out[0], out[1].
//
// A wave takes a piece of an (r, theta) row at a time, its lanes the phi cells,
// so that the spacings are formed once per piece and no flat index is taken
// apart; the acoustic number of a lane's cells is that of their largest T, with
// one square root and the spacings' reciprocals at the piece's end; and a
// workgroup issues one pair of atomics.  Bound by the reads of u_r, u_theta,
// u_phi and T.  A flat index per cell taken apart by 64-bit divisions, a square
// root and six divisions per cell and a pair of atomics per wave took 386 us on
// the 200 x 200 x 100 sector, this about 60 us (30 of them the call's launches and
// copy).  Few long rows are cut into pieces of about 256 cells, up to COUR_CUT of
// them: 3 x 3 x 60000 cells as 9 waves 476 us, flat 221, cut 36; but cut into 8192
// pieces, 40 x 40 x 1000 cells take 54 us for their atomics, whole rows 43.
// PACK: rows of up to half a wave, several to a wave, w lanes (a power of two)
// to a row: 64 x 128 rows of 3 cells, a wave each 53 us, flat 38, packed 31; of
// 32 cells 52, 122, 41.
struct CourShape {
  int w, seg, len, items;  // lanes per row; pieces per row, cells per piece; pieces of work of a wave
};
constexpr int COUR_WAVES = 8192;  // 8 workgroups per CU
constexpr int COUR_CUT = 2048;    // pieces that rows are cut into
static CourShape cour_shape(const Geo &g) {
  const int rows = g.nr * g.nt;
  CourShape c{64, 1, g.np, rows};
  if (g.np <= 32) {
    c.w = 4;
    while (c.w < g.np) c.w *= 2;
    c.items = (rows + 64 / c.w - 1) / (64 / c.w);
  } else if (rows <= COUR_CUT / 2) {
    const int seg = std::min((g.np + 255) / 256, COUR_CUT / rows);
    c.len = ((g.np + seg - 1) / seg + 63) / 64 * 64;
    c.seg = (g.np + c.len - 1) / c.len;
    c.items = rows * c.seg;
  }
  return c;
}

template <bool PACK>
__global__ void __launch_bounds__(256) k_courant(Geo g, Mat m, Fields U, double tau, CourShape s,
                                                 unsigned long long *out) {
  __shared__ double red[8];
  const int rows = g.nr * g.nt, np = g.np;
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  double ca = 0.0, cs = 0.0;
  for (int item = (int)blockIdx.x * 4 + wave; item < s.items; item += (int)gridDim.x * 4) {
    int row, k, ke, dk;
    if (PACK) {
      row = item * (64 / s.w) + lane / s.w;
      k = lane & (s.w - 1);
      ke = row < rows ? np : 0;
      dk = s.w;
      row = min(row, rows - 1);
    } else {
      const int it = __builtin_amdgcn_readfirstlane(item);
      row = it / s.seg;
      const int k0 = (it - row * s.seg) * s.len;
      k = k0 + lane;
      ke = min(np, k0 + s.len);
      dk = 64;
    }
    const int i = row / g.nt, j = row - i * g.nt;
    const double hr = g.dr, ht = g.rc[i] * g.dt, hf = g.rc[i] * g.sc[j] * g.dp;
    const double *r0 = U.ur + idx_r(g, i, j, 0), *r1 = U.ur + idx_r(g, i + 1, j, 0);
    const double *t0 = U.ut + idx_t(g, i, j, 0), *t1 = U.ut + idx_t(g, i, j + 1, 0);
    const double *f0 = U.uf + idx_f(g, i, j, 0), *T = U.T + idx_c(g, i, j, 0);
    double a = 0.0, tm = 0.0;
    for (; k < ke; k += dk) {
      const int k1 = g.periodic && k + 1 == np ? 0 : k + 1;
      const double ur = 0.5 * (r0[k] + r1[k]), ut = 0.5 * (t0[k] + t1[k]), uf = 0.5 * (f0[k] + f0[k1]);
      const double v = fabs(ur) / hr + fabs(ut) / ht + fabs(uf) / hf;
      if (v > a) a = v;
      if (T[k] > tm) tm = T[k];
    }
    a *= tau;
    const double ih = fmax(1.0 / hr, fmax(1.0 / ht, 1.0 / hf)), c = tau * sqrt(m.gam * m.Rg * tm) * ih;
    if (a > ca) ca = a;
    if (c > cs) cs = c;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double a = __shfl_xor(ca, o), c = __shfl_xor(cs, o);
    if (a > ca) ca = a;
    if (c > cs) cs = c;
  }
  if (lane == 0) { red[2 * wave] = ca; red[2 * wave + 1] = cs; }
  __syncthreads();
  if (threadIdx.x < 2) {
    double v = red[threadIdx.x];
    for (int w = 1; w < 4; w++) v = red[2 * w + threadIdx.x] > v ? red[2 * w + threadIdx.x] : v;
    atomicMax(&out[threadIdx.x], (unsigned long long)__double_as_longlong(v));
  }
}

__global__ void k_zero_u64(unsigned long long *p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

void launch_courant(const Geo &g, const Mat &m, const Fields &U, double tau, unsigned long long *out,
                    hipStream_t st) {
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, st, out, 2);
  const CourShape s = cour_shape(g);
  const dim3 gr((unsigned)std::min((s.items + 3) / 4, COUR_WAVES / 4)), bl(256);
  if (s.w < 64) hipLaunchKernelGGL(k_courant<true>, gr, bl, 0, st, g, m, U, tau, s, out);
  else hipLaunchKernelGGL(k_courant<false>, gr, bl, 0, st, g, m, U, tau, s, out);
}

} // namespace dsw
