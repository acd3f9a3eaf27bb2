// rt_part.hip -- partitioned line solver for the r and theta sweeps (paper
// eqs. (spl1), (spl2); operators D_r and D_theta of Appendix B, eqs. (dr),
// (dtheta)).
//
// A workgroup takes L neighbouring lines of one family (consecutive phi
// index: the lanes that read one row of their lines read contiguous memory)
// and splits every line into T chunks of PM rows; thread t = c * L + l holds
// chunk c of line l (the first chunk is the short one).  As in the phi solver:
//   1. each thread assembles its rows and eliminates the interior ones with
//      the block Thomas recurrence, carrying the dependence on the last row
//      of the chunk before ("spike"), then sweeps back so that every interior
//      row reads x_q = g_q + V_q x_left + W_q x_sep;
//   2. the chunks' last rows ("separators") of each line form a
//      block-tridiagonal system, solved in LDS by parallel cyclic reduction
//      (log2 T steps);
//   3. the interior rows are filled in from the separators and stored.
// Every intermediate stays in registers and LDS: no scratch array, so the
// pass moves one read of its inputs and one write of its result.
//
// Every input of a chunk is loaded before its first row is eliminated, byte
// offsets are 32-bit from uniform bases (64-bit on grids whose arrays reach 4 GiB,
// BIG: 128 x 4100 x 1024 cells r 30.7 ms, two-ended 39.8), metric factors come
// from per-row tables, and no row stands under a branch.  Assembling a row at a time under
// a branch on the chunk's length spent half of the instructions on addresses,
// ghost cases and register moves, and one memory latency per row.  Line
// solves, a row at a time against this form: 512 x 256 x 128
// sphere r 1.34 -> 0.98, theta 1.80 -> 1.01 ms; 256 x 128 x 64 sector r 0.145
// -> 0.109, theta 0.183 -> 0.130 ms; 32 x 32 x 16 theta 19.6 -> 13.8 us;
// transposed on the sphere r 1.49 -> 1.03 ms, theta (two-ended before) 1.66 ->
// 1.31, on the sector 0.163 -> 0.108 and 0.282 -> 0.151.  The
// block lines stay at two waves per SIMD (256 registers: 63 doubles of
// intermediates and the reduction's 30) and are bound by their FP64 work and
// the reduction's barriers; the scalar lines by their reads.
#include <algorithm>
#include <type_traits>

#include "rows_fast.hpp"

namespace dsw {

constexpr int RT_PMS = 8;  // rows per thread, scalar lines

// chunks of PM rows on a line of n rows
template <int PM>
__host__ __device__ inline int rt_chunks(int n) { return (n + PM - 1) / PM; }

// ------------------------------------------------------------ block lines --
// The block lines [line0, line0 + L) of sweep D with every input of a chunk's
// rows loaded before the first row is eliminated (rows_fast.hpp); mode 0.
// TR: the transposed systems (adjoint), whose rows take blocks of the rows on
// either side, so a chunk loads one more row at each end; W: a forced pass,
// whose ghosts across a wall are 2 g - u (the r lines read none); PT:
// perturbation-pressure form.  Byte offsets in 32 bits (off32_ok), or in
// 64 (BIG).
template <int D, int PM, bool TR, bool W, bool PT, bool BIG>
__device__ __forceinline__ void rt_block_lines(const PassArgs &a, unsigned line0, double *lds) {
  using O = Off<BIG>;
  const Geo &g = a.g;
  const Mat &m = a.m;
  const double hs = a.tau;
  const int n = D == 0 ? g.nr : g.nt, T = (n + PM - 1) / PM, L = (int)blockDim.x / T, pad = T * PM - n;
  const unsigned nb = (unsigned)(D == 0 ? g.nt : g.nr) * (unsigned)g.np;
  const int t = threadIdx.x, c = (int)((unsigned)t / (unsigned)L), l = t - c * L;
  const bool act = c < T && line0 + l < nb;
  const unsigned line = min(line0 + (unsigned)l, nb - 1);
  const int cc = min(c, T - 1), s0 = cc * PM - pad;  // row of q = 0; negative: fillers
  const int pa = (int)(line / (unsigned)g.np), k = (int)line - pa * g.np;
  if (act && c == 0) {
    const bool edge = pa == 0 || pa == (D == 0 ? g.nt : g.nr) - 1 || (!g.periodic && (k == 0 || k == g.np - 1));
    if (edge) zero_bnd<D>(g, a.o.x, pa, k);
    else if (D == 0) a.o.x.ur[idx_r(g, 0, pa, k)] = 0.0;
    else a.o.x.ut[idx_t(g, pa, 0, k)] = 0.0;
  }
  // byte offsets of row 0 and row strides; the phi face after the cell
  const O sC = 8u * (D == 0 ? (O)g.nt * g.np : (O)g.np);
  const O sT = 8u * (D == 0 ? (O)(g.nt + 1) * g.np : (O)g.np);
  const O sF = 8u * (D == 0 ? (O)g.nt * g.npf : (O)g.npf);
  const O oC = 8u * ((D == 0 ? (O)pa * g.np : (O)(pa * g.nt) * g.np) + k);
  const O oT = 8u * ((D == 0 ? (O)pa * g.np : (O)(pa * (g.nt + 1)) * g.np) + k);
  const O oF = 8u * ((D == 0 ? (O)pa * g.npf : (O)(pa * g.nt) * g.npf) + k);
  const int dF = 8 * (g.periodic && k == g.np - 1 ? 1 - g.np : 1);
  const double *u_r = a.u.a[F_UR], *u_t = a.u.a[F_UT], *u_f = a.u.a[F_UF];
  const double *mt = D == 0 ? a.mr : a.mt;
  // per row what its coefficients need, P and T one cell further: held from
  // here to the row's elimination (row q at index q + X)
  constexpr int X = TR ? 1 : 0, NQ = PM + 2 * X;
  double gG[NQ], gGG[NQ], gTR[NQ], P[NQ + 1], Te[NQ + 1], b0[PM], b1[PM], b2[PM];
  double uw[NQ + 1];  // the line's own velocity on the faces around the rows
  // line index of row q, of its faces and of its neighbours; fillers and rows
  // past the ends read the nearest
  auto row = [&](int q) { return (unsigned)(TR ? min(max(s0 + q, 0), n - 1) : max(s0 + q, 0)); };
  auto face = [&](int q) { return (unsigned)(TR ? min(max(s0 + q, 0), n) : max(s0 + q, 0)); };
  {
    const double irk = D == 0 ? 0.0 : g.irc[pa];
    const double ctk = D == 0 ? g.ctc[pa] : 0.0, isk = D == 0 ? g.isc[pa] : 0.0;
    if constexpr (D == 0) {
#pragma unroll
      for (int q = 0; q <= NQ; q++) uw[q] = ldo(u_r, oC + face(q - X) * sC);
    } else {
#pragma unroll
      for (int q = 0; q <= NQ; q++) uw[q] = ldo(u_t, oT + face(q - X) * sT);
    }
    const O up = 8u * (O)g.nt * g.np;  // one r plane of u_r
    double va[NQ + 2];  // D 1: the centre-averaged u_r of the rows and one more at each end
    double tim[NQ + 1], tip[NQ + 1];  // D 1: u_theta on the planes i - 1, i + 1
    if constexpr (D == 1) {
      const double sgl = g.pole_lo ? 1.0 : -1.0, sgh = g.pole_hi ? 1.0 : -1.0;
#pragma unroll
      for (int q = 0; q < NQ + 2; q++) {
        const int s = s0 + q - 1 - X;
        const O o = oC + (unsigned)min(max(s, 0), n - 1) * sC;
        const double v = 0.5 * (ldo(u_r, o) + ldo(u_r, o + up));
        va[q] = s < 0 ? sgl * v : (s >= n ? sgh * v : v);
        if constexpr (W) {
          const double *w = s < 0 ? (g.pole_lo ? nullptr : a.wall.ur_t1) : (s >= n && !g.pole_hi ? a.wall.ur_t2 : nullptr);
          if (w) va[q] += w[(long)pa * g.np + k] + w[(long)(pa + 1) * g.np + k];
        }
      }
      const O pT = 8u * (O)(g.nt + 1) * g.np;
      const bool lo = pa == 0, hi = pa == g.nr - 1;
      const O om = lo ? oT : oT - pT, op = hi ? oT : oT + pT;
#pragma unroll
      for (int q = 0; q <= NQ; q++) {
        const O ro = face(q - X) * sT;
        const double x = ldo(u_t, om + ro), y = ldo(u_t, op + ro);
        tim[q] = lo ? -x : x;
        tip[q] = hi ? -y : y;
        if constexpr (W) {
          const long f = (long)face(q - X) * g.np + k;
          if (lo) tim[q] += 2.0 * wallv(a.wall.ut_r1, f);
          if (hi) tip[q] += 2.0 * wallv(a.wall.ut_r2, f);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NQ; q++) {
      const unsigned s = row(q - X);
      const O o = oC + s * sC, of = oF + s * sF;
      const double f0 = ldo(u_f, of), f1 = ldo(u_f, of + (O)dF);
      P[q] = ldo(a.u.a[F_P], o);
      Te[q] = ldo(a.u.a[F_T], o);
      if (q >= X && q < PM + X) {
        b0[q - X] = ldo(a.rhs.p, o);
        b1[q - X] = ldo(a.rhs.T, o);
        b2[q - X] = D == 0 ? ldo(a.rhs.ur, o + sC) : ldo(a.rhs.ut, oT + s * sT + sT);
      }
      if constexpr (D == 0) {
        const O ot = oT + s * sT;
        const double t0 = ldo(u_t, ot), t1 = ldo(u_t, ot + 8u * (unsigned)g.np), ir = ldo(mt, 64u * s + 40u);
        const double ur = 0.5 * (uw[q] + uw[q + 1]), ut = 0.5 * (t0 + t1);
        const double gg = ((t1 - t0) * g.idt + 2.0 * ur + (f1 - f0) * (isk * g.idp) + ut * ctk) * ir;  // Gtt + Gff
        gG[q] = 0.0;  // from uw
        gTR[q] = gg;  // less G
        gGG[q] = gg * ir;
        if constexpr (PT) P[q] += a.pref[s];
      } else {
        const double ct = ldo(mt, 64u * s + 40u), is = ldo(mt, 64u * s + 48u);
        const double ur = va[q + 1], ut = 0.5 * (uw[q] + uw[q + 1]);
        // u_r differences across the plane: one more load of each face
        const double grr = (ldo(u_r, o + up) - ldo(u_r, o)) * g.idr;
        const double G = ((uw[q + 1] - uw[q]) * g.idt + ur) * irk;
        const double gff = ((f1 - f0) * (is * g.idp) + ur + ut * ct) * irk;
        const double srt = 0.5 * ((tip[q] + tip[q + 1]) - (tim[q] + tim[q + 1])) * (0.5 * g.idr) +
                           (va[q + 2] - va[q]) * (0.5 * irk * g.idt) - ut * irk;
        gG[q] = G;
        gTR[q] = grr + gff;
        gGG[q] = (gff * ct - 0.5 * srt) * irk;
        if constexpr (PT) P[q] += a.pref[pa];
      }
      P[q] += m.pinf;
    }
    {
      const unsigned s = (unsigned)min(s0 + PM + X, n - 1);
      const O o = oC + s * sC;
      P[NQ] = ldo(a.u.a[F_P], o);
      Te[NQ] = ldo(a.u.a[F_T], o);
      if constexpr (PT) P[NQ] += a.pref[D == 0 ? (int)s : pa];
      P[NQ] += m.pinf;
    }
  }
  const double irl = D == 0 ? 1.0 : g.irc[pa];
  const double h = D == 0 ? g.idr : irl * g.idt;
  // row q of the line (TR: -1 .. PM)
  auto assemble = [&](int q, FRow &R) {
    const int s = s0 + q, z = q + X;
    const unsigned o = 64u * row(q);
    RowMetric x;
    const double2 d = ldo2(mt, o), w = ldo2(mt, o + 16);
    x.h = h;
    x.dp = d.x * irl;
    x.dm = d.y * irl;
    x.lp = x.dp * h;
    x.lm = -x.dm * h;
    const double w2 = irl * irl;
    x.wp = w.x * w2;
    x.w0 = w.y * w2;
    x.wm = ldo(mt, o + 32) * w2;
    RowIn in;
    in.vel = 0.5 * (uw[z] + uw[z + 1]);
    in.un = uw[z + 1];
    in.G = D == 0 ? (uw[z + 1] - uw[z]) * g.idr : gG[z];
    in.tr = in.G + gTR[z];
    in.gg = gGG[z];
    in.P = P[z];
    in.T = Te[z];
    in.irho = 2.0 * m.Rg * Te[z] * Te[z + 1] * rcp_nr(P[z] * Te[z + 1] + P[z + 1] * Te[z]);
    const bool own = q >= 0 && q < PM;
    in.b0 = own ? b0[own ? q : 0] : 0.0;
    in.b1 = own ? b1[own ? q : 0] : 0.0;
    in.b2 = own ? b2[own ? q : 0] : 0.0;
    // the end rows of the line: row PM - 1 of the last chunk and the one before
    // it (TR: also as the row before a chunk)
    const bool end = q == PM - 1 && cc == T - 1;
    const bool before = TR ? s == n - 2 : (q == PM - 2 && cc == T - 1);
    frow(m, hs, in, x, s == 0, end, before, TR || s >= 0, R);
  };
  using Row = std::conditional_t<TR, TRow, FRow>;
  FRow M_, R_;  // TR: the rows before and at the one in turn
  if constexpr (TR) {
    assemble(-1, M_);
    assemble(0, R_);
  }
  auto next = [&](int q, Row &R) {
    if constexpr (TR) {
      FRow N_;
      assemble(q + 1, N_);
      trow(M_, R_, N_, s0 + q == 0, q == PM - 1 && cc == T - 1, s0 + q >= 0, R);
      M_ = R_;
      R_ = N_;
    } else {
      assemble(q, R);
    }
  };
  Chunk<PM> ch;
#pragma unroll
  for (int q = 0; q < PM - 1; q++) {
    Row R;
    next(q, R);
    ch.eliminate(q, R);
  }
  Row S;
  next(PM - 1, S);
  ch.back();
  double *rec = lds + (size_t)t * SEP_REC;
  if (c < T) {
#pragma unroll
    for (int z = 0; z < 3; z++) rec[z] = ch.Y[0][z];
#pragma unroll
    for (int z = 0; z < 9; z++) { rec[3 + z] = ch.E[0][z]; rec[12 + z] = ch.C[0][z]; }
  }
  __syncthreads();
  double A[9], B[9], Cc[9], r[3];
  {
    const double *nx = lds + (size_t)(cc < T - 1 ? t + L : min(t, T * L - 1)) * SEP_REC;
    double P[SEP_REC];
#pragma unroll
    for (int z = 0; z < 21; z++) P[z] = nx[z];
    ch.reduce(S, P, P + 3, P + 12, A, B, Cc, r);
  }
  bool sing = ch.sing;
  for (int hh = 1; hh < T; hh *= 2) {
    __syncthreads();
    if (c < T) sing |= sep_publish(A, B, Cc, r, rec);
    __syncthreads();
    const int lo = max(cc - hh, 0) * L + l, hi = min(cc + hh, T - 1) * L + l;
    sep_fold(A, B, Cc, r, lds + (size_t)lo * SEP_REC, lds + (size_t)hi * SEP_REC);
  }
  double Bi[9], xs[3], xl[3];
  sing |= inv3q(B, Bi);
  mv3(Bi, r, xs);
  if (act && sing) a.status[ST_SINGULAR] = 1;
  __syncthreads();
  if (c < T) {
#pragma unroll
    for (int z = 0; z < 3; z++) rec[z] = xs[z];
  }
  __syncthreads();
  if (!act) return;
  {
    const double *pl = lds + (size_t)(c > 0 ? t - L : t) * SEP_REC;
#pragma unroll
    for (int z = 0; z < 3; z++) xl[z] = c > 0 ? pl[z] : 0.0;
  }
#pragma unroll
  for (int q = 0; q < PM; q++) {
    const int s = s0 + q;
    if (s < 0) continue;
    double v[3];
    if (q < PM - 1) ch.fill(q, xl, xs, v);
    else { v[0] = xs[0]; v[1] = xs[1]; v[2] = xs[2]; }
    const O o = oC + (unsigned)s * sC;
    sto(a.o.x.p, o, v[0]);
    sto(a.o.x.T, o, v[1]);
    if (D == 0) sto(a.o.x.ur, o + sC, v[2]);
    else sto(a.o.x.ut, oT + (unsigned)s * sT + sT, v[2]);
  }
}

// ----------------------------------------------------------- scalar lines --
// The lines [line0, line0 + L) of both scalar families in one form: the row
// of a line reads the two cells on either side of its face (their mean
// density) and the sum of the sweep direction's velocity over the same two
// columns on the row's two faces, so the families differ in byte offsets
// only.  Inputs of all rows of a chunk are loaded first, chunks are aligned to
// their ends (fillers: a = -1, b = 1, c = 0, r = 0), as on the block lines.
// TR: the transposed systems, row s (c_{s-1}, b_s, a_{s+1}).  LDS 4 doubles per
// thread; mode 0.
template <int D, int PM, bool TR, bool PT, bool BIG>
__device__ __forceinline__ void rt_scalar_lines(const PassArgs &a, int fam, unsigned line0, double *lds) {
  using O = Off<BIG>;
  const Geo &g = a.g;
  const Mat &m = a.m;
  const double hs = a.tau;
  const int n = D == 0 ? g.nr : g.nt, T = (n + PM - 1) / PM, L = (int)blockDim.x / T, pad = T * PM - n;
  const unsigned nkf = (unsigned)(g.periodic ? g.np : g.np - 1), wid = fam == 0 ? (unsigned)g.np : nkf;
  const unsigned nl = (unsigned)(D == 0 ? g.nt : g.nr) * wid - (fam == 0 ? wid : 0u);
  const int t = threadIdx.x, c = (int)((unsigned)t / (unsigned)L), l = t - c * L;
  const bool act = c < T && line0 + l < nl;
  const unsigned line = min(line0 + (unsigned)l, nl - 1), q0 = line / wid;
  const int cc = min(c, T - 1), s0 = cc * PM - pad;
  const int k = (int)(line - q0 * wid) + (fam == 0 || g.periodic ? 0 : 1), pa = (int)q0 + (fam == 0 ? 1 : 0);
  // cells A and B (before and after the face), velocity columns A and B, output
  const O N = (O)g.np;
  O oA, oB, vA, vB, oX;
  const O sC = 8u * (D == 0 ? (O)g.nt * N : N);
  const O sV = 8u * (D == 0 ? (O)g.nt * N : N);
  O sX;
  double *X;
  const double *Rh;
  if (fam == 0) {
    if (D == 0) {  // u_theta on theta face pa: cells (., pa - 1, k), (., pa, k)
      oB = 8u * ((O)pa * N + k);
      oA = oB - 8u * N;
      vA = oA; vB = oB; oX = oB;
      sX = 8u * (O)(g.nt + 1) * N;
      X = a.o.x.ut; Rh = a.rhs.ut;
    } else {  // u_r on r face pa: cells (pa - 1, ., k), (pa, ., k)
      oB = 8u * ((O)(pa * g.nt) * N + k);
      oA = oB - 8u * (O)g.nt * N;
      vB = 8u * ((O)(pa * (g.nt + 1)) * N + k);
      vA = vB - 8u * (O)(g.nt + 1) * N;
      oX = oB;
      sX = sC;
      X = a.o.x.ur; Rh = a.rhs.ur;
    }
  } else {  // u_phi on phi face k: cells (., k - 1), (., k)
    const int k1 = g.periodic && k == 0 ? g.np - 1 : k - 1;
    const O ro = D == 0 ? (O)pa * N : (O)(pa * g.nt) * N;
    oA = 8u * (ro + k1); oB = 8u * (ro + k);
    const O vo = D == 0 ? ro : (O)(pa * (g.nt + 1)) * N;
    vA = 8u * (vo + k1); vB = 8u * (vo + k);
    oX = 8u * ((D == 0 ? (O)pa * g.npf : (O)(pa * g.nt) * g.npf) + k);
    sX = 8u * (D == 0 ? (O)g.nt * g.npf : (O)g.npf);
    X = a.o.x.uf; Rh = a.rhs.uf;
  }
  const double *V = a.u.a[D == 0 ? F_UR : F_UT], *mt = D == 0 ? a.mr : a.mt;
  const double irr = D == 0 ? 1.0 : (fam == 0 ? g.irf[pa] : g.irc[pa]);
  const double hh = D == 0 ? g.idr : irr * g.idt, hv = 0.125 * hs * hh, hn = hs * m.mu * 2.0 * m.Rg * hh * irr;
  double sglo = -1.0, sghi = -1.0;
  if (D == 1 && fam == 0) { sglo = g.pole_lo ? 1.0 : -1.0; sghi = g.pole_hi ? 1.0 : -1.0; }
  double ra[PM], rb[PM], rc[PM], rr[PM];
  {
    constexpr int X = TR ? 1 : 0, NQ = PM + 2 * X;
    double vs[NQ + 1], ca[NQ], cn[NQ];
#pragma unroll
    for (int q = 0; q <= NQ; q++) {
      const int f = s0 + q - X;
      const O o = (unsigned)(TR ? min(max(f, 0), n) : max(f, 0)) * sV;
      vs[q] = ldo(V, vA + o) + ldo(V, vB + o);
    }
#pragma unroll
    for (int z = 0; z < NQ; z++) {
      const int q = z - X, s = s0 + q;
      const unsigned sc = (unsigned)(TR ? min(max(s, 0), n - 1) : max(s, 0));
      const O o = sc * sC;
      double Pa = ldo(a.u.a[F_P], oA + o), Pb = ldo(a.u.a[F_P], oB + o);
      const double Ta = ldo(a.u.a[F_T], oA + o), Tb = ldo(a.u.a[F_T], oB + o);
      if constexpr (PT) {
        const int ib = D == 0 ? (int)sc : pa;
        Pa += a.pref[D == 1 && fam == 0 ? ib - 1 : ib];
        Pb += a.pref[ib];
      }
      Pa += m.pinf;
      Pb += m.pinf;
      const double2 d = ldo2(mt, 64u * sc);
      const double nu = hn * Ta * Tb * rcp_nr(Pa * Tb + Pb * Ta);  // tau/2 mu / rho times h
      const double ua = hv * (vs[z] + vs[z + 1]), qp = nu * d.x, qm = nu * d.y;
      ca[z] = qm - ua;
      cn[z] = ua - qp;
      if (q < 0 || q >= PM) continue;
      double cb = qp - qm;
      const double r = ldo(Rh, oX + sc * sX);
      if (s == 0) { cb += sglo * ca[z]; if (!TR) ca[z] = 0.0; }
      if (q == PM - 1 && cc == T - 1) { cb += sghi * cn[z]; if (!TR) cn[z] = 0.0; }
      cb += 1.0;
      const bool real = s >= 0;
      rb[q] = real ? cb : 1.0;
      rr[q] = real ? r : 0.0;
    }
#pragma unroll
    for (int q = 0; q < PM; q++) {
      const int s = s0 + q;
      double lo = ca[q + X], up = cn[q + X];
      if constexpr (TR) {  // c_{s-1}, a_{s+1}; none past the ends
        lo = s == 0 ? 0.0 : cn[q];
        up = q == PM - 1 && cc == T - 1 ? 0.0 : ca[q + 2];
      }
      ra[q] = s >= 0 ? lo : -1.0;
      rc[q] = s >= 0 ? up : 0.0;
    }
  }
  // eliminate: x_q = Y_q - C_q x_{q+1} - E_q x_left, then to (g, V, W)
  bool sing = false;
#pragma unroll
  for (int q = 0; q < PM - 1; q++) {
    double dp = rb[q], y = rr[q], lx = ra[q];
    if (q > 0) {
      dp = fma_(-ra[q], rc[q - 1], dp);
      y = fma_(-ra[q], rr[q - 1], y);
      lx = -ra[q] * ra[q - 1];
    }
    sing |= !(dp != 0.0);
    const double id = rcp_nr(dp);
    rc[q] *= id;
    rr[q] = y * id;
    ra[q] = lx * id;
  }
  ra[PM - 2] = -ra[PM - 2];
  rc[PM - 2] = -rc[PM - 2];
#pragma unroll
  for (int q = PM - 3; q >= 0; q--) {
    rr[q] = fma_(-rc[q], rr[q + 1], rr[q]);
    ra[q] = fma_(-rc[q], ra[q + 1], -ra[q]);
    rc[q] = -rc[q] * rc[q + 1];
  }
  // exchange and reduction: quantity q at ex[q * blockDim + t], so that a
  // wave's accesses are contiguous
  const int nth = (int)blockDim.x;
  double *ex = lds + t;
  if (c < T) { ex[0] = rr[0]; ex[nth] = ra[0]; ex[2 * nth] = rc[0]; }
  __syncthreads();
  const double *nx = lds + (cc < T - 1 ? t + L : min(t, T * L - 1));
  double A = ra[PM - 1] * ra[PM - 2];
  double B = fma_(rc[PM - 1], nx[nth], fma_(ra[PM - 1], rc[PM - 2], rb[PM - 1]));
  double C = rc[PM - 1] * nx[2 * nth];
  double r = fma_(-rc[PM - 1], nx[0], fma_(-ra[PM - 1], rr[PM - 2], rr[PM - 1]));
  for (int h = 1; h < T; h *= 2) {
    const double ib = rcp_nr(B);
    sing |= !(B != 0.0);
    __syncthreads();
    if (c < T) { ex[0] = A * ib; ex[nth] = C * ib; ex[2 * nth] = r * ib; }
    __syncthreads();
    const double *lo = lds + max(cc - h, 0) * L + l, *hi = lds + min(cc + h, T - 1) * L + l;
    B = fma_(-C, hi[0], fma_(-A, lo[nth], B));
    r = fma_(-C, hi[2 * nth], fma_(-A, lo[2 * nth], r));
    A = -A * lo[0];
    C = -C * hi[nth];
  }
  sing |= !(B != 0.0);
  const double xs = r * rcp_nr(B);
  if (act && sing) a.status[ST_SINGULAR] = 1;
  __syncthreads();
  if (c < T) ex[0] = xs;
  __syncthreads();
  if (!act) return;
  const double xl = c > 0 ? lds[t - L] : 0.0;
#pragma unroll
  for (int q = 0; q < PM; q++) {
    const int s = s0 + q;
    if (s < 0) continue;
    const double v = q < PM - 1 ? fma_(rc[q], xs, fma_(ra[q], xl, rr[q])) : xs;
    sto(X, oX + (unsigned)s * sX, v);
  }
}

// ------------------------------------------------------------ the passes --

// pm: rows per thread on the block lines
__host__ __device__ inline int rt_block_chunks(int n, int pm) { return (n + pm - 1) / pm; }
__host__ __device__ inline unsigned rt_block_wgs(const Geo &g, int d, unsigned bs, int pm) {
  const Families F = families(g, d);
  const unsigned L = bs / (unsigned)rt_block_chunks(F.n, pm);
  return (unsigned)((F.nb + L - 1) / L);
}

// workgroups of scalar family A, and of both families
__host__ __device__ inline unsigned rt_scalar_wgs_a(const Geo &g, int d, unsigned bs) {
  const Families F = families(g, d);
  const unsigned L = bs / (unsigned)rt_chunks<RT_PMS>(F.n);
  return (unsigned)((F.na + L - 1) / L);
}
__host__ __device__ inline unsigned rt_scalar_wgs(const Geo &g, int d, unsigned bs) {
  const Families F = families(g, d);
  const unsigned L = bs / (unsigned)rt_chunks<RT_PMS>(F.n);
  return rt_scalar_wgs_a(g, d, bs) + (unsigned)((F.nbb + L - 1) / L);
}

// PART 0: block lines only; 1: scalar lines only; 2: block lines in
// workgroups [0, nbw), then the scalar lines.  COMB: workgroups numbered as
// for PART 2 whatever the part (a batched launch's member table counts both
// kinds), those of the other part leaving at once; else PART 1 numbers the
// scalar workgroups from 0.
template <int D, int PM, int PART, bool W = false, bool TR = false, bool PT = false, bool COMB = false, bool BIG = false>
__device__ __forceinline__ void rt_body(const PassArgs &a, unsigned w, double *lds) {
  const Geo &g = a.g;
  const unsigned bs = blockDim.x;
  const unsigned nbw = (PART == 1 && !COMB) ? 0u : rt_block_wgs(g, D, bs, PM);
  if (w < nbw) {
    if constexpr (PART != 1) {
      const unsigned L = bs / (unsigned)rt_chunks<PM>(families(g, D).n);
      rt_block_lines<D, PM, TR, W, PT, BIG>(a, (COMB ? xcd_contiguous(w, nbw) : w) * L, lds);
    }
    return;
  }
  if constexpr (PART != 0) {
    const unsigned w2 = COMB ? xcd_contiguous(w - nbw, rt_scalar_wgs(g, D, bs)) : w - nbw;
    const unsigned L = bs / (unsigned)rt_chunks<RT_PMS>(families(g, D).n);
    const unsigned nwa = rt_scalar_wgs_a(g, D, bs);
    rt_scalar_lines<D, RT_PMS, TR, PT, BIG>(a, w2 < nwa ? 0 : 1, (w2 < nwa ? w2 : w2 - nwa) * L, lds);
  }
}

// Workgroups are numbered XCD-contiguously within a launch, so that the
// neighbouring lines of neighbouring workgroups (which share cache lines and
// neighbour cells) meet in one L2; in a batch within each member's block lines
// and within its scalar lines (over the whole launch the XCDs would get unequal
// shares of the two).
template <int D, int PM, int PART, bool B, bool BIG>
__global__ void __launch_bounds__(PART == 1 ? 512 : 256) DSW_OCC(PART == 1 ? 0 : 2) k_rt_part(PassArgs a, Batch bt) {
  extern __shared__ double lds[];
  if constexpr (B) {
    const int mb = batch_member(bt, blockIdx.x);
    rt_body<D, PM, PART, false, false, false, true, BIG>(batch_args(bt, mb), blockIdx.x - bt.woff[mb], lds);
  } else {
    rt_body<D, PM, PART, false, false, false, false, BIG>(a, xcd_contiguous(blockIdx.x, gridDim.x), lds);
  }
}

// forced theta sweep, one grid: the block lines (PART 0), or with the scalar
// lines (2; those see no wall data, nor do the r lines)
template <int PM, int PART, bool BIG>
__global__ void __launch_bounds__(256) DSW_OCC(2) k_rt_partF(PassArgs a) {
  extern __shared__ double lds[];
  rt_body<1, PM, PART, true, false, false, false, BIG>(a, xcd_contiguous(blockIdx.x, gridDim.x), lds);
}

// perturbation-pressure form, one grid
template <int D, int PM, int PART, bool BIG>
__global__ void __launch_bounds__(PART == 1 ? 512 : 256) DSW_OCC(PART == 1 ? 0 : 2) k_rt_partP(PassArgs a) {
  extern __shared__ double lds[];
  rt_body<D, PM, PART, false, false, true, false, BIG>(a, xcd_contiguous(blockIdx.x, gridDim.x), lds);
}

// transposed systems (adjoint), one grid
template <int D, int PM, int PART, bool BIG>
__global__ void __launch_bounds__(PART == 1 ? 512 : 256) DSW_OCC(PART == 1 ? 0 : 2) k_rt_partT(PassArgs a) {
  extern __shared__ double lds[];
  rt_body<D, PM, PART, false, true, false, false, BIG>(a, xcd_contiguous(blockIdx.x, gridDim.x), lds);
}

// From this many workgroups on, one grid's block and scalar lines run as two
// launches (the scalar lines need a fraction of the block lines' registers
// and run at a higher occupancy on their own).  Measured on the 256 x 128 x 64
// sector (4084 workgroups): r 0.22 -> 0.16 ms, theta 0.28 -> 0.19 ms; the
// same from 256 to 1024.
constexpr unsigned RT_SPLIT_WGS = 1024;

// Lines from which on narrow workgroups (sweep_block below 256) leave long lines
// to the two-ended solver.
constexpr long RT_NARROW_LINES = 30000;

// Threads per workgroup of a launch of scalar lines: lines of more than 16
// chunks (128 rows) take 512 where the blocks take 256, so that a row's loads
// cover 16 neighbouring lines (128 bytes) up to 256 rows.  Measured, theta
// scalar lines with 256, 512: 180 rows 57, 55 us, 200 rows 83, 71, 256 rows 312,
// 279, 512 rows 875, 679.  (The block lines keep 256: at 512 one workgroup fits
// a CU and nothing runs beside its barriers, 256 rows 699, 899 us.)
unsigned rt_scalar_threads(const Geo &g, int d, unsigned bs) {
  return bs == 256u && rt_chunks<RT_PMS>(families(g, d).n) > 16 ? 512u : bs;
}

bool rt_part_supported(const Geo &g, int d, unsigned bs, int pm) {
  const Families F = families(g, d);
  return d < 2 && pm == 4 && bs <= 256 && rt_block_chunks(F.n, pm) <= (int)bs &&
         rt_chunks<RT_PMS>(F.n) <= (int)bs;
}

unsigned rt_part_blocks(const Geo &g, int d, unsigned bs, int pm) {
  return rt_block_wgs(g, d, bs, pm) + rt_scalar_wgs(g, d, bs);
}

size_t rt_part_lds(unsigned bs) { return sizeof(double) * 24 * (size_t)bs; }

template <int D, int PM, bool BIG>
static void launch_rt_d(const PassArgs &a, const Batch &b, unsigned blocks, unsigned threads, hipStream_t st) {
  const size_t lds = rt_part_lds(threads), lds_s = sizeof(double) * 4 * (size_t)threads;
  if (b.tab) {
    // a batch: the members' block and scalar workgroups as two launches over
    // the same table (each leaves the other kind's workgroups at once)
    if (!BIG && blocks < RT_SPLIT_WGS) {
      hipLaunchKernelGGL((k_rt_part<D, PM, 2, true, false>), dim3(blocks), dim3(threads), lds, st, a, b);
    } else {
      hipLaunchKernelGGL((k_rt_part<D, PM, 0, true, BIG>), dim3(blocks), dim3(threads), lds, st, a, b);
      hipLaunchKernelGGL((k_rt_part<D, PM, 1, true, BIG>), dim3(blocks), dim3(threads), lds_s, st, a, b);
    }
    return;
  }
  if (!BIG && blocks < RT_SPLIT_WGS) {
    hipLaunchKernelGGL((k_rt_part<D, PM, 2, false, false>), dim3(blocks), dim3(threads), lds, st, a, b);
    return;
  }
  const unsigned ts = rt_scalar_threads(a.g, D, threads);
  hipLaunchKernelGGL((k_rt_part<D, PM, 0, false, BIG>), dim3(rt_block_wgs(a.g, D, threads, PM)), dim3(threads), lds, st, a, b);
  hipLaunchKernelGGL((k_rt_part<D, PM, 1, false, BIG>), dim3(rt_scalar_wgs(a.g, D, ts)), dim3(ts), rt_scalar_lds(ts), st, a,
                     b);
}

void launch_rt_pass(int d, int pm, const PassArgs &a, const Batch &b, unsigned blocks, unsigned threads,
                    hipStream_t st) {
  (void)pm;  // 4: the only chunk size built (8 measured slower: one wave per SIMD)
  const bool big = b.tab ? b.big : !off32_ok(a.g);
  if (d == 0) {
    if (big) launch_rt_d<0, 4, true>(a, b, blocks, threads, st);
    else launch_rt_d<0, 4, false>(a, b, blocks, threads, st);
  } else {
    if (big) launch_rt_d<1, 4, true>(a, b, blocks, threads, st);
    else launch_rt_d<1, 4, false>(a, b, blocks, threads, st);
  }
}

// The transposed theta block and scalar lines share a launch while all its
// workgroups are resident at once, two of 256 threads per CU (in workgroups of
// 256).  Measured, one launch / two, at 100 phi cells: 468 workgroups (400 x 3)
// 17.5 / 18.7 us, 499 (160 x 16) 21.7 / 23.4, 547 (200 x 9) 29.6 / 23.2, 585
// (500 x 3) 24.8 / 19.9, 800 (256 x 16) 37.4 / 31.1.  (The r lines as the forward
// ones: 12 x 256 x 100 22.9 / 24.6.)
constexpr unsigned RT_T_ONE_WGS = 512;
static unsigned wgs256(unsigned wgs, unsigned bs) { return (unsigned)(((unsigned long)wgs * bs + 255) / 256); }

// Whether transposed theta lines take the two-ended solver where the solver is
// chosen by line length.  Short lines are a short chain for its two threads per
// line, which fill the chip from some 30000 lines on, while the partitioned
// solver's workgroups run in several rounds by then.  Estimates of both times in
// units of 10 ns at 256 threads, from the measured grid of 3 to 40 rows by 8000
// to 130000 lines.  Measured, two-ended / partitioned (us): 3 rows, 25600 lines
// 10.4 / 15.1, 64000 21.5 / 20.4; 5 rows, 40000 19.9 / 26.7, 130000 54.6 / 47.8; 9
// rows, 8000 16.3 / 13.7, 25600 21.0 / 29.0, 64000 46.7 / 45.6; 16 rows, 16000
// 29.6 / 21.7; 17 rows, 32000 40.6 / 46.0, 50000 66.5 / 59.8; 24 rows and more,
// partitioned at every count.  And many lines of more than 128 rows in
// workgroups of 128 threads, which hold two or three of them: 192 rows, 32768
// lines 614 / 702, 256 rows 817 / 868, 200 rows, 25600 lines 565 / 567.  In
// workgroups of 64 threads the two-ended solver is the slower one throughout (6
// rows, 40000 lines 33.9 / 23.8).
bool rt_T_two_ended(const Geo &g, unsigned bs) {
  const long n = g.nt, lines = families(g, 1).nb;
  if (bs < 128u) return false;
  if (n > 128) return bs < 256u && lines >= RT_NARROW_LINES;
  if (n > 24) return false;
  const unsigned nbw = wgs256(rt_block_wgs(g, 1, bs, 4), bs), all = nbw + wgs256(rt_scalar_wgs(g, 1, bs), bs);
  const long two = std::max(1000L, (12 + 7 * n) * std::max(25000L, lines) / 1000);
  long part;
  if (all <= 256u) part = 1150;
  else if (all <= RT_T_ONE_WGS) part = 1750;
  else if (nbw <= 256u) part = 2400;
  else part = 300 + 1100L * ((nbw + 255) / 256) + 200L * rt_block_chunks((int)n, 4);
  return two <= part;
}

template <int D, int PM, bool BIG>
static void launch_rt_T_d(const PassArgs &a, unsigned threads, hipStream_t st) {
  const size_t lds = rt_part_lds(threads);
  const unsigned nbw = rt_block_wgs(a.g, D, threads, PM), nsw = rt_scalar_wgs(a.g, D, threads);
  if (!BIG && (D == 0 ? nbw + nsw < RT_SPLIT_WGS : wgs256(nbw, threads) + wgs256(nsw, threads) <= RT_T_ONE_WGS)) {
    hipLaunchKernelGGL((k_rt_partT<D, PM, 2, false>), dim3(nbw + nsw), dim3(threads), lds, st, a);
    return;
  }
  hipLaunchKernelGGL((k_rt_partT<D, PM, 0, BIG>), dim3(nbw), dim3(threads), lds, st, a);
  const unsigned ts = rt_scalar_threads(a.g, D, threads);
  hipLaunchKernelGGL((k_rt_partT<D, PM, 1, BIG>), dim3(rt_scalar_wgs(a.g, D, ts)), dim3(ts), rt_scalar_lds(ts), st, a);
}

template <int D, int PM, bool BIG>
static void launch_rt_pert_d(const PassArgs &a, unsigned threads, hipStream_t st) {
  const size_t lds = rt_part_lds(threads);
  const unsigned nbw = rt_block_wgs(a.g, D, threads, PM), nsw = rt_scalar_wgs(a.g, D, threads);
  if (!BIG && nbw + nsw < RT_SPLIT_WGS) {
    hipLaunchKernelGGL((k_rt_partP<D, PM, 2, false>), dim3(nbw + nsw), dim3(threads), lds, st, a);
    return;
  }
  hipLaunchKernelGGL((k_rt_partP<D, PM, 0, BIG>), dim3(nbw), dim3(threads), lds, st, a);
  const unsigned ts = rt_scalar_threads(a.g, D, threads);
  hipLaunchKernelGGL((k_rt_partP<D, PM, 1, BIG>), dim3(rt_scalar_wgs(a.g, D, ts)), dim3(ts), rt_scalar_lds(ts), st, a);
}

void launch_rt_pert(int d, const PassArgs &a, unsigned threads, hipStream_t st) {
  const bool big = !off32_ok(a.g);
  if (d == 0) {
    if (big) launch_rt_pert_d<0, 4, true>(a, threads, st);
    else launch_rt_pert_d<0, 4, false>(a, threads, st);
  } else {
    if (big) launch_rt_pert_d<1, 4, true>(a, threads, st);
    else launch_rt_pert_d<1, 4, false>(a, threads, st);
  }
}

void launch_rt_T(int d, const PassArgs &a, unsigned threads, hipStream_t st) {
  const bool big = !off32_ok(a.g);
  if (d == 0) {
    if (big) launch_rt_T_d<0, 4, true>(a, threads, st);
    else launch_rt_T_d<0, 4, false>(a, threads, st);
  } else {
    if (big) launch_rt_T_d<1, 4, true>(a, threads, st);
    else launch_rt_T_d<1, 4, false>(a, threads, st);
  }
}

// Where the scalar lines of a two-ended sweep run apart, by the partitioned
// solver: lines whose chunks are all full and fill the workgroup (n a
// multiple of the rows per thread, a chunk count dividing the workgroup).
// Measured: theta on the 512 x 256 x 128 sphere (256 rows) 1.53 -> 1.43 ms;
// on 64 uneven sectors (lines of 64 to 256 rows) the ragged chunks and idle
// lanes made the two passes slower than the one two-ended launch.
// Not on grids whose byte offsets outgrow 32 bits: 1024 x 1024 x 513 cells, apart
// r 49.1, theta 51.4 ms, in the two-ended launch 42.7 and 47.1.
bool rt_scalar_supported(const Geo &g, int d, unsigned bs) {
  if (d > 1 || bs > 256 || !off32_ok(g)) return false;
  const int n = families(g, d).n, T = rt_chunks<RT_PMS>(n);
  return n % RT_PMS == 0 && T <= (int)bs && bs % (unsigned)T == 0 && rt_scalar_wgs(g, d, bs) > 0;
}

unsigned rt_scalar_blocks(const Geo &g, int d, unsigned bs) { return rt_scalar_wgs(g, d, bs); }

size_t rt_scalar_lds(unsigned bs) { return sizeof(double) * 4 * (size_t)bs; }

// The scalar lines of an r or theta sweep alone (after a two-ended solve of
// its block lines): one grid (workgroups numbered XCD-contiguously) or a
// batch (each member's scalar workgroups from 0).  Without the scalar lines
// the two-ended solve's scratch traffic drops by a sixth: theta on the
// 512 x 256 x 128 sphere 1.53 -> 1.43 ms.
template <int D, bool B>
__global__ void __launch_bounds__(512) k_rt_scal(PassArgs a, Batch bt) {
  extern __shared__ double lds[];
  if constexpr (B) {
    const int mb = batch_member(bt, blockIdx.x);
    const unsigned n = bt.woff[mb + 1] - bt.woff[mb];
    rt_body<D, 4, 1>(batch_args(bt, mb), xcd_contiguous(blockIdx.x - bt.woff[mb], n), lds);
  } else {
    rt_body<D, 4, 1>(a, xcd_contiguous(blockIdx.x, gridDim.x), lds);
  }
}

void launch_rt_scalar_pass(int d, const PassArgs &a, const Batch &b, unsigned blocks, unsigned threads,
                           hipStream_t st) {
  const size_t lds = rt_scalar_lds(threads);
  const dim3 gr(blocks), bl(threads);
  if (b.tab) {
    if (d == 0) hipLaunchKernelGGL((k_rt_scal<0, true>), gr, bl, lds, st, a, b);
    else hipLaunchKernelGGL((k_rt_scal<1, true>), gr, bl, lds, st, a, b);
  } else {
    if (d == 0) hipLaunchKernelGGL((k_rt_scal<0, false>), gr, bl, lds, st, a, b);
    else hipLaunchKernelGGL((k_rt_scal<1, false>), gr, bl, lds, st, a, b);
  }
}

// the solver a grid takes by default: partitioned where a block line
// splits into at most 64 chunks (L >= 4 neighbouring lines per 256-thread
// workgroup), else two-ended.  Measured, partitioned against two-ended, line
// solves: theta on the 512 x 256 x 128 sphere (256 rows) 1.01 / 1.37 ms, theta
// and r on 200 x 200 x 200 cells 0.56 / 0.81 and 0.67 / 0.74 ms, theta on the
// 1024 x 512 x 64 sector (512 rows, 128 chunks) 3.2 / 3.0 ms.
// r lines of more than 128 rows in narrower workgroups, one to three lines each,
// load memory in pieces of as many values: partitioned while there are few
// lines.  Measured, r, 192 rows, two-ended / partitioned: 64 threads, 25600 lines
// 799 / 583 us, 32768 888 / 942, 65536 1703 / 2724, transposed 745 / 627, 853 / 1015,
// 1679 / 3154; 128 threads 520 / 422, 580 / 606, 1166 / 1458, transposed 499 / 455,
// 585 / 657, 1196 / 1563.  (theta, neighbouring rows next to each other: 64
// threads, 65536 lines 1749 / 1502.)
int rt_default_pm(const Geo &g, int d, unsigned bs) {
  const Families F = families(g, d);
  if (d == 0 && bs < 256u && F.n > 128 && F.nb >= RT_NARROW_LINES) return 0;
  return rt_part_supported(g, d, 256, 4) && rt_block_chunks(F.n, 4) <= 64 ? 4 : 0;
}

void launch_rt_forced(int d, int pm, const PassArgs &a, unsigned threads, hipStream_t st) {
  const Batch none{nullptr, nullptr, 0};
  const unsigned nbw = rt_block_wgs(a.g, d, threads, pm), nsw = rt_scalar_wgs(a.g, d, threads);
  if (d == 0) {
    launch_rt_pass(0, pm, a, none, nbw + nsw, threads, st);
  } else if (off32_ok(a.g) && nbw + nsw < RT_SPLIT_WGS) {
    hipLaunchKernelGGL((k_rt_partF<4, 2, false>), dim3(nbw + nsw), dim3(threads), rt_part_lds(threads), st, a);
  } else {
    const unsigned ts = rt_scalar_threads(a.g, 1, threads), nts = rt_scalar_wgs(a.g, 1, ts);
    if (off32_ok(a.g)) {
      hipLaunchKernelGGL((k_rt_partF<4, 0, false>), dim3(nbw), dim3(threads), rt_part_lds(threads), st, a);
      launch_rt_scalar_pass(1, a, none, nts, ts, st);
    } else {
      hipLaunchKernelGGL((k_rt_partF<4, 0, true>), dim3(nbw), dim3(threads), rt_part_lds(threads), st, a);
      hipLaunchKernelGGL((k_rt_part<1, 4, 1, false, true>), dim3(nts), dim3(ts), rt_scalar_lds(ts), st, a, none);
    }
  }
}

} // namespace dsw
