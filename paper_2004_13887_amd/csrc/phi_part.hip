// phi_part.hip -- partitioned line solver for the phi sweep (paper eq. (spl3),
// operator D_phi of Appendix B eq. (dphi)).
//
// A slot (i, j) holds a 3x3-block line in (p, T, u_phi) and two scalar lines,
// u_r on r face i and u_theta on theta face j.  A workgroup takes as many
// neighbouring slots as its lanes hold; a thread owns a chunk of up to 4 rows:
//   1. it assembles its rows (consecutive threads read consecutive phi cells:
//      contiguous loads) and eliminates its interior rows with the block
//      Thomas recurrence, carrying the dependence on the previous chunk's last
//      row ("spike"), then sweeps back so that every interior row reads
//      x_q = g_q + V_q x_left + W_q x_sep;
//   2. the chunks' last rows ("separators") form a block-tridiagonal system
//      (cyclic when phi is periodic) that is solved in LDS by parallel cyclic
//      reduction, log2(#chunks) steps;
//   3. interior rows are filled in from the separators.
// All intermediates stay in registers and LDS: no scratch traffic.
//
// Every input of a chunk is loaded before its first row is eliminated, with
// ghosts by clamped offsets and signs instead of branches (so no slot needs a
// launch or a source of its own); byte offsets take 32 bits, or 64 on grids
// whose arrays reach 4 GiB (BIG: 1024 x 1024 x 513 cells 47 ms, transposed 54, a
// row at a time 68 and 128).  Line solves, one row at a time, a workgroup
// per slot, against this: 512 x 256 x 128 sphere 1.24 -> 0.98 ms, 200 x 200 x
// 200 cells 0.66 -> 0.51, 150 x 101 x 37 84 -> 55 us, 32 x 32 x 16 28 -> 14 us;
// transposed, on the sphere 2.00 -> 0.97 ms, on the 256 x 128 x 64 sector 0.262
// -> 0.144 (2 rows per chunk, the better choice a row at a time, 0.167).  The
// block lines are bound by their FP64 work at two waves per SIMD (a third of it
// the cyclic reduction) and its barriers, the scalar lines by their reads; the
// scalar reductions keep each quantity contiguous over the lanes (a record per
// lane, as the block reductions have, put 16 lanes on one bank: 0.55 against
// 0.45 ms).
#include <algorithm>
#include <type_traits>

#include "rows_fast.hpp"

namespace dsw {

constexpr int PT_MAX = 256;  // chunks per line (lines up to PM * 256 cells)

// Chunks of a line of n rows, at most pm rows each.  A cyclic line takes the
// next power of two (the cyclic reduction closes on itself only then), its
// rows spread over the chunks as evenly as they go (never fewer than one: the
// power of two is at most n); any other line takes full chunks and a last
// one with the rest.  A 360-cell circle is 128 chunks of 2 or 3 rows; solved
// by one thread per line, as every circle without a power-of-two count of
// full chunks once was, the phi pass of a 360 x 180 x 40 sphere took 3.29 ms.
__host__ __device__ inline int phi_chunks(int n, int cyc, int pm) {
  const int full = (n + pm - 1) / pm;
  if (!cyc) return full;
  int T = 1;
  while (T < full) T *= 2;
  return T;
}

// A workgroup takes L = blockDim / T neighbouring slots; thread t = l T + c
// holds chunk c of slot l's lines.  Ghosts across r and theta are a clamped
// index and a sign per lane, across phi the wrap (CYC) or the same.

// the rows of a lane's chunk: row q is cell s0 + q; rows before the chunk's
// first one (real) are fillers
struct PhiChunk {
  int T, L, l, c, s0, pad;  // pad: fillers of this chunk
  bool act;
  unsigned line;
};

template <int PM, bool CYC>
__device__ __forceinline__ PhiChunk phi_lane(const Geo &g, unsigned w) {
  PhiChunk p;
  p.T = phi_chunks(g.np, CYC, PM);
  p.L = (int)blockDim.x / p.T;
  const int t = threadIdx.x;
  p.l = (int)((unsigned)t / (unsigned)p.T);
  p.c = t - p.l * p.T;
  const unsigned n = (unsigned)g.nr * (unsigned)g.nt;
  p.act = p.l < p.L && w * p.L + p.l < n;
  p.line = min(w * (unsigned)p.L + (unsigned)min(p.l, p.L - 1), n - 1);
  if (CYC) {  // rows spread evenly over the chunks
    const int lg = 31 - __builtin_clz((unsigned)p.T), base = g.np >> lg, rem = g.np & (p.T - 1);
    const int len = base + (p.c < rem ? 1 : 0);
    p.pad = PM - len;
    p.s0 = p.c * base + min(p.c, rem) - p.pad;
  } else {  // the first chunk is the short one
    p.s0 = p.c * PM - (p.T * PM - g.np);
    p.pad = max(-p.s0, 0);
  }
  return p;
}

// byte offset of cell (or face) s along phi: wrapped, or the nearest cell
template <bool CYC>
__device__ __forceinline__ unsigned phi_pos(const Geo &g, int s) {
  if (CYC) s = s < 0 ? s + g.np : (s >= g.np ? s - g.np : s);
  else s = min(max(s, 0), g.np - 1);
  return 8u * (unsigned)s;
}

// The block line of every slot of the workgroup.  TR: the transposed systems
// (adjoint), whose rows take blocks of the rows on either side, so a chunk
// loads one more row at each end; W: a forced pass, whose ghosts across a wall
// are 2 g - u (the scalar lines read none); PT: perturbation-pressure form.
// BIG: 64-bit byte offsets.  LDS SEP_REC doubles per thread.
template <int PM, bool CYC, bool TR, bool W, bool PT, bool BIG>
__device__ __forceinline__ void phi_block_fast(const PassArgs &a, unsigned w, double *lds) {
  using O = Off<BIG>;
  const Geo &g = a.g;
  const Mat &m = a.m;
  const double hs = a.tau;
  const PhiChunk pc = phi_lane<PM, CYC>(g, w);
  const int T = pc.T, t = threadIdx.x, c = pc.c, s0 = pc.s0, np = g.np;
  const O N8 = 8u * (O)np, F8 = 8u * (O)g.npf;
  const int i = (int)(pc.line / (unsigned)g.nt), j = (int)pc.line - i * g.nt;
  const double ir = g.irc[i], is = g.isc[j], ct = g.ctc[j], irs = ir * is;
  const double h = irs * g.idp;  // 1 / spacing; dp = h, dm = -h
  // row q at index q + X.  Per row: v = u_r + cot u_theta there and one further
  // at each end, e = Grr + Gtt; per face: own velocity uw, wf the r and theta
  // differences of u_phi
  constexpr int X = TR ? 1 : 0, NQ = PM + 2 * X;
  double v[NQ + 2], e[NQ], uw[NQ + 1], wf[NQ + 1], P[NQ + 1], Te[NQ + 1], b0[PM], b1[PM], b2[PM];
  {
    unsigned pos[NQ + 2];  // cells s0 - 1 - X .. s0 + PM + X
#pragma unroll
    for (int q = 0; q < NQ + 2; q++) pos[q] = phi_pos<CYC>(g, s0 + q - 1 - X);
    unsigned fpos[NQ + 1];  // faces s0 - X .. s0 + PM + X (a bounded line has face np)
#pragma unroll
    for (int q = 0; q <= NQ; q++) fpos[q] = CYC ? pos[q + 1] : 8u * (unsigned)min(max(s0 + q - X, 0), np);
    const double *u_r = a.u.a[F_UR], *u_t = a.u.a[F_UT], *u_f = a.u.a[F_UF];
    const O oC = pc.line * N8, pl = (unsigned)g.nt * N8;
    const O oT = (unsigned)(i * (g.nt + 1) + j) * N8, oF = pc.line * F8, pF = (unsigned)g.nt * F8;
    // u_phi on the four neighbouring lines: a wall or pole negates it
    const double sim = i == 0 ? -1.0 : 1.0, sip = i == g.nr - 1 ? -1.0 : 1.0;
    const double sjm = j == 0 ? -1.0 : 1.0, sjp = j == g.nt - 1 ? -1.0 : 1.0;
    const O oim = i == 0 ? oF : oF - pF, oip = i == g.nr - 1 ? oF : oF + pF;
    const O ojm = j == 0 ? oF : oF - F8, ojp = j == g.nt - 1 ? oF : oF + F8;
    const double kr = 0.5 * g.idr, kt = 0.5 * ir * g.idt * ct;
    const double kip = kr * sip, kim = kr * sim, kjp = kt * sjp, kjm = kt * sjm;
#pragma unroll
    for (int q = 0; q <= NQ; q++) uw[q] = ldo(u_f, oF + fpos[q]);
#pragma unroll
    for (int q = 0; q <= NQ; q++) wf[q] = kip * ldo(u_f, oip + fpos[q]);
#pragma unroll
    for (int q = 0; q <= NQ; q++) wf[q] = fma_(-kim, ldo(u_f, oim + fpos[q]), wf[q]);
#pragma unroll
    for (int q = 0; q <= NQ; q++) wf[q] = fma_(kjp, ldo(u_f, ojp + fpos[q]), wf[q]);
#pragma unroll
    for (int q = 0; q <= NQ; q++) wf[q] = fma_(-kjm, ldo(u_f, ojm + fpos[q]), wf[q]);
    if constexpr (W) {
      const Wall &wl = a.wall;
      const O fj = (unsigned)j * F8, fi = (unsigned)i * F8;
      auto add = [&](const double *w_, O o, double sc) {
        if (!w_) return;
#pragma unroll
        for (int q = 0; q <= NQ; q++) wf[q] = fma_(sc, ldo(w_, o + fpos[q]), wf[q]);
      };
      if (i == 0) add(wl.uf_r1, fj, -2.0 * kr);
      if (i == g.nr - 1) add(wl.uf_r2, fj, 2.0 * kr);
      if (j == 0 && !g.pole_lo) add(wl.uf_t1, fi, -2.0 * kt);
      if (j == g.nt - 1 && !g.pole_hi) add(wl.uf_t2, fi, 2.0 * kt);
    }
#pragma unroll
    for (int q = 0; q < NQ + 2; q++) {
      const int s = s0 + q - 1 - X;
      const double r0 = ldo(u_r, oC + pos[q]), r1 = ldo(u_r, oC + pl + pos[q]);
      const double t0 = ldo(u_t, oT + pos[q]), t1 = ldo(u_t, oT + N8 + pos[q]);
      const double ur = 0.5 * (r0 + r1), ut = 0.5 * (t0 + t1);
      v[q] = fma_(ut, ct, ur);
      if (!CYC && (s < 0 || s >= np)) {  // no slip
        v[q] = -v[q];
        if constexpr (W) {
          const bool lo = s < 0;
          const double *wr = lo ? a.wall.ur_p1 : a.wall.ur_p2, *wt = lo ? a.wall.ut_p1 : a.wall.ut_p2;
          const int wi = i * g.nt + j, wj = i * (g.nt + 1) + j;
          v[q] += wallv(wr, wi) + wallv(wr, wi + g.nt) + ct * (wallv(wt, wj) + wallv(wt, wj + 1));
        }
      }
      if (q >= 1 && q <= NQ) e[q - 1] = (r1 - r0) * g.idr + fma_(t1 - t0, g.idt, ur) * ir;
    }
#pragma unroll
    for (int q = 0; q <= NQ; q++) P[q] = ldo(a.u.a[F_P], oC + pos[q + 1]);
#pragma unroll
    for (int q = 0; q <= NQ; q++) Te[q] = ldo(a.u.a[F_T], oC + pos[q + 1]);
#pragma unroll
    for (int q = 0; q < PM; q++) b0[q] = ldo(a.rhs.p, oC + pos[q + 1 + X]);
#pragma unroll
    for (int q = 0; q < PM; q++) b1[q] = ldo(a.rhs.T, oC + pos[q + 1 + X]);
#pragma unroll
    for (int q = 0; q < PM; q++) b2[q] = ldo(a.rhs.uf, oF + fpos[q + 1 + X]);
    if constexpr (PT) {
      const double pr = a.pref[i];
#pragma unroll
      for (int q = 0; q <= NQ; q++) P[q] += pr;
    }
#pragma unroll
    for (int q = 0; q <= NQ; q++) P[q] += m.pinf;
  }
  RowMetric x;
  x.h = h;
  x.dp = h;
  x.dm = -h;
  x.lp = x.lm = h * h;
  x.wp = x.wm = (-4.0 / 3.0) * (h * h);
  x.w0 = (8.0 / 3.0) * (h * h);
  // row q of the line (TR: -1 .. PM, without the fillers)
  auto assemble = [&](int q, FRow &R) {
    const int z = q + X;
    RowIn in;
    in.vel = 0.5 * (uw[z] + uw[z + 1]);
    in.un = uw[z + 1];
    in.G = fma_(uw[z + 1] - uw[z], h, v[z + 1] * ir);
    in.tr = e[z] + in.G;
    in.gg = (-0.5 * ir) * (0.5 * (wf[z] + wf[z + 1]) + (v[z + 2] - v[z]) * (0.5 * h) - in.vel * (ir * (1.0 + ct * ct)));
    in.P = P[z];
    in.T = Te[z];
    in.irho = 2.0 * m.Rg * Te[z] * Te[z + 1] * rcp_nr(P[z] * Te[z + 1] + P[z + 1] * Te[z]);
    const bool own = q >= 0 && q < PM;
    in.b0 = own ? b0[own ? q : 0] : 0.0;
    in.b1 = own ? b1[own ? q : 0] : 0.0;
    in.b2 = own ? b2[own ? q : 0] : 0.0;
    const bool before = !CYC && (TR ? s0 + q == np - 2 : (q == PM - 2 && c == T - 1));
    frow(m, hs, in, x, !CYC && s0 + q == 0, !CYC && q == PM - 1 && c == T - 1, before, TR || q >= pc.pad, R);
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
      trow(M_, R_, N_, !CYC && s0 + q == 0, !CYC && q == PM - 1 && c == T - 1, q >= pc.pad, R);
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
  // the first row of the chunk, for the chunk before it (a circle's first
  // chunk follows its last one, and uneven chunks start after their fillers)
  double *rec = lds + (size_t)t * SEP_REC;
  if (pc.l < pc.L) {
    double f[21];
#pragma unroll
    for (int z = 0; z < 3; z++) f[z] = ch.Y[0][z];
#pragma unroll
    for (int z = 0; z < 9; z++) { f[3 + z] = ch.E[0][z]; f[12 + z] = ch.C[0][z]; }
    if (CYC && T * PM != np) {
#pragma unroll
      for (int q = 1; q < PM - 1; q++)
        if (pc.pad == q) {
#pragma unroll
          for (int z = 0; z < 3; z++) f[z] = ch.Y[q][z];
#pragma unroll
          for (int z = 0; z < 9; z++) { f[3 + z] = ch.E[q][z]; f[12 + z] = ch.C[q][z]; }
        }
      if (pc.pad == PM - 1) {  // the separator itself
#pragma unroll
        for (int z = 0; z < 21; z++) f[z] = z == 12 || z == 16 || z == 20 ? 1.0 : 0.0;
      }
    }
#pragma unroll
    for (int z = 0; z < 20; z += 2) *(double2 *)(rec + z) = double2{f[z], f[z + 1]};
    rec[20] = f[20];
  }
  __syncthreads();
  const int base = t - c;  // this line's first thread
  double A[9], B[9], Cc[9], r[3];
  {
    const int nx = CYC ? ((c + 1) & (T - 1)) : min(c + 1, T - 1);
    const double *src = lds + (size_t)(pc.l < pc.L ? base + nx : 0) * SEP_REC;
    double f[SEP_REC];
#pragma unroll
    for (int z = 0; z < 20; z += 2) { const double2 y = *(const double2 *)(src + z); f[z] = y.x; f[z + 1] = y.y; }
    f[20] = src[20];
    ch.reduce(S, f, f + 3, f + 12, A, B, Cc, r);
  }
  bool sing = ch.sing;
  for (int hh = 1; hh < T; hh *= 2) {
    __syncthreads();
    if (pc.l < pc.L) sing |= sep_publish(A, B, Cc, r, rec);
    __syncthreads();
    const int lo = CYC ? ((c - hh) & (T - 1)) : max(c - hh, 0), hi = CYC ? ((c + hh) & (T - 1)) : min(c + hh, T - 1);
    const int b = pc.l < pc.L ? base : 0;
    sep_fold(A, B, Cc, r, lds + (size_t)(b + lo) * SEP_REC, lds + (size_t)(b + hi) * SEP_REC);
  }
  double xs[3], xl[3];
  {
    double Si[9];
    if (CYC) {  // the couplings left over point at the separator itself
#pragma unroll
      for (int z = 0; z < 9; z++) B[z] += A[z] + Cc[z];
    }
    sing |= inv3q(B, Si);
    mv3(Si, r, xs);
  }
  if (pc.act && sing) a.status[ST_SINGULAR] = 1;
  __syncthreads();
  if (pc.l < pc.L) {
#pragma unroll
    for (int z = 0; z < 3; z++) rec[z] = xs[z];
  }
  __syncthreads();
  {
    const int lt = c > 0 ? t - 1 : (CYC ? base + T - 1 : t);
    const double *pl = lds + (size_t)(pc.l < pc.L ? lt : 0) * SEP_REC;
#pragma unroll
    for (int z = 0; z < 3; z++) xl[z] = CYC || c > 0 ? pl[z] : 0.0;
  }
  __syncthreads();
  // staged in LDS, stored row by row: whole lines per store instruction
  const int LN = pc.L * np;
  if (pc.act) {
    double *sx = lds + pc.l * np + s0;
#pragma unroll
    for (int q = 0; q < PM; q++) {
      if (q < pc.pad) continue;
      double y[3];
      if (q < PM - 1) ch.fill(q, xl, xs, y);
      else { y[0] = xs[0]; y[1] = xs[1]; y[2] = xs[2]; }
      sx[q] = y[0];
      sx[LN + q] = y[1];
      sx[2 * LN + q] = y[2];
    }
  }
  __syncthreads();
  const unsigned line0 = w * (unsigned)pc.L;
  const int todo = (int)min((unsigned)pc.L, (unsigned)g.nr * (unsigned)g.nt - line0) * np;
  const long c0 = (long)line0 * np, f0 = (long)line0 * g.npf;
  for (int q = t; q < todo; q += blockDim.x) {
    put(a.o, F_P, c0 + q, lds[q]);
    put(a.o, F_T, c0 + q, lds[LN + q]);
    const int lq = pc.L > 1 ? (int)((unsigned)q / (unsigned)np) : 0, k = q - lq * np;
    put(a.o, F_UF, f0 + lq * g.npf + (CYC ? (k + 1 == np ? 0 : k + 1) : k + 1), lds[2 * LN + q]);
  }
}

// Both scalar lines of every slot: u_r on its r face (i >= 1) and u_theta on
// its theta face (j >= 1).  The two lines share the slot's own cell and u_phi
// loads and one set of barriers.  TR: the transposed systems, row s (c_{s-1},
// b_s, a_{s+1}).  LDS 8 doubles per thread.
template <int PM, bool CYC, bool TR, bool PT, bool BIG>
__device__ __forceinline__ void phi_scalar_fast(const PassArgs &a, unsigned w, double *lds) {
  using O = Off<BIG>;
  const Geo &g = a.g;
  const Mat &m = a.m;
  const double hs = a.tau;
  const PhiChunk pc = phi_lane<PM, CYC>(g, w);
  const int T = pc.T, t = threadIdx.x, c = pc.c, s0 = pc.s0, np = g.np;
  const O N8 = 8u * (O)np, F8 = 8u * (O)g.npf;
  const int i = (int)(pc.line / (unsigned)g.nt), j = (int)pc.line - i * g.nt;
  const int im = max(i - 1, 0), jm = max(j - 1, 0);
  double ra[2][PM], rb[2][PM], rc[2][PM], rr[2][PM];
  {
    constexpr int X = TR ? 1 : 0, NQ = PM + 2 * X;
    unsigned pos[NQ], fpos[NQ + 1];
#pragma unroll
    for (int q = 0; q < NQ; q++) pos[q] = phi_pos<CYC>(g, s0 + q - X);
#pragma unroll
    for (int q = 0; q <= NQ; q++)
      fpos[q] = CYC ? phi_pos<true>(g, s0 + q - X) : 8u * (unsigned)min(max(s0 + q - X, 0), np);
    const unsigned l0 = pc.line, li = (unsigned)(im * g.nt + j), lj = (unsigned)(i * g.nt + jm);
    const double *u_f = a.u.a[F_UF], *Pp = a.u.a[F_P], *Tp = a.u.a[F_T];
    double f[3][NQ + 1];
#pragma unroll
    for (int q = 0; q <= NQ; q++) f[0][q] = ldo(u_f, l0 * F8 + fpos[q]);
#pragma unroll
    for (int q = 0; q <= NQ; q++) f[1][q] = ldo(u_f, li * F8 + fpos[q]);
#pragma unroll
    for (int q = 0; q <= NQ; q++) f[2][q] = ldo(u_f, lj * F8 + fpos[q]);
    double P[3][NQ], Te[3][NQ];
#pragma unroll
    for (int z = 0; z < 3; z++) {
      const O o = (z == 0 ? l0 : z == 1 ? li : lj) * N8;
#pragma unroll
      for (int q = 0; q < NQ; q++) P[z][q] = ldo(Pp, o + pos[q]);
#pragma unroll
      for (int q = 0; q < NQ; q++) Te[z][q] = ldo(Tp, o + pos[q]);
    }
    const O oT = (unsigned)(i * (g.nt + 1) + j) * N8;
#pragma unroll
    for (int q = 0; q < PM; q++) rr[0][q] = ldo(a.rhs.ur, l0 * N8 + pos[q + X]);
#pragma unroll
    for (int q = 0; q < PM; q++) rr[1][q] = ldo(a.rhs.ut, oT + pos[q + X]);
    if constexpr (PT) {
      const double p0 = a.pref[i], pm = a.pref[im];
#pragma unroll
      for (int q = 0; q < NQ; q++) { P[0][q] += p0; P[1][q] += pm; P[2][q] += p0; }
    }
#pragma unroll
    for (int z = 0; z < 3; z++)
#pragma unroll
      for (int q = 0; q < NQ; q++) P[z][q] += m.pinf;
#pragma unroll
    for (int z = 0; z < 2; z++) {
      // u_r: 1 / r of its face; u_theta: 1 / sin of its face (0 at a pole,
      // whose line is not solved)
      const double h = (z == 0 ? g.irf[i] * g.isc[j] : g.irc[i] * g.isf[j]) * g.idp;
      const double hv = 0.125 * hs * h, hn = hs * m.mu * 2.0 * m.Rg * (h * h);
      double ca[NQ], cn[NQ];
#pragma unroll
      for (int y = 0; y < NQ; y++) {
        const int q = y - X;
        const double Ta = Te[0][y], Tb = Te[1 + z][y];
        const double nu = hn * Ta * Tb * rcp_nr(P[0][y] * Tb + P[1 + z][y] * Ta);
        const double ua = hv * ((f[0][y] + f[0][y + 1]) + (f[1 + z][y] + f[1 + z][y + 1]));
        ca[y] = -ua - nu;
        cn[y] = ua - nu;
        if (q < 0 || q >= PM) continue;
        double cb = 2.0 * nu;
        if (!CYC && s0 + q == 0) { cb -= ca[y]; if (!TR) ca[y] = 0.0; }
        if (!CYC && q == PM - 1 && c == T - 1) { cb -= cn[y]; if (!TR) cn[y] = 0.0; }
        const bool real = q >= pc.pad;
        rb[z][q] = real ? 1.0 + cb : 1.0;
        rr[z][q] = real ? rr[z][q] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < PM; q++) {
        double lo = ca[q + X], up = cn[q + X];
        if constexpr (TR) {  // c_{s-1}, a_{s+1}; none past the ends of an open line
          lo = !CYC && s0 + q == 0 ? 0.0 : cn[q];
          up = !CYC && q == PM - 1 && c == T - 1 ? 0.0 : ca[q + 2];
        }
        ra[z][q] = q >= pc.pad ? lo : -1.0;
        rc[z][q] = q >= pc.pad ? up : 0.0;
      }
    }
  }
  bool sing[2] = {false, false};
#pragma unroll
  for (int z = 0; z < 2; z++) {
#pragma unroll
    for (int q = 0; q < PM - 1; q++) {
      double dp = rb[z][q], y = rr[z][q], lx = ra[z][q];
      if (q > 0) {
        dp = fma_(-ra[z][q], rc[z][q - 1], dp);
        y = fma_(-ra[z][q], rr[z][q - 1], y);
        lx = -ra[z][q] * ra[z][q - 1];
      }
      sing[z] |= !(dp != 0.0);
      const double id = rcp_nr(dp);
      rc[z][q] *= id;
      rr[z][q] = y * id;
      ra[z][q] = lx * id;
    }
    ra[z][PM - 2] = -ra[z][PM - 2];
    rc[z][PM - 2] = -rc[z][PM - 2];
#pragma unroll
    for (int q = PM - 3; q >= 0; q--) {
      rr[z][q] = fma_(-rc[z][q], rr[z][q + 1], rr[z][q]);
      ra[z][q] = fma_(-rc[z][q], ra[z][q + 1], -ra[z][q]);
      rc[z][q] = -rc[z][q] * rc[z][q + 1];
    }
  }
  // exchange and reduction: quantity q of line z at ex[(4 z + q) * blockDim + t],
  // so that a wave's accesses are contiguous
  const int nth = (int)blockDim.x;
  double *ex = lds + t;
  if (pc.l < pc.L) {
#pragma unroll
    for (int z = 0; z < 2; z++) {
      double gq = rr[z][0], vq = ra[z][0], wq = rc[z][0];
      if (CYC && T * PM != np) {
#pragma unroll
        for (int q = 1; q < PM - 1; q++)
          if (pc.pad == q) { gq = rr[z][q]; vq = ra[z][q]; wq = rc[z][q]; }
        if (pc.pad == PM - 1) { gq = 0.0; vq = 0.0; wq = 1.0; }
      }
      ex[4 * z * nth] = gq; ex[(4 * z + 1) * nth] = vq; ex[(4 * z + 2) * nth] = wq;
    }
  }
  __syncthreads();
  const int base = pc.l < pc.L ? t - c : 0;
  const int nxc = CYC ? ((c + 1) & (T - 1)) : min(c + 1, T - 1);
  double A[2], B[2], C[2], r[2];
#pragma unroll
  for (int z = 0; z < 2; z++) {
    const double *nx = lds + base + nxc + 4 * z * nth;
    const double sa = ra[z][PM - 1], sc = rc[z][PM - 1];
    A[z] = sa * ra[z][PM - 2];
    B[z] = fma_(sc, nx[nth], fma_(sa, rc[z][PM - 2], rb[z][PM - 1]));
    C[z] = sc * nx[2 * nth];
    r[z] = fma_(-sc, nx[0], fma_(-sa, rr[z][PM - 2], rr[z][PM - 1]));
  }
  for (int hh = 1; hh < T; hh *= 2) {
    const int lo = CYC ? ((c - hh) & (T - 1)) : max(c - hh, 0), hi = CYC ? ((c + hh) & (T - 1)) : min(c + hh, T - 1);
    const double *pl = lds + base + lo, *ph = lds + base + hi;
    double ib[2];
#pragma unroll
    for (int z = 0; z < 2; z++) { ib[z] = rcp_nr(B[z]); sing[z] |= !(B[z] != 0.0); }
    __syncthreads();
    if (pc.l < pc.L) {
#pragma unroll
      for (int z = 0; z < 2; z++) {
        ex[4 * z * nth] = A[z] * ib[z];
        ex[(4 * z + 1) * nth] = C[z] * ib[z];
        ex[(4 * z + 2) * nth] = r[z] * ib[z];
      }
    }
    __syncthreads();
#pragma unroll
    for (int z = 0; z < 2; z++) {
      const double *x = pl + 4 * z * nth, *y = ph + 4 * z * nth;
      B[z] = fma_(-C[z], y[0], fma_(-A[z], x[nth], B[z]));
      r[z] = fma_(-C[z], y[2 * nth], fma_(-A[z], x[2 * nth], r[z]));
      A[z] = -A[z] * x[0];
      C[z] = -C[z] * y[nth];
    }
  }
  double xs[2], xl[2];
#pragma unroll
  for (int z = 0; z < 2; z++) {
    const double S = CYC ? A[z] + B[z] + C[z] : B[z];
    sing[z] |= !(S != 0.0);
    xs[z] = r[z] * rcp_nr(S);
  }
  const bool on[2] = {pc.act && i >= 1, pc.act && j >= 1};
  if ((on[0] && sing[0]) || (on[1] && sing[1])) a.status[ST_SINGULAR] = 1;
  __syncthreads();
  if (pc.l < pc.L) { ex[0] = xs[0]; ex[nth] = xs[1]; }
  __syncthreads();
  {
    const int lt = c > 0 ? c - 1 : (CYC ? T - 1 : 0);
#pragma unroll
    for (int z = 0; z < 2; z++) xl[z] = CYC || c > 0 ? lds[base + lt + z * nth] : 0.0;
  }
  __syncthreads();
  const int LN = pc.L * np;
  if (pc.act) {
    double *sx = lds + pc.l * np + s0;
#pragma unroll
    for (int z = 0; z < 2; z++)
#pragma unroll
      for (int q = 0; q < PM; q++)
        if (q >= pc.pad) sx[z * LN + q] = q < PM - 1 ? fma_(rc[z][q], xs[z], fma_(ra[z][q], xl[z], rr[z][q])) : xs[z];
  }
  __syncthreads();
  const unsigned line0 = w * (unsigned)pc.L;
  const int todo = (int)min((unsigned)pc.L, (unsigned)g.nr * (unsigned)g.nt - line0) * np;
  for (int q = t; q < todo; q += blockDim.x) {
    const unsigned lq = pc.L > 1 ? (unsigned)q / (unsigned)np : 0u, ln = line0 + lq, ii = ln / (unsigned)g.nt;
    const int k = q - (int)lq * np;
    if (ii >= 1) put(a.o, F_UR, (long)line0 * np + q, lds[q]);
    if (ln - ii * g.nt >= 1) put(a.o, F_UT, ((long)ln + ii) * np + k, lds[LN + q]);  // i (nt + 1) + j
  }
}

// workgroups of a grid's block lines (and as many of its scalar lines)
__host__ __device__ inline unsigned phi_fast_wgs(const Geo &g, int pm, unsigned bs) {
  const unsigned L = bs / (unsigned)phi_chunks(g.np, g.periodic, pm);
  return ((unsigned)g.nr * (unsigned)g.nt + L - 1) / L;
}

// PART 0: the block lines; 1: the scalar lines; 2: both, the block lines in the
// first half of the workgroups.  COMB: workgroups numbered as for PART 2
// whatever the part (a batched launch's member table counts both halves).
template <int PM, int PART, bool CYC, bool TR, bool W, bool PT, bool COMB, bool BIG>
__device__ __forceinline__ void phi_fast_body(const PassArgs &a, unsigned w, double *lds) {
  const Geo &g = a.g;
  const unsigned nbw = PART == 2 || COMB ? phi_fast_wgs(g, PM, blockDim.x) : 0u;
  const bool block = PART == 0 ? (!COMB || w < nbw) : (PART == 2 && w < nbw);
  if constexpr (PART != 1) {
    if (block) {
      if (a.o.mode == 0) {  // boundary-normal faces of x that no phi line owns
        const PhiChunk pc = phi_lane<PM, CYC>(g, w);
        if (pc.act) {
          const Fields &x = a.o.x;
          const int i = (int)(pc.line / (unsigned)g.nt), j = (int)pc.line - i * g.nt;
          if (i == 0 || j == 0 || i == g.nr - 1 || j == g.nt - 1)
            for (int k = pc.c; k < g.np; k += pc.T) {
              if (i == 0) x.ur[idx_r(g, 0, j, k)] = 0.0;
              if (i == g.nr - 1) x.ur[idx_r(g, g.nr, j, k)] = 0.0;
              if (j == 0) x.ut[idx_t(g, i, 0, k)] = 0.0;
              if (j == g.nt - 1) x.ut[idx_t(g, i, g.nt, k)] = 0.0;
            }
          if (!CYC && pc.c == 0) x.uf[idx_f(g, i, j, 0)] = 0.0;
        }
      }
      phi_block_fast<PM, CYC, TR, W, PT, BIG>(a, w, lds);
      return;
    }
  }
  if constexpr (PART != 0) {
    if (COMB && w < nbw) return;
    phi_scalar_fast<PM, CYC, TR, PT, BIG>(a, PART == 2 || COMB ? w - nbw : w, lds);
  }
}

template <int PM, int PART, bool CYC, bool W, bool PT, bool BIG>
__global__ void __launch_bounds__(256) DSW_OCC(PART == 1 ? 0 : 2) k_phi_fast(PassArgs a) {
  extern __shared__ double lds[];
  phi_fast_body<PM, PART, CYC, false, W, PT, false, BIG>(a, PART == 1 ? xcd_contiguous(blockIdx.x, gridDim.x) : blockIdx.x, lds);
}
// transposed systems (adjoint), one grid
template <int PM, int PART, bool CYC, bool BIG>
__global__ void __launch_bounds__(256) DSW_OCC(PART == 1 ? 0 : 2) k_phi_fastT(PassArgs a) {
  extern __shared__ double lds[];
  phi_fast_body<PM, PART, CYC, true, false, false, false, BIG>(
      a, PART == 1 ? xcd_contiguous(blockIdx.x, gridDim.x) : blockIdx.x, lds);
}
template <int PM, int PART, bool CYC, bool BIG>
__global__ void __launch_bounds__(256) DSW_OCC(PART == 1 ? 0 : 2) k_phi_fastB(PassArgs a, Batch bt) {
  extern __shared__ double lds[];
  const int mb = batch_member(bt, blockIdx.x);
  phi_fast_body<PM, PART, CYC, false, false, false, true, BIG>(batch_args(bt, mb), blockIdx.x - bt.woff[mb], lds);
}

bool phi_part_supported(const Geo &g, int pm) {
  if (pm != 2 && pm != 4) return false;
  return phi_chunks(g.np, g.periodic, pm) <= PT_MAX;
}

bool phi_part_equal(const Geo &g, int pm) {
  if (!phi_part_supported(g, pm)) return false;
  return !g.periodic || g.np == pm * phi_chunks(g.np, 1, pm);
}

// Workgroup width of the fast kernels: the narrowest whose lanes the slots'
// chunks fill to within 5 % of what any width reaches (narrower workgroups
// wait less at their barriers; 34 chunks fill 238 of 256 lanes but 34 of 64).
unsigned phi_fast_threads(const Geo &g, int pm) {
  const unsigned T = (unsigned)phi_chunks(g.np, g.periodic, pm);
  auto use = [&](unsigned bs) { return (double)(bs / T * T) / bs; };
  const double best = std::max(use(64), std::max(use(128), use(256)));
  for (const unsigned bs : {64u, 128u})
    if (use(bs) >= 0.95 * best) return bs;
  return 256;
}

unsigned phi_fast_blocks(const Geo &g, int pm, unsigned threads) { return 2 * phi_fast_wgs(g, pm, threads); }

size_t phi_fast_lds(unsigned threads) { return sizeof(double) * SEP_REC * (size_t)threads; }

// From this many lanes on, the block and the scalar lines run as two launches
// (the scalar lines need half of the block lines' registers and a third of
// their LDS); below it one launch runs both side by side.  Measured, one launch
// against two: 128 x 64 x 32 sphere (2^17 lanes) 17.9 / 22.2 us, 128 x 64 x 64
// sector (2^18) 29.6 / 35.1, 256 x 128 x 32 (2^19) 54.9 / 58.8, 256 x 128 x 64
// (2^20) 101 / 102; transposed 18.2 / 23.0, 38.2 / 41.6, 73.6 / 72.2, 131 / 126.
constexpr unsigned PHI_SPLIT_LANES = 1u << 19;

template <int PM, bool CYC, bool W, bool PT, bool BIG>
static void launch_phi_fast(const PassArgs &a, const Batch &b, unsigned blocks, unsigned threads, size_t lds,
                            hipStream_t st) {
  const size_t lds_s = sizeof(double) * 8 * (size_t)threads;
  const dim3 gr(blocks), half(blocks / 2), bl(threads);
  if (b.tab) {
    if constexpr (!W && !PT) {
      if (!BIG && (unsigned long)blocks * threads < PHI_SPLIT_LANES) {
        hipLaunchKernelGGL((k_phi_fastB<PM, 2, CYC, false>), gr, bl, lds, st, a, b);
      } else {
        hipLaunchKernelGGL((k_phi_fastB<PM, 0, CYC, BIG>), gr, bl, lds, st, a, b);
        hipLaunchKernelGGL((k_phi_fastB<PM, 1, CYC, BIG>), gr, bl, lds_s, st, a, b);
      }
    }
  } else if (!BIG && (unsigned long)blocks * threads < PHI_SPLIT_LANES) {
    hipLaunchKernelGGL((k_phi_fast<PM, 2, CYC, W, PT, false>), gr, bl, lds, st, a);
  } else {
    hipLaunchKernelGGL((k_phi_fast<PM, 0, CYC, W, PT, BIG>), half, bl, lds, st, a);
    hipLaunchKernelGGL((k_phi_fast<PM, 1, CYC, false, PT, BIG>), half, bl, lds_s, st, a);
  }
}

template <int PM, bool CYC, bool W, bool PT>
static void launch_phi_fast_o(const PassArgs &a, const Batch &b, unsigned blocks, unsigned threads, size_t lds,
                              hipStream_t st) {
  if (b.tab ? b.big : !off32_ok(a.g)) launch_phi_fast<PM, CYC, W, PT, true>(a, b, blocks, threads, lds, st);
  else launch_phi_fast<PM, CYC, W, PT, false>(a, b, blocks, threads, lds, st);
}

template <bool W, bool PT>
static void launch_phi_fast_pm(int pm, bool periodic, const PassArgs &a, const Batch &b, unsigned blocks,
                               unsigned threads, size_t lds, hipStream_t st) {
  if (pm == 2) {
    if (periodic) launch_phi_fast_o<2, true, W, PT>(a, b, blocks, threads, lds, st);
    else launch_phi_fast_o<2, false, W, PT>(a, b, blocks, threads, lds, st);
  } else {
    if (periodic) launch_phi_fast_o<4, true, W, PT>(a, b, blocks, threads, lds, st);
    else launch_phi_fast_o<4, false, W, PT>(a, b, blocks, threads, lds, st);
  }
}

void launch_phi_pass_c(int pm, bool periodic, const PassArgs &a, const Batch &b, unsigned blocks,
                       unsigned threads, size_t lds, hipStream_t st) {
  launch_phi_fast_pm<false, false>(pm, periodic, a, b, blocks, threads, lds, st);
}

void launch_phi_pert_c(int pm, bool periodic, const PassArgs &a, unsigned blocks, unsigned threads, size_t lds,
                       hipStream_t st) {
  launch_phi_fast_pm<false, true>(pm, periodic, a, Batch{nullptr, nullptr, 0}, blocks, threads, lds, st);
}

// transposed: as the plain pass
template <int PM, bool CYC, bool BIG>
static void launch_phi_fast_T(const PassArgs &a, unsigned blocks, unsigned threads, hipStream_t st) {
  const size_t lds = phi_fast_lds(threads), lds_s = sizeof(double) * 8 * (size_t)threads;
  if (!BIG && (unsigned long)blocks * threads < PHI_SPLIT_LANES) {
    hipLaunchKernelGGL((k_phi_fastT<PM, 2, CYC, false>), dim3(blocks), dim3(threads), lds, st, a);
    return;
  }
  hipLaunchKernelGGL((k_phi_fastT<PM, 0, CYC, BIG>), dim3(blocks / 2), dim3(threads), lds, st, a);
  hipLaunchKernelGGL((k_phi_fastT<PM, 1, CYC, BIG>), dim3(blocks / 2), dim3(threads), lds_s, st, a);
}

template <int PM>
static void launch_phi_T_pm(const PassArgs &a, hipStream_t st) {
  const unsigned th = phi_fast_threads(a.g, PM), nb = phi_fast_blocks(a.g, PM, th);
  const bool big = !off32_ok(a.g);
  if (a.g.periodic) {
    if (big) launch_phi_fast_T<PM, true, true>(a, nb, th, st);
    else launch_phi_fast_T<PM, true, false>(a, nb, th, st);
  } else {
    if (big) launch_phi_fast_T<PM, false, true>(a, nb, th, st);
    else launch_phi_fast_T<PM, false, false>(a, nb, th, st);
  }
}
void launch_phi_T_c(int pm, const PassArgs &a, hipStream_t st) {
  if (pm == 2) launch_phi_T_pm<2>(a, st);
  else launch_phi_T_pm<4>(a, st);
}

// forced: as the plain pass
void launch_phi_forced(int pm, const PassArgs &a, hipStream_t st) {
  const Geo &g = a.g;
  const unsigned th = phi_fast_threads(g, pm);
  launch_phi_fast_pm<true, false>(pm, g.periodic != 0, a, Batch{nullptr, nullptr, 0}, phi_fast_blocks(g, pm, th), th,
                                  phi_fast_lds(th), st);
}

} // namespace dsw
