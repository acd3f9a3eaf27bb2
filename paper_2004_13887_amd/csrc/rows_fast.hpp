// rows_fast.hpp -- rows and eliminations of the partitioned block-line solvers
// (rt_part.hip, phi_part.hip) in the form their chunks take: the inputs of all
// rows of a chunk are loaded before any row is eliminated and reduced at once
// to the few values a row's coefficients need, and the products run over the
// structural non-zeros only.
//
// A chunk always has PM rows, aligned to its end: row PM - 1 is the separator.
// Where a chunk holds fewer rows of the line, its first rows are fillers, x_q =
// x_{q-1} (L = -I, D = I, U = 0, b = 0), which pass the dependence on the
// separator before the chunk through unchanged.  So no row and no store of
// intermediates stands under a branch, and the last row of the line is a
// separator whatever its length.
#pragma once

#include <type_traits>

#include "rows.hpp"

namespace dsw {

// a load at a byte offset from a uniform base: base in scalar registers, one
// 32-bit offset register for any number of arrays of the same layout (O:
// unsigned), or a 64-bit offset on grids whose arrays reach 4 GiB (size_t)
template <class O>
__device__ __forceinline__ double ldo(const double *base, O off) {
  return *(const double *)((const char *)base + off);
}
__device__ __forceinline__ double2 ldo2(const double *base, unsigned off) {
  return *(const double2 *)((const char *)base + off);
}
template <class O>
__device__ __forceinline__ void sto(double *base, O off, double v) {
  *(double *)((char *)base + off) = v;
}
template <bool BIG>
using Off = std::conditional_t<BIG, size_t, unsigned>;

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The state with the ghost rules of dsw_common.hpp for the rows of the boundary
// shell at uniform (i, j), by selects on clamped indices: no load under a condition that differs between lanes.
// (With early returns in divergent branches the compiler, clang 22 of ROCm 7.2,
// left a uniform row index undefined in waves where no lane took the branch.)
struct SrcShell {
  const double *a[5];
  Geo g;  // for at() alone
  static constexpr bool INTERIOR = false;
  static constexpr bool PERIODIC = false;
  static constexpr bool WALL = false;
  static constexpr bool PERT = false;
  static constexpr bool WIN = true;
  __device__ __forceinline__ double ld(int f, long x) const { return a[f][x]; }
  __device__ __forceinline__ double at(int f, int i, int j, int k) const;
};
__device__ __forceinline__ int phi_in(const Geo &g, int k) { return g.periodic ? wrapk(g, k) : clampi(k, 0, g.np - 1); }
__device__ __forceinline__ double gC(const Geo &g, const SrcShell &s, int fid, int i, int j, int k) {
  const long row = ((long)clampi(i, 0, g.nr - 1) * g.nt + clampi(j, 0, g.nt - 1)) * g.np;
  return ldo(s.a[fid] + row, (unsigned)phi_in(g, k) * 8u);
}
__device__ __forceinline__ double gR(const Geo &g, const SrcShell &s, int f, int j, int k) {
  const int kk = phi_in(g, k);
  const bool flip = (j < 0 && !g.pole_lo) || (j >= g.nt && !g.pole_hi);
  const double v = ldo(s.a[F_UR] + ((long)f * g.nt + clampi(j, 0, g.nt - 1)) * g.np, (unsigned)kk * 8u);
  return flip != (!g.periodic && kk != k) ? -v : v;
}
__device__ __forceinline__ double gT(const Geo &g, const SrcShell &s, int i, int f, int k) {
  const int kk = phi_in(g, k), ii = clampi(i, 0, g.nr - 1);
  const double v = ldo(s.a[F_UT] + ((long)ii * (g.nt + 1) + f) * g.np, (unsigned)kk * 8u);
  return (ii != i) != (!g.periodic && kk != k) ? -v : v;
}
__device__ __forceinline__ double gF(const Geo &g, const SrcShell &s, int i, int j, int f) {
  const int ff = g.periodic ? wrapk(g, f) : f, ii = clampi(i, 0, g.nr - 1), jj = clampi(j, 0, g.nt - 1);
  const double v = ldo(s.a[F_UF] + ((long)ii * g.nt + jj) * g.npf, (unsigned)ff * 8u);
  return (ii != i) != (jj != j) ? -v : v;
}
__device__ __forceinline__ double SrcShell::at(int f, int i, int j, int k) const {
  if (f == F_UR) return gR(g, *this, i, j, k);
  if (f == F_UT) return gT(g, *this, i, j, k);
  if (f == F_UF) return gF(g, *this, i, j, k);
  return gC(g, *this, f, i, j, k);
}

// the same for a forced pass: wall velocities (gR_wall and its like), source
struct SrcShellW {
  const double *a[5];
  Geo g;
  Wall w;
  bool has[4];  // as SrcInW
  __device__ __forceinline__ double wu(int q, const double *p, long x) const {
    const double v = p[x];
    return has[q] ? v : 0.0;
  }
  const double *f[5];
  static constexpr bool INTERIOR = false;
  static constexpr bool PERIODIC = false;
  static constexpr bool WALL = true;
  static constexpr bool PERT = false;
  static constexpr bool WIN = true;
  __device__ __forceinline__ double ld(int fid, long x) const { return a[fid][x]; }
  __device__ __forceinline__ double at(int fid, int i, int j, int k) const {
    if (fid == F_P || fid == F_T) {
      const long row = ((long)clampi(i, 0, g.nr - 1) * g.nt + clampi(j, 0, g.nt - 1)) * g.np;
      return ldo(a[fid] + row, (unsigned)phi_in(g, k) * 8u);
    }
    const int kk = fid == F_UF && !g.periodic ? k : phi_in(g, k), ii = clampi(i, 0, g.nr - 1), jj = clampi(j, 0, g.nt - 1);
    const unsigned o = (unsigned)kk * 8u;
    double sg = 1.0, add = 0.0;
    if (fid != F_UF && !g.periodic) { // phi wall
      const long x = fid == F_UR ? (long)i * g.nt + jj : (long)ii * (g.nt + 1) + j;
      const double w1 = fid == F_UR ? wu(0, w.ur_p1, x) : wu(2, w.ut_p1, x);
      const double w2 = fid == F_UR ? wu(1, w.ur_p2, x) : wu(3, w.ut_p2, x);
      add = kk == k ? 0.0 : 2.0 * (k < 0 ? w1 : w2);
      sg = kk == k ? 1.0 : -1.0;
    }
    if (fid != F_UT && jj != j) { // theta wall or pole
      const bool pole = j < 0 ? g.pole_lo : g.pole_hi;
      const long x = fid == F_UR ? (long)i * g.np : (long)ii * g.npf;
      const double *p = fid == F_UR ? (j < 0 ? w.ur_t1 : w.ur_t2) : (j < 0 ? w.uf_t1 : w.uf_t2);
      if (!pole && p) add += sg * 2.0 * ldo(p + x, o);
      if (!pole || fid == F_UF) sg = -sg;
    }
    if (fid != F_UR && ii != i) { // r wall
      const long x = fid == F_UT ? (long)j * g.np : (long)jj * g.npf;
      const double *p = fid == F_UT ? (i < 0 ? w.ut_r1 : w.ut_r2) : (i < 0 ? w.uf_r1 : w.uf_r2);
      if (p) add += sg * 2.0 * ldo(p + x, o);
      sg = -sg;
    }
    const long row = fid == F_UR ? ((long)i * g.nt + jj) * g.np
                                 : (fid == F_UT ? ((long)ii * (g.nt + 1) + j) * g.np : ((long)ii * g.nt + jj) * g.npf);
    return add + sg * ldo(a[fid] + row, o);
  }
};

// One block row, scaled by tau/2 with the identity added, structural
// non-zeros only (unknowns p, T, w).
struct FRow {
  double L0, L1, L2, L4, L5, L8;
  double D0, D1, D2, D4, D5, D6, D8;
  double U0, U1, U4, U6, U8;
  double b0, b1, b2;
};

// What a block row's coefficients depend on.  vel, G, gg, tr: the advecting
// velocity, the velocity gradient's entry and the curvature sum of the
// direction and the trace (Cent); irho: inverse mean density across the face
// after the cell; un: the velocity on it.  h: 1 / spacing of the direction;
// dp, dm: the divergence factors of the faces after and before the cell; lp,
// lm: the conduction factors; wp, w0, wm: the viscous factors of the face row.
struct RowIn {
  double vel, G, gg, tr, P, T, irho, un, b0, b1, b2;
};
struct RowMetric {
  double h, dp, dm, lp, lm, wp, w0, wm;
};

// first / last / before_last: the row's place on a line that does not close on
// itself (row 0, n - 1, n - 2); real: false for a filler
__device__ __forceinline__ void frow(const Mat &m, double hs, const RowIn &q, const RowMetric &x, bool first,
                                     bool last, bool before_last, bool real, FRow &R) {
  const double g1 = m.gam - 1.0, lp = last ? 0.0 : x.lp, lm = first ? 0.0 : x.lm;
  const double chi = g1 * q.T * rcp_nr(q.P);
  const double a = hs * (0.5 * x.h) * q.vel;
  const double tg = 2.0 * q.G * x.h, t3 = (2.0 / 3.0) * q.tr;
  const double ap = m.mu * (tg + q.gg - t3 * x.dp), am = m.mu * (q.gg - tg - t3 * x.dm);
  const double kp = hs * g1 * m.kap, kT = hs * chi * m.kap;
  const double gP = hs * m.gam * q.P, gT = hs * g1 * q.T, hg = hs * g1, hc = hs * chi;
  R.L0 = -a;
  R.U0 = a;
  R.L1 = -kp * lm;
  R.U1 = -kp * lp;
  R.D1 = kp * (lp + lm);
  R.L2 = gP * x.dm - hg * am;
  R.D2 = gP * x.dp - hg * ap;
  R.L4 = -a - kT * lm;
  R.U4 = a - kT * lp;
  R.D4 = 1.0 + kT * (lp + lm);
  R.L5 = gT * x.dm - hc * am;
  R.D5 = gT * x.dp - hc * ap;
  const double gp = hs * q.irho * x.h, hn = hs * m.mu * q.irho, au = hs * (0.5 * x.h) * q.un;
  R.D6 = -gp;
  R.U6 = gp;
  R.L8 = hn * x.wm - au;
  R.D8 = 1.0 + hn * x.w0;
  R.U8 = hn * x.wp + au;
  R.D0 = 1.0;
  R.b0 = q.b0;
  R.b1 = q.b1;
  R.b2 = q.b2;
  if (first) {  // advection ghosts p_{-1} = p_0, T_{-1} = T_0; no row before
    R.D0 -= a;
    R.D4 -= a;
    R.L0 = R.L1 = R.L2 = R.L4 = R.L5 = R.L8 = 0.0;
  }
  if (last) {  // ghosts alike; w is the boundary face
    R.D0 += a;
    R.D4 += a;
    R.D2 = R.D5 = R.D6 = 0.0;
    R.D8 = 1.0;
    R.L8 = 0.0;
    R.U0 = R.U1 = R.U4 = R.U6 = R.U8 = 0.0;
    R.b2 = 0.0;
  }
  if (before_last) R.U8 = 0.0;
  if (!real) {
    R.L0 = R.L4 = R.L8 = -1.0;
    R.D0 = R.D4 = R.D8 = 1.0;
    R.L1 = R.L2 = R.L5 = R.D1 = R.D2 = R.D5 = R.D6 = 0.0;
    R.U0 = R.U1 = R.U4 = R.U6 = R.U8 = 0.0;
    R.b0 = R.b1 = R.b2 = 0.0;
  }
}

// X = A^{-1} of a row's diagonal block, whose entries (1,0) and (2,1) are zero
__device__ __forceinline__ bool inv3d(const FRow &R, double *X) {
  const double c00 = R.D4 * R.D8, c01 = R.D5 * R.D6, c02 = -R.D4 * R.D6;
  const double det = fma_(R.D2, c02, fma_(R.D1, c01, R.D0 * c00));
  const double id = rcp_nr(det);
  X[0] = c00 * id;
  X[1] = -R.D1 * R.D8 * id;
  X[2] = fma_(R.D1, R.D5, -R.D2 * R.D4) * id;
  X[3] = c01 * id;
  X[4] = fma_(R.D0, R.D8, -R.D2 * R.D6) * id;
  X[5] = -R.D0 * R.D5 * id;
  X[6] = c02 * id;
  X[7] = R.D1 * R.D6 * id;
  X[8] = R.D0 * R.D4 * id;
  return !(det != 0.0) || !isfinite(det);
}

// A row of the transposed line: lower block U_{s-1}^T, diagonal D_s^T, upper
// block L_{s+1}^T, the right-hand side at row s's unknowns.
struct TRow {
  double l0, l1, l4, l6, l8;      // U_{s-1}
  double D0, D1, D2, D4, D5, D6, D8;
  double u0, u1, u2, u4, u5, u8;  // L_{s+1}
  double b0, b1, b2;
};
// from the rows before, at and after it; first / last of an open line: no row
// on that side; real: as in frow
__device__ __forceinline__ void trow(const FRow &M, const FRow &R, const FRow &P, bool first, bool last, bool real,
                                     TRow &t) {
  t.l0 = M.U0; t.l1 = M.U1; t.l4 = M.U4; t.l6 = M.U6; t.l8 = M.U8;
  t.D0 = R.D0; t.D1 = R.D1; t.D2 = R.D2; t.D4 = R.D4; t.D5 = R.D5; t.D6 = R.D6; t.D8 = R.D8;
  t.u0 = P.L0; t.u1 = P.L1; t.u2 = P.L2; t.u4 = P.L4; t.u5 = P.L5; t.u8 = P.L8;
  t.b0 = R.b0; t.b1 = R.b1; t.b2 = R.b2;
  if (first) t.l0 = t.l1 = t.l4 = t.l6 = t.l8 = 0.0;
  if (last || !real) t.u0 = t.u1 = t.u2 = t.u4 = t.u5 = t.u8 = 0.0;
  if (!real) {
    t.l0 = t.l4 = t.l8 = -1.0;
    t.l1 = t.l6 = 0.0;
    t.D0 = t.D4 = t.D8 = 1.0;
    t.D1 = t.D2 = t.D5 = t.D6 = 0.0;
    t.b0 = t.b1 = t.b2 = 0.0;
  }
}
__device__ __forceinline__ bool inv3d(const TRow &t, double *X) {
  FRow R;
  R.D0 = t.D0; R.D1 = t.D1; R.D2 = t.D2; R.D4 = t.D4; R.D5 = t.D5; R.D6 = t.D6; R.D8 = t.D8;
  double Y[9];
  const bool sing = inv3d(R, Y);
#pragma unroll
  for (int r = 0; r < 3; r++)
#pragma unroll
    for (int c = 0; c < 3; c++) X[r * 3 + c] = Y[c * 3 + r];
  return sing;
}

// Products with the sparse blocks of a row: C = L X, C = U X, B -= L X,
// y -= L x, y -= U x, C = A L, C = A U (A, X full), and the diagonal block.
__device__ __forceinline__ void diag3(const FRow &R, double *D) {
  D[0] = R.D0; D[1] = R.D1; D[2] = R.D2; D[3] = 0.0; D[4] = R.D4; D[5] = R.D5; D[6] = R.D6; D[7] = 0.0; D[8] = R.D8;
}
__device__ __forceinline__ void diag3(const TRow &R, double *D) {
  D[0] = R.D0; D[1] = 0.0; D[2] = R.D6; D[3] = R.D1; D[4] = R.D4; D[5] = 0.0; D[6] = R.D2; D[7] = R.D5; D[8] = R.D8;
}
__device__ __forceinline__ void mulL(const FRow &R, const double *X, double *C) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    C[c] = fma_(R.L2, X[6 + c], fma_(R.L1, X[3 + c], R.L0 * X[c]));
    C[3 + c] = fma_(R.L5, X[6 + c], R.L4 * X[3 + c]);
    C[6 + c] = R.L8 * X[6 + c];
  }
}
__device__ __forceinline__ void mulL(const TRow &R, const double *X, double *C) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    C[c] = fma_(R.l6, X[6 + c], R.l0 * X[c]);
    C[3 + c] = fma_(R.l4, X[3 + c], R.l1 * X[c]);
    C[6 + c] = R.l8 * X[6 + c];
  }
}
__device__ __forceinline__ void mulU(const FRow &R, const double *X, double *C) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    C[c] = fma_(R.U1, X[3 + c], R.U0 * X[c]);
    C[3 + c] = R.U4 * X[3 + c];
    C[6 + c] = fma_(R.U8, X[6 + c], R.U6 * X[c]);
  }
}
__device__ __forceinline__ void mulU(const TRow &R, const double *X, double *C) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    C[c] = R.u0 * X[c];
    C[3 + c] = fma_(R.u4, X[3 + c], R.u1 * X[c]);
    C[6 + c] = fma_(R.u8, X[6 + c], fma_(R.u5, X[3 + c], R.u2 * X[c]));
  }
}
__device__ __forceinline__ void subL(const FRow &R, const double *X, double *B) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    B[c] = fma_(-R.L2, X[6 + c], fma_(-R.L1, X[3 + c], fma_(-R.L0, X[c], B[c])));
    B[3 + c] = fma_(-R.L5, X[6 + c], fma_(-R.L4, X[3 + c], B[3 + c]));
    B[6 + c] = fma_(-R.L8, X[6 + c], B[6 + c]);
  }
}
__device__ __forceinline__ void subL(const TRow &R, const double *X, double *B) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    B[c] = fma_(-R.l6, X[6 + c], fma_(-R.l0, X[c], B[c]));
    B[3 + c] = fma_(-R.l4, X[3 + c], fma_(-R.l1, X[c], B[3 + c]));
    B[6 + c] = fma_(-R.l8, X[6 + c], B[6 + c]);
  }
}
__device__ __forceinline__ void subLv(const FRow &R, const double *x, double *y) {
  y[0] = fma_(-R.L2, x[2], fma_(-R.L1, x[1], fma_(-R.L0, x[0], y[0])));
  y[1] = fma_(-R.L5, x[2], fma_(-R.L4, x[1], y[1]));
  y[2] = fma_(-R.L8, x[2], y[2]);
}
__device__ __forceinline__ void subLv(const TRow &R, const double *x, double *y) {
  y[0] = fma_(-R.l6, x[2], fma_(-R.l0, x[0], y[0]));
  y[1] = fma_(-R.l4, x[1], fma_(-R.l1, x[0], y[1]));
  y[2] = fma_(-R.l8, x[2], y[2]);
}
__device__ __forceinline__ void subUv(const FRow &R, const double *x, double *y) {
  y[0] = fma_(-R.U1, x[1], fma_(-R.U0, x[0], y[0]));
  y[1] = fma_(-R.U4, x[1], y[1]);
  y[2] = fma_(-R.U8, x[2], fma_(-R.U6, x[0], y[2]));
}
__device__ __forceinline__ void subUv(const TRow &R, const double *x, double *y) {
  y[0] = fma_(-R.u0, x[0], y[0]);
  y[1] = fma_(-R.u4, x[1], fma_(-R.u1, x[0], y[1]));
  y[2] = fma_(-R.u8, x[2], fma_(-R.u5, x[1], fma_(-R.u2, x[0], y[2])));
}
__device__ __forceinline__ void mul_rU(const double *A, const FRow &R, double *C) {
#pragma unroll
  for (int r = 0; r < 3; r++) {
    C[r * 3] = fma_(A[r * 3 + 2], R.U6, A[r * 3] * R.U0);
    C[r * 3 + 1] = fma_(A[r * 3 + 1], R.U4, A[r * 3] * R.U1);
    C[r * 3 + 2] = A[r * 3 + 2] * R.U8;
  }
}
__device__ __forceinline__ void mul_rU(const double *A, const TRow &R, double *C) {
#pragma unroll
  for (int r = 0; r < 3; r++) {
    C[r * 3] = fma_(A[r * 3 + 2], R.u2, fma_(A[r * 3 + 1], R.u1, A[r * 3] * R.u0));
    C[r * 3 + 1] = fma_(A[r * 3 + 2], R.u5, A[r * 3 + 1] * R.u4);
    C[r * 3 + 2] = A[r * 3 + 2] * R.u8;
  }
}
__device__ __forceinline__ void mul_rL(const double *A, const FRow &R, double *C) {
#pragma unroll
  for (int r = 0; r < 3; r++) {
    C[r * 3] = A[r * 3] * R.L0;
    C[r * 3 + 1] = fma_(A[r * 3 + 1], R.L4, A[r * 3] * R.L1);
    C[r * 3 + 2] = fma_(A[r * 3 + 2], R.L8, fma_(A[r * 3 + 1], R.L5, A[r * 3] * R.L2));
  }
}
__device__ __forceinline__ void mul_rL(const double *A, const TRow &R, double *C) {
#pragma unroll
  for (int r = 0; r < 3; r++) {
    C[r * 3] = fma_(A[r * 3 + 1], R.l1, A[r * 3] * R.l0);
    C[r * 3 + 1] = A[r * 3 + 1] * R.l4;
    C[r * 3 + 2] = fma_(A[r * 3 + 2], R.l8, A[r * 3] * R.l6);
  }
}
// acc -= A B, y -= A x, A <- -(A B) for full blocks, one rounding per term
__device__ __forceinline__ void fsub3(const double *A, const double *P, double *B) {
#pragma unroll
  for (int r = 0; r < 3; r++)
#pragma unroll
    for (int c = 0; c < 3; c++)
      B[r * 3 + c] = fma_(-A[r * 3 + 2], P[6 + c], fma_(-A[r * 3 + 1], P[3 + c], fma_(-A[r * 3], P[c], B[r * 3 + c])));
}
__device__ __forceinline__ void fsubv(const double *A, const double *x, double *y) {
#pragma unroll
  for (int r = 0; r < 3; r++)
    y[r] = fma_(-A[r * 3 + 2], x[2], fma_(-A[r * 3 + 1], x[1], fma_(-A[r * 3], x[0], y[r])));
}
__device__ __forceinline__ void fneg3(double *A, const double *P) {
#pragma unroll
  for (int r = 0; r < 3; r++) {
    double t[3];
#pragma unroll
    for (int c = 0; c < 3; c++)
      t[c] = fma_(-A[r * 3 + 2], P[6 + c], fma_(-A[r * 3 + 1], P[3 + c], -A[r * 3] * P[c]));
#pragma unroll
    for (int c = 0; c < 3; c++) A[r * 3 + c] = t[c];
  }
}

// The chunk elimination, a row at a time.  State after row q (interior rows):
// x_q = Y_q - C_q x_{q+1} - E_q x_left.
template <int PM>
struct Chunk {
  double C[PM - 1][9], E[PM - 1][9], Y[PM - 1][3];
  bool sing = false;
  template <class Row>
  __device__ __forceinline__ void eliminate(int q, const Row &R) {
    double Ai[9], rr[3] = {R.b0, R.b1, R.b2};
    if (q == 0) {
      sing |= inv3d(R, Ai);
      mul_rL(Ai, R, E[0]);
    } else {
      double Dp[9], Lx[9];
      diag3(R, Dp);
      subL(R, C[q - 1], Dp);
      subLv(R, Y[q - 1], rr);
      mulL(R, E[q - 1], Lx);
      sing |= inv3q(Dp, Ai);
#pragma unroll
      for (int r = 0; r < 3; r++)
#pragma unroll
        for (int c = 0; c < 3; c++)
          E[q][r * 3 + c] = fma_(-Ai[r * 3 + 2], Lx[6 + c], fma_(-Ai[r * 3 + 1], Lx[3 + c], -Ai[r * 3] * Lx[c]));
    }
    mul_rU(Ai, R, C[q]);
    mv3(Ai, rr, Y[q]);
  }
  // (Y, C, E) -> x_q = Y_q + E_q x_left + C_q x_sep
  __device__ __forceinline__ void back() {
#pragma unroll
    for (int z = 0; z < 9; z++) { E[PM - 2][z] = -E[PM - 2][z]; C[PM - 2][z] = -C[PM - 2][z]; }
#pragma unroll
    for (int q = PM - 3; q >= 0; q--) {
      fsubv(C[q], Y[q + 1], Y[q]);
      double t[9];
#pragma unroll
      for (int z = 0; z < 9; z++) t[z] = -E[q][z];
      fsub3(C[q], E[q + 1], t);
#pragma unroll
      for (int z = 0; z < 9; z++) E[q][z] = t[z];
      fneg3(C[q], C[q + 1]);
    }
  }
  // the separator's row, the last interior row substituted and the first
  // interior row (g, V, W) of the chunk after: A x_left + B x + Cc x_next = r
  template <class Row>
  __device__ __forceinline__ void reduce(const Row &S, const double *gn, const double *Vn, const double *Wn,
                                         double *A, double *B, double *Cc, double *r) {
    double t9[9];
    mulL(S, E[PM - 2], A);
    mulL(S, C[PM - 2], t9);
    diag3(S, B);
#pragma unroll
    for (int z = 0; z < 9; z++) B[z] += t9[z];
    mulU(S, Vn, t9);
#pragma unroll
    for (int z = 0; z < 9; z++) B[z] += t9[z];
    mulU(S, Wn, Cc);
    r[0] = S.b0;
    r[1] = S.b1;
    r[2] = S.b2;
    subLv(S, Y[PM - 2], r);
    subUv(S, gn, r);
  }
  __device__ __forceinline__ void fill(int q, const double *xl, const double *xs, double *v) const {
#pragma unroll
    for (int r = 0; r < 3; r++)
      v[r] = fma_(C[q][r * 3 + 2], xs[2], fma_(C[q][r * 3 + 1], xs[1], fma_(C[q][r * 3], xs[0],
             fma_(E[q][r * 3 + 2], xl[2], fma_(E[q][r * 3 + 1], xl[1], fma_(E[q][r * 3], xl[0], Y[q][r]))))));
  }
};

// LDS record of a separator in the reductions: B^{-1} A, B^{-1} C, B^{-1} r,
// 22 doubles apart (16-byte aligned; 16 lanes of 16-byte accesses cover all
// banks once)
constexpr int SEP_REC = 22;

// One step of the parallel cyclic reduction is publish, barrier, fold, barrier:
// publish writes a separator's record, fold eliminates the separators at lo and
// hi.  Rows past either end of an open line need no test: their couplings are
// exactly zero, and lo / hi are any separator of the same line.
__device__ __forceinline__ bool sep_publish(const double *A, const double *B, const double *C, const double *r,
                                            double *rec) {
  double Bi[9], P[SEP_REC];
  const bool sing = inv3q(B, Bi);
  mm3(Bi, A, P);
  mm3(Bi, C, P + 9);
  mv3(Bi, r, P + 18);
  P[21] = 0.0;
#pragma unroll
  for (int z = 0; z < SEP_REC; z += 2) *(double2 *)(rec + z) = double2{P[z], P[z + 1]};
  return sing;
}
__device__ __forceinline__ void sep_fold(double *A, double *B, double *C, double *r, const double *lo,
                                         const double *hi) {
  double P[SEP_REC];
#pragma unroll
  for (int z = 0; z < SEP_REC; z += 2) { const double2 v = *(const double2 *)(lo + z); P[z] = v.x; P[z + 1] = v.y; }
  fsub3(A, P + 9, B);
  fsubv(A, P + 18, r);
  fneg3(A, P);
#pragma unroll
  for (int z = 0; z < SEP_REC; z += 2) { const double2 v = *(const double2 *)(hi + z); P[z] = v.x; P[z + 1] = v.y; }
  fsub3(C, P, B);
  fsubv(C, P + 18, r);
  fneg3(C, P + 9);
}

} // namespace dsw
