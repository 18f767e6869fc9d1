// Three-dimensional residual distribution on tetrahedra (the method of
// Section 3 with a row and a column added to every matrix, as the paper's
// closing discussion describes): bodies of the gfx950 kernels in
// rd3_kernels.hip. FP64 throughout.
//
// The algebra of a tetrahedron runs in symmetrising variables. At its Roe
// state (u, H, c) a conserved perturbation x is held as y = (P, a, s),
//   a = x_1..3 - u x_0,  P = dp / c,  s = x_0 - P / c,
//   dp = (gamma - 1) (x_4 - (|u|^2 / 2) x_0 - u.a),
// in which every K(n) is symmetric and the entropy component s decouples:
// with N the inward normal of the face opposite a corner (twice its area
// long), n = N / |N|, w = u.N and C = |N| c (up to the scale below),
//   K y = (w P + C n.a, w a + n C P, w s),
//   K^+ y = (p0 P + A P + B n.a, p0 a + n (B P + A n.a), p0 s)
// with p0 = w^+, A = ((w + C)^+ + (w - C)^+) / 2 - p0, B = ((w + C)^+ -
// (w - C)^+) / 2; K^- = K - K^+ has w - p0, -A and C - B. The distribution is
// invariant under this change of variables; only the blends, whose
// coefficients are per conserved component, need x itself. sum_i K_i^+ is a
// symmetric 4x4 block, positive definite at every state (a null vector would
// need P + n_i.a = 0 for four normals that span space), beside the scalar
// sum_i p0_i: it is factored as L D L^T without pivoting, and a fluid at rest
// is the scalar alone, whose unknown is 0 where the sum is at most 2^-45 of
// the block's trace. A pivoted 5x5 elimination of the conserved matrix takes
// more than twice the instructions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rd_math.h"

namespace rd3 {

using rd::len_rcp;
using rd::rcp_normal;
using rd::rmax;
using rd::rmin;

constexpr int kBlock = 256;
constexpr int kTileTets = 256;    // most tetrahedra of a tile (one thread each)
constexpr int kTileVerts = 256;   // most vertices
// Doubles between two components' part planes in LDS: 4 parts of every
// tetrahedron, and 13 more modulo 32, so that the sums of 13 neighbouring
// vertices' five components fall on different banks.
__host__ __device__ inline int part_plane(int tets) { return (4 * tets + 31) / 32 * 32 + 13; }

enum { S_N = 0, S_LDA = 1, S_B = 2, S_BMAX = 3, S_BMIN = 4 };

// One tile: at most kTileTets tetrahedra, their vertices (by falling number of
// the tile's tetrahedra at each), and the jagged diagonals their parts are
// summed along.
struct Tile3 {
  int32_t t0, nt;    // tetrahedra
  int32_t l0, nlv;   // local vertices
  int32_t j0, nj;    // the tile's diagonals in jb
};

// Device view of a tetrahedral mesh and its state, vertices in internal order
// (tile by tile).
struct Dev3 {
  int64_t nv = 0;
  int32_t ntiles = 0, threads = 0, max_lv = 0, max_tet = 0;
  int32_t jb_at = 0, lds = 0;       // LDS of a tile workgroup: where its diagonals start, bytes
  double gamma = 1.4, g1 = 0.4, ig1 = 2.5, gfac = 0.4 / 1.4;
  double per[3] = {0, 0, 0}, half[3] = {0, 0, 0};  // periods, and half of each (infinite where not periodic)
  const Tile3* tile = nullptr;      // [ntiles]
  const uint4* tet = nullptr;       // [nt] of each corner its local vertex, and its part's slot << 16
  const int32_t* lv = nullptr;      // vertex of each local vertex
  const uint16_t* deg = nullptr;    // tile's tetrahedra at each local vertex
  const int32_t* rpos = nullptr;    // record its sum goes to
  const int32_t* jb = nullptr;      // first slot of each diagonal
  const int32_t* rbeg = nullptr;    // [nv + 1] records of vertex v (ascending tile)
  const int32_t* inv = nullptr;     // [nv] vertex of each of the caller's
  const double* V = nullptr;        // [nv] vertex volume (sum of |T| / 4)
  double* W = nullptr;              // [5][nv] state
  double* Ws = nullptr;             // [5][nv] first-stage state
  double2* r1 = nullptr;            // [nv][5] Z of W, |u| + c, position, unused
  double2* r2 = nullptr;            // [nv][5] Z of W*, (W* - W^n) / dt
  double* rec = nullptr;            // [records][6] a tile's sum of parts at a vertex, and of CFL terms
  double* dt = nullptr;             // device scalar: the step's time step
  double* bmin = nullptr;           // [blocks] partial minima of the CFL limit
  int* flag = nullptr;              // non-physical state latch (rho <= 0, p <= 0 or not finite)
};

// Z and |u| + c of a state; returns whether it is physical (rho > 0, p > 0,
// finite).
__device__ inline bool to_z(const double w[5], double gamma, double z[5], double& sig) {
  const double rho = w[0], iu = 1.0 / rho;
  const double u = w[1] * iu, v = w[2] * iu, ww = w[3] * iu;
  const double q2 = u * u + v * v + ww * ww;
  const double p = (gamma - 1.0) * (w[4] - 0.5 * rho * q2);
  const double s = sqrt(rho);
  z[0] = s;
  z[1] = s * u;
  z[2] = s * v;
  z[3] = s * ww;
  z[4] = s * (w[4] + p) * iu;
  sig = sqrt(q2) + sqrt(gamma * p * iu);
  return rho > 0.0 && p > 0.0 && isfinite(sig) && isfinite(z[4]) && isfinite(z[1] + z[2] + z[3]);
}

// Scale. The distribution is homogeneous in K and linear in the differences:
// the code keeps K_i for 2 |N_i| where the scheme has |N_i| / 6 (the halves in
// A and B are free then) and the differences from the sum of the corners'
// parameter vectors where it has their mean, so residual and parts are 48
// times the scheme's; stage 2 leaves out the halves of its means too (96).
constexpr double kScale1 = 1.0 / 48.0, kScale2 = 1.0 / 96.0;

struct Flow {
  double u[3], c, ic, hq, cg, gc;  // hq = |u|^2 / 2, cg = c / (gamma - 1), gc = (gamma - 1) / c
};

// Unit normal of a corner and p0, A, B of its K^+.
struct Corner {
  double n[3], p0, A, B;
};

// L D L^T of the acoustic 4x4 block (reciprocal pivots) and the reciprocal of
// the entropy sum (0 at rest).
struct Factor {
  double i[4], l10, l20, l30, l21, l31, l32, ia;
};

__device__ inline void to_conserved(const Flow& f, const double y[5], double x[5]) {
  x[0] = y[4] + y[0] * f.ic;
  for (int k = 0; k < 3; ++k) x[1 + k] = f.u[k] * x[0] + y[1 + k];
  x[4] = f.cg * y[0] + f.hq * x[0] + f.u[0] * y[1] + f.u[1] * y[2] + f.u[2] * y[3];
}

__device__ inline void from_conserved(const Flow& f, const double x[5], double y[5]) {
  for (int k = 0; k < 3; ++k) y[1 + k] = x[1 + k] - f.u[k] * x[0];
  y[0] = f.gc * (x[4] - f.hq * x[0] - f.u[0] * y[1] - f.u[1] * y[2] - f.u[2] * y[3]);
  y[4] = x[0] - y[0] * f.ic;
}

// out = K^+ y
__device__ inline void split(const double n[3], double p0, double A, double B, const double y[5], double out[5]) {
  const double d = n[0] * y[1] + n[1] * y[2] + n[2] * y[3];
  const double g = B * y[0] + A * d;
  out[0] = (p0 + A) * y[0] + B * d;
  for (int k = 0; k < 3; ++k) out[1 + k] = p0 * y[1 + k] + n[k] * g;
  out[4] = p0 * y[4];
}

__device__ inline void solve(const Factor& q, const double b[5], double x[5]) {
  const double y1 = b[1] - q.l10 * b[0];
  const double y2 = b[2] - q.l20 * b[0] - q.l21 * y1;
  const double y3 = b[3] - q.l30 * b[0] - q.l31 * y1 - q.l32 * y2;
  x[3] = y3 * q.i[3];
  x[2] = y2 * q.i[2] - q.l32 * x[3];
  x[1] = y1 * q.i[1] - q.l21 * x[2] - q.l31 * x[3];
  x[0] = b[0] * q.i[0] - q.l10 * x[1] - q.l20 * x[2] - q.l30 * x[3];
  x[4] = b[4] * q.ia;
}

// sum_i K_i^+ as its corners are added.
struct Matrix {
  double al = 0.0, a = 0.0, m[3] = {0.0, 0.0, 0.0}, s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // 11 12 13 22 23 33
  __device__ void add(const Corner& k) {
    al += k.p0;
    a += k.A;
    for (int j = 0; j < 3; ++j) m[j] += k.B * k.n[j];
    const double x = k.A * k.n[0], y = k.A * k.n[1], z = k.A * k.n[2];
    s[0] += x * k.n[0];
    s[1] += x * k.n[1];
    s[2] += x * k.n[2];
    s[3] += y * k.n[1];
    s[4] += y * k.n[2];
    s[5] += z * k.n[2];
  }
};

__device__ inline Factor factor(const Matrix& m) {
  Factor q;
  const double m00 = m.al + m.a, m11 = m.al + m.s[0], m22 = m.al + m.s[3], m33 = m.al + m.s[5];
  q.i[0] = rcp_normal(m00);
  q.l10 = m.m[0] * q.i[0];
  q.l20 = m.m[1] * q.i[0];
  q.l30 = m.m[2] * q.i[0];
  q.i[1] = rcp_normal(m11 - q.l10 * m.m[0]);
  const double t21 = m.s[1] - q.l20 * m.m[0], t31 = m.s[2] - q.l30 * m.m[0];
  q.l21 = t21 * q.i[1];
  q.l31 = t31 * q.i[1];
  q.i[2] = rcp_normal(m22 - q.l20 * m.m[1] - q.l21 * t21);
  const double t32 = m.s[4] - q.l30 * m.m[1] - q.l31 * t21;
  q.l32 = t32 * q.i[2];
  q.i[3] = rcp_normal(m33 - q.l30 * m.m[2] - q.l31 * t31 - q.l32 * t32);
  const double tol = (m00 + m11 + m22 + m33) * 2.8421709430404007e-14;  // 2^-45
  q.ia = m.al > tol ? rcp_normal(m.al) : 0.0;
  return q;
}

// A tetrahedron at given corner parameter vectors: what its parts need.
struct Tet {
  Flow f;
  Corner k[3];          // corners 0, 1, 2 (the parts sum to the residual, which gives corner 3's)
  double dy[2][5];      // differences of corners 1 and 2 from corner 0
  double phi[5], xN[5]; // residual, sum_i K_i^- dW_i solved (symmetrising variables)
  Factor q;
};

// Keeps the scheduler from interleaving what stands before and after it.
__device__ inline void fence() { __builtin_amdgcn_sched_barrier(0); }

// Corner from its face normal; adds K y to phi and K^- y to b where y is given.
__device__ inline Corner corner(const Flow& f, const double N[3], const double* y, double phi[5], double b[5],
                                bool needn) {
  Corner k;
  double L, iL;
  len_rcp(N[0] * N[0] + N[1] * N[1] + N[2] * N[2], L, iL);
  for (int j = 0; j < 3; ++j) k.n[j] = N[j] * iL;
  const double hw = f.u[0] * N[0] + f.u[1] * N[1] + f.u[2] * N[2], hC = L * f.c;
  const double p = rmax(hw + hC, 0.0), m = rmax(hw - hC, 0.0);
  const double w = hw + hw, C = hC + hC;
  k.p0 = rmax(w, 0.0);
  k.A = (p + m) - k.p0;
  k.B = p - m;
  if (y) {
    const double d = k.n[0] * y[1] + k.n[1] * y[2] + k.n[2] * y[3], cp = C * y[0];
    phi[0] += w * y[0] + C * d;
    for (int j = 0; j < 3; ++j) phi[1 + j] += w * y[1 + j] + k.n[j] * cp;
    phi[4] += w * y[4];
    if (needn) {
      double t[5];
      split(k.n, w - k.p0, -k.A, C - k.B, y, t);
      for (int j = 0; j < 5; ++j) b[j] += t[j];
    }
  }
  return k;
}

// z(i): parameter vector of corner i; N: face normals of corners 0..3.
template <bool NEEDN, class Z>
__device__ inline void tet_eval(const Dev3& d, const Z& z, const double N[4][3], Tet& s) {
  double z0[5], z1[5], z2[5], z3[5], zs[5];
  z(0, z0);
  z(1, z1);
  z(2, z2);
  z(3, z3);
  for (int k = 0; k < 5; ++k) zs[k] = z0[k] + z1[k] + z2[k] + z3[k];
  Flow& f = s.f;
  const double iz = rcp_normal(zs[0]);
  for (int k = 0; k < 3; ++k) f.u[k] = zs[1 + k] * iz;
  f.hq = 0.5 * (f.u[0] * f.u[0] + f.u[1] * f.u[1] + f.u[2] * f.u[2]);
  len_rcp(d.g1 * (zs[4] * iz - f.hq), f.c, f.ic);
  f.cg = f.c * d.ig1;
  f.gc = f.ic * d.g1;
  const double gf = d.gfac * f.ic;
  auto diff = [&](const double zi[5], double y[5]) {
    double dz[5];
    for (int k = 0; k < 5; ++k) dz[k] = zi[k] - z0[k];
    y[0] = gf * (zs[4] * dz[0] + zs[0] * dz[4] - zs[1] * dz[1] - zs[2] * dz[2] - zs[3] * dz[3]);
    for (int k = 1; k < 4; ++k) y[k] = zs[0] * dz[k] - zs[k] * dz[0];
    y[4] = 2.0 * zs[0] * dz[0] - y[0] * f.ic;
  };
  Matrix m;
  double b[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, dy3[5];
  for (int k = 0; k < 5; ++k) s.phi[k] = 0.0;
  diff(z3, dy3);
  diff(z2, s.dy[1]);
  diff(z1, s.dy[0]);
  m.add(corner(f, N[3], dy3, s.phi, b, NEEDN));
  s.k[2] = corner(f, N[2], s.dy[1], s.phi, b, NEEDN);
  m.add(s.k[2]);
  s.k[1] = corner(f, N[1], s.dy[0], s.phi, b, NEEDN);
  m.add(s.k[1]);
  s.k[0] = corner(f, N[0], nullptr, s.phi, b, false);
  m.add(s.k[0]);
  s.q = factor(m);
  if (NEEDN) solve(s.q, b, s.xN);
}

// N part of corner i < 3 in conserved variables.
__device__ inline void n_part(const Tet& s, int i, double out[5]) {
  double y[5], o[5];
  for (int k = 0; k < 5; ++k) y[k] = i == 0 ? s.xN[k] : s.dy[i - 1][k] + s.xN[k];
  split(s.k[i].n, s.k[i].p0, s.k[i].A, s.k[i].B, y, o);
  to_conserved(s.f, o, out);
}

// The scheme's parts of the four corners from the residual being split, the N
// parts of corners 0..2 and the unknown xT of the LDA parts. Blends: Theta_k =
// min(1, |res_k| / sum_i |N_ik|), 0 for a zero sum (1e-300 added to the sum
// changes no quotient whose sum is above 1e-284), one common value for Bmax
// and Bmin.
template <int SCHEME>
__device__ inline void scheme_parts(const Tet& s, const double res[5], const double pn[3][5], const double xT[5],
                                    double out[4][5]) {
  double th[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (SCHEME >= S_B) {
    for (int k = 0; k < 5; ++k) {
      const double den = fabs(pn[0][k]) + fabs(pn[1][k]) + fabs(pn[2][k]) +
                         fabs(res[k] - pn[0][k] - pn[1][k] - pn[2][k]);
      th[k] = rmin(fabs(res[k]) * rcp_normal(den + 1e-300), 1.0);
    }
    if (SCHEME != S_B) {
      double t = th[0];
      for (int k = 1; k < 5; ++k) t = SCHEME == S_BMAX ? rmax(t, th[k]) : rmin(t, th[k]);
      for (int k = 0; k < 5; ++k) th[k] = t;
    }
  }
  for (int k = 0; k < 5; ++k) out[3][k] = res[k];
  for (int i = 0; i < 3; ++i) {
    if (SCHEME == S_N) {
      for (int k = 0; k < 5; ++k) out[i][k] = pn[i][k];
    } else {
      double o[5], pl[5];
      split(s.k[i].n, s.k[i].p0, s.k[i].A, s.k[i].B, xT, o);
      to_conserved(s.f, o, pl);
      for (int k = 0; k < 5; ++k) out[i][k] = SCHEME == S_LDA ? pl[k] : pl[k] + th[k] * (pn[i][k] - pl[k]);
    }
    for (int k = 0; k < 5; ++k) out[3][k] -= out[i][k];
  }
}

}  // namespace rd3
