// Triangle algebra in symmetrising variables.
//
// At the Roe state (u, v, h, c) of a triangle a conserved perturbation x is
// held as y = (P, a, b, s),
//   a = x1 - u x0,  b = x2 - v x0,  P = dp / c,  s = x0 - P / c,
//   dp = (gamma - 1) (x3 - (q^2 / 2) x0 - u a - v b)    (q^2 = u^2 + v^2),
// and back by x0 = s + P / c, x1 = u x0 + a, x2 = v x0 + b,
// x3 = c P / (gamma - 1) + (q^2 / 2) x0 + u a + v b. In these variables every
// K(n) is symmetric and the entropy component s decouples: with m = n_i / 2
// the scaled normal of a corner, l = |m|, n = m / l its unit normal,
// w = u.m and C = l c (l up to the scale below),
//   K y = (w P + c m.(a, b),  w (a, b) + m c P,  w s),
// with the eigenvalues w + C, w - C (acoustic) and w (shear and entropy), so
// its positive part is, with p0 = w^+, A = ((w + C)^+ + (w - C)^+) / 2 - p0,
// B = ((w + C)^+ - (w - C)^+) / 2 and d = n.(a, b),
//   K^+ y = (p0 P + A P + B d,  p0 (a, b) + n (B P + A d),  p0 s),
// and K^- = K - K^+ has the coefficients w - p0, -A, C - B. The distribution
// is the same as in conserved variables (N, LDA and the residual are
// invariant under a linear change of variables at the Roe state); only the
// blends, whose coefficients are per conserved component, need x itself.
//
// A = sum_i K_i^+ is then a symmetric 3x3 matrix, positive definite at every
// state (a common null vector of the three K_i in (P, a, b) would need
// n.(a, b) = 0 for two independent normals and P = 0), beside the scalar
// sum_i p0_i of the entropy component: it is factored as L D L^T without
// pivoting, and the stagnant case of Section 3.3.1 is the scalar alone, whose
// unknown is 0 where sum_i p0_i is at most 2^-45 of the trace of the matrix.
// Against a pivoted 4x4 elimination of the conserved matrix this takes about
// half the instructions of a triangle, with no row selects.
#pragma once

#include "rd_math.h"

namespace rd {

// Scale. The distribution is homogeneous in K (the N unknown and the LDA
// coefficients do not change when every K_i is scaled, the residual and the
// parts scale with it) and linear in the differences dW, so the code below
// keeps K_i for the length 2 L_i of its edge where the scheme has L_i / 2
// (l = 2 L makes the halves in A and B free), and dW from the sum of the
// corners' parameter vectors where the scheme has their mean: what it returns
// is 12 times the residual and the parts.
constexpr double kSymScale = 1.0 / 12.0;

// Constants of the gas, made once on the host.
struct SymGas {
  double g1 = 0.4, ig1 = 2.5, gfac = 0.4 / 1.4;  // gamma - 1, its reciprocal, (gamma - 1) / gamma
  SymGas() = default;
  explicit SymGas(double gamma) : g1(gamma - 1.0), ig1(1.0 / (gamma - 1.0)), gfac((gamma - 1.0) / gamma) {}
};

template <typename R>
struct SymFlow {
  R u, v, c, ic, hq, cg, gc;  // hq = q^2 / 2, cg = c / (gamma - 1), gc = (gamma - 1) / c
};

// Unit normal and length of an edge's inward normal.
template <typename R>
struct SymEdge {
  R nx, ny, L;
};

// Coefficients of K_i: w, C = l c, and p0, A, B of its positive part.
template <typename R>
struct SymK {
  R w, C, p0, A, B;
};

// L D L^T of the acoustic 3x3 block (reciprocal pivots i0, i1, i2) and the
// reciprocal of the entropy sum (0 when stagnant).
template <typename R>
struct SymFactor {
  R i0, i1, i2, l1, l2, l3, ia;
};

// zs: the sum of the corners' parameter vectors.
template <typename R>
__host__ __device__ inline SymFlow<R> sym_flow(const R zs[4], const SymGas& gas) {
  SymFlow<R> f;
  const R iz = rcp_normal(zs[0]);
  f.u = zs[1] * iz;
  f.v = zs[2] * iz;
  f.hq = R(0.5) * (f.u * f.u + f.v * f.v);
  len_rcp(gas.g1 * (zs[3] * iz - f.hq), f.c, f.ic);
  f.cg = f.c * gas.ig1;
  f.gc = f.ic * gas.g1;
  return f;
}

// y of M(Zbar)(Z_i - Z_0), M = dW/dZ: x0 = 2 z0 dz0, x1 - u x0 = z0 dz1 - z1
// dz0, dp = (gamma - 1)/gamma (z3 dz0 + z0 dz3 - z1 dz1 - z2 dz2).
template <typename R>
__host__ __device__ inline void sym_difference(const SymFlow<R>& f, const R zb[4], R gfac, const R dz[4], R y[4]) {
  y[0] = gfac * (zb[3] * dz[0] + zb[0] * dz[3] - zb[1] * dz[1] - zb[2] * dz[2]);  // gfac = (gamma-1)/(gamma c)
  y[1] = zb[0] * dz[1] - zb[1] * dz[0];
  y[2] = zb[0] * dz[2] - zb[2] * dz[0];
  y[3] = R(2) * zb[0] * dz[0] - y[0] * f.ic;
}

template <typename R>
__host__ __device__ inline void sym_from_conserved(const SymFlow<R>& f, const R x[4], R y[4]) {
  y[1] = x[1] - f.u * x[0];
  y[2] = x[2] - f.v * x[0];
  y[0] = f.gc * (x[3] - f.hq * x[0] - f.u * y[1] - f.v * y[2]);
  y[3] = x[0] - y[0] * f.ic;
}

template <typename R>
__host__ __device__ inline void sym_to_conserved(const SymFlow<R>& f, const R y[4], R x[4]) {
  x[0] = y[3] + y[0] * f.ic;
  x[1] = f.u * x[0] + y[1];
  x[2] = f.v * x[0] + y[2];
  x[3] = f.cg * y[0] + f.hq * x[0] + f.u * y[1] + f.v * y[2];
}

template <typename R>
__host__ __device__ inline SymK<R> sym_k(const SymFlow<R>& f, const SymEdge<R>& e) {
  SymK<R> k;
  const R hw = e.L * (f.u * e.nx + f.v * e.ny), hC = e.L * f.c;  // w / 2, C / 2
  const R a = rmax(hw + hC, R(0)), b = rmax(hw - hC, R(0));
  k.w = hw + hw;
  k.C = hC + hC;
  k.p0 = rmax(k.w, R(0));
  k.A = (a + b) - k.p0;
  k.B = a - b;
  return k;
}

// out = p0 y + A, B terms (K^+ with (p0, A, B), K^- with (w - p0, -A, C - B)).
template <typename R>
__host__ __device__ inline void sym_split(const SymEdge<R>& e, R p0, R A, R B, const R y[4], R out[4]) {
  const R d = e.nx * y[1] + e.ny * y[2];
  const R g = B * y[0] + A * d;
  out[0] = (p0 + A) * y[0] + B * d;
  out[1] = p0 * y[1] + e.nx * g;
  out[2] = p0 * y[2] + e.ny * g;
  out[3] = p0 * y[3];
}

// out += K y
template <typename R>
__host__ __device__ inline void sym_full_add(const SymFlow<R>& f, const SymEdge<R>& e, const SymK<R>& k, const R y[4],
                                             R out[4]) {
  const R cp = k.C * y[0];
  out[0] = out[0] + (k.w * y[0] + k.C * (e.nx * y[1] + e.ny * y[2]));
  out[1] = out[1] + (k.w * y[1] + e.nx * cp);
  out[2] = out[2] + (k.w * y[2] + e.ny * cp);
  out[3] = out[3] + k.w * y[3];
}

// The entries of sum_i K_i^+ as its corners are added.
template <typename R>
struct SymMatrix {
  R al = R(0), a = R(0), m01 = R(0), m02 = R(0), s11 = R(0), s12 = R(0), s22 = R(0);
  __host__ __device__ void add(const SymEdge<R>& e, const SymK<R>& k) {
    al = al + k.p0;
    a = a + k.A;
    m01 = m01 + k.B * e.nx;
    m02 = m02 + k.B * e.ny;
    const R ax = k.A * e.nx, ay = k.A * e.ny;
    s11 = s11 + ax * e.nx;
    s12 = s12 + ax * e.ny;
    s22 = s22 + ay * e.ny;
  }
};

template <typename R>
__host__ __device__ inline SymFactor<R> sym_factor(const SymMatrix<R>& m) {
  const R m00 = m.al + m.a, m11 = m.al + m.s11, m22 = m.al + m.s22;
  SymFactor<R> q;
  q.i0 = rcp_normal(m00);
  q.l1 = m.m01 * q.i0;
  q.l2 = m.m02 * q.i0;
  q.i1 = rcp_normal(m11 - q.l1 * m.m01);
  const R t = m.s12 - q.l1 * m.m02;
  q.l3 = t * q.i1;
  q.i2 = rcp_normal(m22 - q.l2 * m.m02 - q.l3 * t);
  const R tol = (m00 + m11 + m22) * R(2.8421709430404007e-14);  // 2^-45
  q.ia = m.al > tol ? rcp_normal(m.al) : R(0);
  return q;
}

// x = A^{-1} b
template <typename R>
__host__ __device__ inline void sym_solve(const SymFactor<R>& q, const R b[4], R x[4]) {
  const R y1 = b[1] - q.l1 * b[0];
  const R y2 = b[2] - q.l2 * b[0] - q.l3 * y1;
  x[2] = y2 * q.i2;
  x[1] = y1 * q.i1 - q.l3 * x[2];
  x[0] = b[0] * q.i0 - q.l1 * x[1] - q.l2 * x[2];
  x[3] = b[3] * q.ia;
}

// Edges of a triangle from its unwrapped corner differences (corner 1 minus
// 0, corner 2 minus 0); returns the longest edge's length.
template <typename R>
__host__ __device__ inline R sym_edges(R d1x, R d1y, R d2x, R d2y, SymEdge<R> e[3]) {
  // inward normals scaled by edge length: the opposite edge rotated by +90 degrees
  const R nx[3] = {d1y - d2y, d2y, -d1y}, ny[3] = {d2x - d1x, -d2x, d1x};
  R lmax = R(0);
  for (int i = 0; i < 3; ++i) {
    R L, iL;
    len_rcp(nx[i] * nx[i] + ny[i] * ny[i], L, iL);
    lmax = rmax(lmax, L);
    e[i].nx = nx[i] * iL;
    e[i].ny = ny[i] * iL;
    e[i].L = L;
  }
  return lmax;
}

// A triangle at given corner parameter vectors, what its parts need: flow,
// coefficients of corners 0 and 1, difference of corner 1, residual phi^T,
// factored matrix and (NEEDN) x_N = A^{-1} sum_i K_i^- dW_i.
template <typename R>
struct SymTri {
  SymFlow<R> f;
  SymK<R> k[2];
  SymFactor<R> q;
  R dy1[4], phi[4], xN[4];
};

// Keeps the scheduler from interleaving what stands before and after it
// (which would hold both sides' values in registers at once).
__host__ __device__ inline void sched_fence() {
#ifdef __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_sched_barrier(0);
#endif
}

template <typename R, bool NEEDN>
__host__ __device__ inline void sym_triangle(const R z0[4], const R z1[4], const R z2[4], const SymEdge<R> e[3],
                                             const SymGas& gas, SymTri<R>& s) {
  R zb[4], dz[4];
  for (int k = 0; k < 4; ++k) zb[k] = z0[k] + z1[k] + z2[k];
  s.f = sym_flow(zb, gas);
  const R gfac = R(gas.gfac) * s.f.ic;
  // corners 2, 1, 0 in turn, so that corner 2's edge, difference and
  // coefficients are done with first
  SymMatrix<R> m;
  R b[4], t[4], dy2[4];
  for (int k = 0; k < 4; ++k) dz[k] = z2[k] - z0[k];
  sym_difference(s.f, zb, gfac, dz, dy2);
  for (int k = 0; k < 4; ++k) dz[k] = z1[k] - z0[k];
  sym_difference(s.f, zb, gfac, dz, s.dy1);
  for (int k = 0; k < 4; ++k) s.phi[k] = R(0);
  {
    const SymK<R> k2 = sym_k(s.f, e[2]);
    m.add(e[2], k2);
    sym_full_add(s.f, e[2], k2, dy2, s.phi);
    if (NEEDN) sym_split(e[2], k2.w - k2.p0, -k2.A, k2.C - k2.B, dy2, b);
  }
  s.k[1] = sym_k(s.f, e[1]);
  m.add(e[1], s.k[1]);
  sym_full_add(s.f, e[1], s.k[1], s.dy1, s.phi);
  if (NEEDN) {
    sym_split(e[1], s.k[1].w - s.k[1].p0, -s.k[1].A, s.k[1].C - s.k[1].B, s.dy1, t);
    for (int k = 0; k < 4; ++k) b[k] = b[k] + t[k];
  }
  s.k[0] = sym_k(s.f, e[0]);
  m.add(e[0], s.k[0]);
  s.q = sym_factor(m);
  if (NEEDN) sym_solve(s.q, b, s.xN);
}

// N parts phi^N_i = K_i^+ (dW_i + x_N) of corners 0 and 1, in conserved
// variables (the parts sum to phi^T, which gives corner 2's).
template <typename R>
__host__ __device__ inline void sym_n_parts(const SymTri<R>& s, const SymEdge<R> e[3], R p0[4], R p1[4]) {
  R y[4], o[4];
  sym_split(e[0], s.k[0].p0, s.k[0].A, s.k[0].B, s.xN, o);
  sym_to_conserved(s.f, o, p0);
  for (int k = 0; k < 4; ++k) y[k] = s.dy1[k] + s.xN[k];
  sym_split(e[1], s.k[1].p0, s.k[1].A, s.k[1].B, y, o);
  sym_to_conserved(s.f, o, p1);
}

// LDA parts K_i^+ A^{-1} y of corners 0 and 1 of the residual y (symmetrising
// variables), in conserved variables.
template <typename R>
__host__ __device__ inline void sym_lda_parts(const SymTri<R>& s, const SymEdge<R> e[3], const R y[4], R p0[4],
                                              R p1[4]) {
  R x[4], o[4];
  sym_solve(s.q, y, x);
  sym_split(e[0], s.k[0].p0, s.k[0].A, s.k[0].B, x, o);
  sym_to_conserved(s.f, o, p0);
  sym_split(e[1], s.k[1].p0, s.k[1].A, s.k[1].B, x, o);
  sym_to_conserved(s.f, o, p1);
}

}  // namespace rd
