// Shared per-element bodies: records and layouts, the vertex's parameter
// vector, the ordered sums, and the second view of a mesh that the
// residual, the adjoint and the FP32 step use: a triangle pass writes parts, a
// vertex pass sums a vertex's parts over the vertex->(triangle, corner) CSR in
// ascending triangle order (no atomics) and adds the wall term. The FP64 step
// runs in the patch form (rd_patch.h); the triangle algebra of FP64 is in
// rd_sym.h, that of FP32 in rd_fp32.h.
//
// Parts of the second view are stored sliced: vertices are taken 64 at a time
// (one wavefront of the gather), a slice is as wide as its largest vertex
// degree, and the j-th part (ascending triangle order) of the slice's l-th
// vertex sits at slice_base + 64 j + l. The triangle pass writes each corner's
// part straight to its slot; the gather's j-th load is then one contiguous,
// fully coalesced read across the wavefront. A corner's slot is formed from
// its vertex v (slice v / 64, lane v % 64) and the rank j of the triangle
// among v's triangles; the three ranks of a triangle are packed 10 bits
// each into one word, so a triangle pass reads 4 bytes of slot data per
// triangle instead of three 32-bit slot positions.
//
// Algebra of the FP32 step and of the adjoint's reverse passes (equal in exact
// arithmetic to Appendix A's explicit entries; the adjoint's stage-1
// recomputation uses rd_sym.h): with unit normal n, Roe state (u, v, h, c),
// w = u n_x + v n_y,
//   E = (1, u, v, h), N = (0, n_x, n_y, w),
//   g(y) = alpha/c y0 - (gamma-1)(u/c y1 + v/c y2 - y3/c),
//   d(y) = -w y0 + n_x y1 + n_y y2,
// the matrix with eigenvalues (l1, l2, l3, l3) on the acoustic and the two
// linear waves acts as
//   K(l) y = l3 y + (l1-l3)/(2c) (g+d) (E + c N) + (l2-l3)/(2c) (g-d) (E - c N),
// i.e. K(l) = l3 I + (l1-l3) r1 l1^T + (l2-l3) r2 l2^T with r_{1,2} = E +- c N
// the acoustic right eigenvectors and l_{1,2}^T the matching rows of R^{-1}.
// This needs no 4x4 matrix per corner; only A = sum_i K_i^+ is built.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "rd_math.h"
#include "rd_sym.h"

namespace rd {

template <typename R>
struct alignas(4 * sizeof(R)) Q4 {
  R v[4];
};
using D4 = Q4<double>;
using F4 = Q4<float>;

// One wall-edge incidence of a wall vertex (Section 3.5).
struct alignas(16) WallEnt {
  int32_t other;  // the edge's other vertex
  int32_t role;   // 0: this vertex is the edge's start a, 1: its end b
  double hl;      // half the edge length
  double nx, ny;  // outward unit normal
};

enum { SCH_N = 0, SCH_LDA = 1, SCH_B = 2, SCH_BMAX = 3, SCH_BMIN = 4, SCH_BX = 5 };

// Where the state is: in one of the two buffers of the patch form (internal
// order), or, after FP32 steps, in the FP32 form's own. Which, is held on the
// device (cur[0]), so that captured steps replay correctly however many ran
// before. A stage-1 pass reads cur[0] and its first workgroup copies it to
// cur[1], which no workgroup of that pass reads; a stage-2 pass reads cur[1],
// writes the other buffer, and its first workgroup sets cur[0] to it, which no
// workgroup of that pass reads.
constexpr int kForm32 = 2;
struct State {
  D4* W[2];
  const int* cur;
  const int32_t* inv;  // internal vertex of each of the caller's
  D4* W32;             // the FP32 form's, the caller's order
  // record of the caller's vertex v
  __host__ __device__ D4* at(int64_t v) const {
    const int c = *cur;
    return c == kForm32 ? W32 + v : W[c] + inv[v];
  }
};

// The second view of a mesh (or of a batch laid end to end): vertices and
// triangles in the caller's order.
struct Dev {
  int64_t nv = 0, nt = 0;
  int32_t nwv = 0;
  double gamma = 1.4, px = 0.0, py = 0.0;
  double hpx = 0.0, hpy = 0.0;  // half periods, +inf on an axis that is not periodic
  double igamma = 1.0 / 1.4;  // 1 / gamma (set with gamma on the host)
  SymGas gas;
  // geometry and connectivity
  const double2* xy = nullptr;   // [nv]
  const double* V = nullptr;     // [nv] vertex volume
  const int32_t* row = nullptr;  // [nv+1] CSR row pointers (row[v+1] - row[v] = degree of v)
  const int32_t* sbase = nullptr; // [ceil(nv/64)] first part slot of each 64-vertex slice
  int64_t ns = 0;                // part slots, including the padding of the 64-vertex slices
  const int32_t* vtri = nullptr; // [ns] triangle of each part slot (padding slots unused)
  const int32_t* bc = nullptr;   // [nv] or null: boundary code, see is_ghost / wall_index
  const int32_t* tv = nullptr;   // [3][nt] corner vertex ids
  const uint32_t* rk = nullptr;  // [nt] rank of t among the triangles of corner i's vertex, bits 10 i .. 10 i + 9
  const int32_t* wv = nullptr;   // [nwv] wall vertex ids
  const int32_t* wptr = nullptr; // [nwv+1]
  const WallEnt* went = nullptr; // wall incidences, ascending edge id per vertex
  const int32_t* tmesh = nullptr; // [nt] mesh id (batch) or null
  const int32_t* vmesh = nullptr; // [nv] mesh id (batch) or null
  // state
  D4* W = nullptr;    // [nv] state
  D4* Ws = nullptr;   // [nv] first-stage state
  D4* Z = nullptr;    // [nv] parameter vector
  double* sig = nullptr;   // [nv] |v| + c
  // triangle buffers
  void* C = nullptr;      // [ns] distributed parts, sliced layout (D4 records in 16-byte planes)
  void* keepN = nullptr;  // stage-1 N parts of corners 0 and 1 (2 nt records; 16-byte planes)
  void* keepT = nullptr;  // stage-1 triangle residual (nt records; 16-byte planes)
  D4* WCn = nullptr;      // [nwv] wall term at W^n
  D4* WCs = nullptr;      // [nwv] wall term at W*
  void* lam = nullptr;    // [nt] l_max^T lambda_max^T per triangle
  double* dt = nullptr;   // [nmesh] time step
  double* vr = nullptr;   // [3 nmesh] Bx sensor: smallest and largest |v| at the stage's state, domain size L
  int* flag = nullptr;    // [nmesh] non-physical state latch
};

// Boundary code of a vertex: -1 interior, -2 ghost, b >= 0 wall vertex b,
// -3 - b ghost that is also wall vertex b (its wall term is never applied,
// but its state enters its neighbours' wall terms).
__host__ __device__ inline bool is_ghost(int32_t bc) { return bc == -2 || bc <= -3; }
__host__ __device__ inline int32_t wall_index(int32_t bc) { return bc >= 0 ? bc : (bc <= -3 ? -3 - bc : -1); }

// First part slot of vertex v: its j-th part is at vslot(d, v) + 64 j.
__host__ __device__ inline int64_t vslot(const Dev& d, int64_t v) { return (int64_t)d.sbase[v >> 6] + (v & 63); }

// Part slot of corner i (vertex v) of a triangle with rank word rk.
__host__ __device__ inline int32_t corner_slot(const Dev& d, int32_t v, uint32_t rk, int i) {
  return d.sbase[v >> 6] + (v & 63) + 64 * (int32_t)((rk >> (10 * i)) & 1023u);
}

template <typename R>
__host__ __device__ inline R sel4(int r, R a0, R a1, R a2, R a3) {
  R t = r == 1 ? a1 : a0;
  t = r == 2 ? a2 : t;
  return r == 3 ? a3 : t;
}

// Per-corner coefficients of K_i^{+-} (scaled by s = |n_i|/2).
template <typename R>
struct Corner {
  R nx, ny, w, s;
  R l3p, h1p, h2p;  // s l3^+, s (l1^+ - l3^+)/(2c), s (l2^+ - l3^+)/(2c)
  R l3m, h1m, h2m;  // same for the negative parts
};

template <typename R>
struct Roe {
  R u, v, h, c, ic, ac, uc, vc, g1;
};

// y -> K^{+} y or K^{-} y of one corner.
template <typename R>
__host__ __device__ inline void apply_split(const Roe<R>& q, const Corner<R>& k, R sl3, R h1, R h2,
                                            const R y[4], R out[4]) {
  R g = q.ac * y[0] - q.g1 * (q.uc * y[1] + q.vc * y[2] - q.ic * y[3]);
  R d = -k.w * y[0] + k.nx * y[1] + k.ny * y[2];
  R a1 = h1 * (g + d), a2 = h2 * (g - d);
  R sp = a1 + a2, sm = (a1 - a2) * q.c;
  out[0] = sl3 * y[0] + sp;
  out[1] = sl3 * y[1] + sp * q.u + sm * k.nx;
  out[2] = sl3 * y[2] + sp * q.v + sm * k.ny;
  out[3] = sl3 * y[3] + sp * q.h + sm * k.w;
}

// y -> K y (l = lambda): s (w y + d E + c g N).
template <typename R>
__host__ __device__ inline void apply_full(const Roe<R>& q, const Corner<R>& k, const R y[4], R out[4]) {
  R g = q.ac * y[0] - q.g1 * (q.uc * y[1] + q.vc * y[2] - q.ic * y[3]);
  R d = -k.w * y[0] + k.nx * y[1] + k.ny * y[2];
  R cg = q.c * g;
  out[0] = k.s * (k.w * y[0] + d);
  out[1] = k.s * (k.w * y[1] + d * q.u + cg * k.nx);
  out[2] = k.s * (k.w * y[2] + d * q.v + cg * k.ny);
  out[3] = k.s * (k.w * y[3] + d * q.h + cg * k.w);
}

// A = sum_i K_i^+ as a dense 4x4 matrix:
// A = L3 I + E ev^T + c (sum Q_i N_i) G^T + c sum_i P_i N_i D_i^T with
// P = h1 + h2, Q = h1 - h2, G = (alpha/c, -g1 u/c, -g1 v/c, g1/c), D_i = (-w, nx, ny, 0).
template <typename R>
__host__ __device__ inline void build_A(const Roe<R>& q, const Corner<R> k[3], R A[4][4]) {
  R G[4] = {q.ac, -q.g1 * q.uc, -q.g1 * q.vc, q.g1 * q.ic};
  R E[4] = {R(1), q.u, q.v, q.h};
  R L3 = k[0].l3p + k[1].l3p + k[2].l3p;
  R P[3], Qv[3];
  for (int i = 0; i < 3; ++i) {
    P[i] = k[i].h1p + k[i].h2p;
    Qv[i] = k[i].h1p - k[i].h2p;
  }
  R sP = P[0] + P[1] + P[2];
  R ev[4];
  ev[0] = sP * G[0] - (Qv[0] * k[0].w + Qv[1] * k[1].w + Qv[2] * k[2].w);
  ev[1] = sP * G[1] + (Qv[0] * k[0].nx + Qv[1] * k[1].nx + Qv[2] * k[2].nx);
  ev[2] = sP * G[2] + (Qv[0] * k[0].ny + Qv[1] * k[1].ny + Qv[2] * k[2].ny);
  ev[3] = sP * G[3];
  R nvv[4];
  nvv[0] = R(0);
  nvv[1] = q.c * (Qv[0] * k[0].nx + Qv[1] * k[1].nx + Qv[2] * k[2].nx);
  nvv[2] = q.c * (Qv[0] * k[0].ny + Qv[1] * k[1].ny + Qv[2] * k[2].ny);
  nvv[3] = q.c * (Qv[0] * k[0].w + Qv[1] * k[1].w + Qv[2] * k[2].w);
  // S[r][j] for r = 1..3 (N rows nx, ny, w) and j = 0..2 (D cols -w, nx, ny)
  R S[4][4];
  for (int r = 0; r < 4; ++r)
    for (int j = 0; j < 4; ++j) S[r][j] = R(0);
  for (int i = 0; i < 3; ++i) {
    R cp = q.c * P[i];
    R Nr[4] = {R(0), k[i].nx, k[i].ny, k[i].w};
    R Dc[4] = {-k[i].w, k[i].nx, k[i].ny, R(0)};
    for (int r = 1; r < 4; ++r) {
      R t = cp * Nr[r];
      for (int j = 0; j < 3; ++j) S[r][j] = S[r][j] + t * Dc[j];
    }
  }
  for (int r = 0; r < 4; ++r)
    for (int j = 0; j < 4; ++j) {
      R a = E[r] * ev[j] + nvv[r] * G[j] + S[r][j];
      A[r][j] = r == j ? a + L3 : a;
    }
}

// Reciprocal of a pivot: FP64 by IEEE division, FP32 by the hardware
// reciprocal (about 1 ulp).
__host__ __device__ inline double pivot_rcp(double x) { return 1.0 / x; }
__host__ __device__ inline float rcp32(float x) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}
__host__ __device__ inline float pivot_rcp(float x) { return rcp32(x); }

// Gaussian elimination with partial pivoting for two right-hand sides
// (A, b0 and b1 are overwritten).
// Pivot: largest |entry| among rows not yet used, lowest row on ties; a
// column whose best pivot is at most 2^-45 max|A| is skipped and its unknown
// set to 0 (A is singular at stagnation; the K^+ x products stay unique).
// `skipped` reports whether any column was skipped.
template <typename R>
__host__ __device__ inline void solve2(R A[4][4], R b0[4], R b1[4], R x0[4], R x1[4], bool& skipped) {
  R amax = R(0);
  for (int r = 0; r < 4; ++r)
    for (int c = 0; c < 4; ++c) amax = rmax(amax, (R)fabs(A[r][c]));
  const R tol = amax * R(2.8421709430404007e-14);  // 2^-45
  bool used[4] = {false, false, false, false};
  R P[4][4], PB0[4], PB1[4], PI[4];
  bool OK[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    R best = R(-1);
    int r = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      R a = (R)fabs(A[i][k]);
      bool take = !used[i] && a > best;
      best = take ? a : best;
      r = take ? i : r;
    }
    const bool ok = best > tol;
    OK[k] = ok;
#pragma unroll
    for (int j = k; j < 4; ++j) P[k][j] = sel4(r, A[0][j], A[1][j], A[2][j], A[3][j]);
    PB0[k] = sel4(r, b0[0], b0[1], b0[2], b0[3]);
    PB1[k] = sel4(r, b1[0], b1[1], b1[2], b1[3]);
    PI[k] = ok ? pivot_rcp(P[k][k]) : R(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) used[i] = used[i] || (ok && r == i);
    // rows not eliminated get factor 0, which leaves them exactly unchanged
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const R f = (ok && !used[i]) ? A[i][k] * PI[k] : R(0);
#pragma unroll
      for (int j = k + 1; j < 4; ++j) A[i][j] = A[i][j] - f * P[k][j];
      b0[i] = b0[i] - f * PB0[k];
      b1[i] = b1[i] - f * PB1[k];
    }
  }
#pragma unroll
  for (int k = 3; k >= 0; --k) {
    R s0 = PB0[k], s1 = PB1[k];
#pragma unroll
    for (int j = k + 1; j < 4; ++j) {
      s0 = s0 - P[k][j] * x0[j];
      s1 = s1 - P[k][j] * x1[j];
    }
    x0[k] = OK[k] ? s0 * PI[k] : R(0);
    x1[k] = OK[k] ? s1 * PI[k] : R(0);
  }
  skipped = !(OK[0] && OK[1] && OK[2] && OK[3]);
}

template <typename R>
__host__ __device__ inline void solve2(R A[4][4], R b0[4], R b1[4], R x0[4], R x1[4]) {
  bool skipped;
  solve2(A, b0, b1, x0, x1, skipped);
}

// Blend coefficient of Section 3.3.3: Theta_k = |res_k| / sum_i |N_{i,k}|,
// 0 if the sum (den) is 0, at most 1. 1e-300 is added to the sum: it changes
// no quotient whose sum is above 1e-284, makes 0 / 0 a 0, and keeps the
// reciprocal finite at the edge of a uniform state at rest, where the parts
// decay to subnormal values.
__host__ __device__ inline double blend_quotient(double res, double den) {
  return rmin(fabs(res) * rcp_normal(den + 1e-300), 1.0);
}

// The scheme's parts of the three corners from the N and LDA parts of corners
// 0 and 1 and the residual being split, which the parts of every scheme sum
// to; BMAX / BMIN use the largest / smallest Theta_k for all components, BX
// the coefficient bx.
template <int SCHEME>
__host__ __device__ inline void blend_parts(const double res[4], const double n0[4], const double n1[4],
                                            const double l0[4], const double l1[4], double bx, double out[3][4]) {
  double th[4] = {bx, bx, bx, bx};
  if (SCHEME >= SCH_B && SCHEME <= SCH_BMIN)
    for (int k = 0; k < 4; ++k)
      th[k] = blend_quotient(res[k], fabs(n0[k]) + fabs(n1[k]) + fabs(res[k] - n0[k] - n1[k]));
  if (SCHEME == SCH_BMAX || SCHEME == SCH_BMIN) {
    const double t = SCHEME == SCH_BMAX ? rmax(rmax(th[0], th[1]), rmax(th[2], th[3]))
                                        : rmin(rmin(th[0], th[1]), rmin(th[2], th[3]));
    for (int k = 0; k < 4; ++k) th[k] = t;
  }
  for (int k = 0; k < 4; ++k) {
    if (SCHEME == SCH_N) {
      out[0][k] = n0[k];
      out[1][k] = n1[k];
    } else if (SCHEME == SCH_LDA) {
      out[0][k] = l0[k];
      out[1][k] = l1[k];
    } else {
      out[0][k] = l0[k] + th[k] * (n0[k] - l0[k]);
      out[1][k] = l1[k] + th[k] * (n1[k] - l1[k]);
    }
    out[2][k] = res[k] - out[0][k] - out[1][k];
  }
}

template <typename R>
__host__ __device__ inline Q4<R> ld4(const void* base, int64_t i) {
  return reinterpret_cast<const Q4<R>*>(base)[i];
}
template <typename R>
__host__ __device__ inline void st4(void* base, int64_t i, const R a[4]) {
  Q4<R> q;
  q.v[0] = a[0];
  q.v[1] = a[1];
  q.v[2] = a[2];
  q.v[3] = a[3];
  reinterpret_cast<Q4<R>*>(base)[i] = q;
}

// Records of four reals in planes of 16-byte chunks: chunk c of record j of
// item i sits at chunk index (KC j + c) n + i, where n is the number of items
// and KC the number of chunks per record (2 for FP64, 1 for FP32). One store
// or load instruction of a wavefront over consecutive items then covers one
// contiguous kilobyte instead of a strided span of partly written lines.
// Used for the distributed parts (item = part slot, one record) and for the
// kept stage-1 records of a triangle (N parts of corners 0 and 1 in keepN,
// phi^T in keepT), which are read back only by the stage-2 pass, after the
// gather: those are stored non-temporally (NT), so that they do not evict
// from the caches the parts and parameter vectors the next kernel reads.
template <typename R> struct Chunk16;
template <> struct Chunk16<double> { typedef double V __attribute__((ext_vector_type(2))); };
template <> struct Chunk16<float> { typedef float V __attribute__((ext_vector_type(4))); };

template <typename R, bool NT>
__host__ __device__ inline void plane_store(void* base, int64_t n, int64_t i, int j, const R a[4]) {
  typedef typename Chunk16<R>::V V;
  constexpr int per = 16 / sizeof(R), kc = 4 / per;
  V* p = reinterpret_cast<V*>(base);
  for (int c = 0; c < kc; ++c) {
    V q;
    for (int e = 0; e < per; ++e) q[e] = a[c * per + e];
#ifdef __HIP_DEVICE_COMPILE__
    if (NT) __builtin_nontemporal_store(q, p + (kc * j + c) * n + i);
    else p[(kc * j + c) * n + i] = q;
#else
    p[(kc * j + c) * n + i] = q;
#endif
  }
}

template <typename R>
__host__ __device__ inline Q4<R> plane_load(const void* base, int64_t n, int64_t i, int j) {
  typedef typename Chunk16<R>::V V;
  constexpr int per = 16 / sizeof(R), kc = 4 / per;
  const V* p = reinterpret_cast<const V*>(base);
  Q4<R> q;
  for (int c = 0; c < kc; ++c) {
    const V x = p[(kc * j + c) * n + i];
    for (int e = 0; e < per; ++e) q.v[c * per + e] = x[e];
  }
  return q;
}

template <typename R>
__host__ __device__ inline void keep_store(void* base, int64_t nt, int64_t t, int j, const R a[4]) {
  plane_store<R, true>(base, nt, t, j, a);
}
template <typename R>
__host__ __device__ inline Q4<R> keep_load(const void* base, int64_t nt, int64_t t, int j) {
  return plane_load<R>(base, nt, t, j);
}
// Part of slot s in C.
template <typename R>
__host__ __device__ inline void part_store(const Dev& d, int64_t s, const R a[4]) {
  plane_store<R, false>(d.C, d.ns, s, 0, a);
}
template <typename R>
__host__ __device__ inline Q4<R> part_load(const Dev& d, int64_t s) {
  return plane_load<R>(d.C, d.ns, s, 0);
}

// Unwrapped corner differences of a triangle (corner 1 minus 0, 2 minus 0).
struct TriDiff {
  double d1x, d1y, d2x, d2y;
};
// M: anything with the periods px, py and half periods hpx, hpy.
template <class M>
__host__ __device__ inline TriDiff tri_diff(const M& m, const double2& a, const double2& b, const double2& c) {
  return TriDiff{unwrap_select(b.x - a.x, m.px, m.hpx), unwrap_select(b.y - a.y, m.py, m.hpy),
                 unwrap_select(c.x - a.x, m.px, m.hpx), unwrap_select(c.y - a.y, m.py, m.hpy)};
}

// Bx blend coefficient (Section 3.3.3): theta = min(1, s^2 h / L) with the
// shock sensor s = (-L div v / (|v|max - |v|min))^+, div v that of the linear
// interpolant of the corner velocities (u = Z_1 / Z_0, v = Z_2 / Z_0), h =
// sqrt(2 |T|); r: range of |v| at this stage's state, domain size L.
__host__ __device__ inline double bx_theta(const TriDiff& g, const D4 z[3], const double* r) {
  const double nx[3] = {g.d1y - g.d2y, g.d2y, -g.d1y}, ny[3] = {g.d2x - g.d1x, -g.d2x, g.d1x};
  double div = 0.0;
  for (int i = 0; i < 3; ++i) div = div + (z[i].v[1] * nx[i] + z[i].v[2] * ny[i]) / z[i].v[0];
  const double a2 = g.d1x * g.d2y - g.d1y * g.d2x;  // 2 |T|
  const double range = r[1] - r[0], L = r[2];
  const double s = range > 0.0 ? rmax(-(L * div) / (a2 * range), 0.0) : 0.0;
  return rmin(s * s * sqrt(a2) / L, 1.0);
}

// Stage 1 of one triangle (Sections 3.2-3.3): the scheme's parts of its
// corners, the N parts of corners 0 and 1 and the residual, all divided by
// kSymScale; returns its longest edge. vr: the Bx sensor's range (bx_theta).
template <int SCHEME>
__host__ __device__ inline double stage1_parts(const TriDiff& g, const D4 z[3], const SymGas& gas, const double* vr,
                                               double out[3][4], double pN[2][4], double phi[4]) {
  constexpr bool needN = SCHEME != SCH_LDA, needL = SCHEME != SCH_N;
  const double bx = SCHEME == SCH_BX ? bx_theta(g, z, vr) : 0.0;
  SymEdge<double> e[3];
  const double lmax = sym_edges(g.d1x, g.d1y, g.d2x, g.d2y, e);
  SymTri<double> s;
  sym_triangle<double, needN>(z[0].v, z[1].v, z[2].v, e, gas, s);
  double pl[2][4];
  sym_to_conserved(s.f, s.phi, phi);
  if (needN) sym_n_parts(s, e, pN[0], pN[1]);
  if (needL) sym_lda_parts(s, e, s.phi, pl[0], pl[1]);
  blend_parts<SCHEME>(phi, pN[0], pN[1], pl[0], pl[1], bx, out);
  return lmax;
}

// Stage 1 of triangle t of the second view: its parts to C, the N parts of
// corners 0 and 1 and the residual to keepN, keepT (corner 2's N part is phi^T
// minus those two).
template <int SCHEME>
__host__ __device__ inline void tri_body(int64_t t, const Dev& d) {
  int32_t iv[3];
  D4 z[3];
  for (int i = 0; i < 3; ++i) {
    iv[i] = d.tv[i * d.nt + t];
    z[i] = d.Z[iv[i]];
  }
  const uint32_t rk = d.rk[t];
  double out[3][4], pN[2][4], phi[4];
  stage1_parts<SCHEME>(tri_diff(d, d.xy[iv[0]], d.xy[iv[1]], d.xy[iv[2]]), z, d.gas, d.vr, out, pN, phi);
  for (int k = 0; k < 4; ++k) {
    phi[k] *= kSymScale;
    if (SCHEME != SCH_LDA) {
      pN[0][k] *= kSymScale;
      pN[1][k] *= kSymScale;
    }
    for (int i = 0; i < 3; ++i) out[i][k] *= kSymScale;
  }
  if (SCHEME != SCH_LDA) {
    keep_store<double>(d.keepN, d.nt, t, 0, pN[0]);
    keep_store<double>(d.keepN, d.nt, t, 1, pN[1]);
  }
  keep_store<double>(d.keepT, d.nt, t, 0, phi);
  for (int i = 0; i < 3; ++i) part_store<double>(d, corner_slot(d, iv[i], rk, i), out[i]);
}

// Flow speed |v| of a conserved state.
__host__ __device__ inline double flow_speed(const D4& w) {
  const double u = w.v[1] / w.v[0], v = w.v[2] / w.v[0];
  return sqrt(u * u + v * v);
}

// Parameter vector, signal speed and physicality of one state.
struct VertexDerived {
  double z[4];
  double sig;
  bool ok;
};

// Square root of x >= 0 (NaN for x < 0): on the device x times the reciprocal
// square root (rsq_step; within about an ulp or two, exactly 0 at 0), on the
// host IEEE.
__host__ __device__ inline double sqrt_nr(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  const double y = rsq_step(x, __builtin_amdgcn_rsq(x));
  return x == 0.0 ? 0.0 : x * y;
#else
  return sqrt(x);
#endif
}

// Parameter vector Z = sqrt(rho) (1, u, v, h) and |v| + c of a conserved
// state, with one reciprocal of rho (rcp) and Newton-Raphson square roots.
__host__ __device__ inline VertexDerived derive(double gamma, const double w[4]) {
  VertexDerived o;
  const double g1 = gamma - 1.0;
  const double rho = w[0], ir = rcp(rho), u = w[1] * ir, vv = w[2] * ir;
  const double p = g1 * (w[3] - 0.5 * rho * (u * u + vv * vv));
  const double h = (w[3] + p) * ir;
  const double s = sqrt_nr(rho);
  o.z[0] = s;
  o.z[1] = s * u;
  o.z[2] = s * vv;
  o.z[3] = s * h;
  const double q2 = u * u + vv * vv, a2 = gamma * p * ir;
  o.sig = sqrt_nr(q2) + sqrt_nr(a2);
  const bool finite = q2 < INFINITY && a2 < INFINITY && fabs(w[1]) < INFINITY && fabs(w[2]) < INFINITY &&
                      fabs(w[3]) < INFINITY;
  o.ok = rho > 0.0 && p > 0.0 && finite;
  return o;
}

// Z of a conserved state into the second view; returns whether it is physical.
__host__ __device__ inline bool vertex_z(const Dev& d, int64_t v, const double w[4]) {
  const VertexDerived o = derive(d.gamma, w);
  D4 z;
  for (int k = 0; k < 4; ++k) z.v[k] = o.z[k];
  d.Z[v] = z;
  return o.ok;
}

// f(j, get(j)) for j = 0, ..., n-1 in that order. The loads of J consecutive
// j are issued before any is consumed, so a wavefront keeps several
// independent loads in flight instead of one.
template <int J = 4, class Get, class F>
__host__ __device__ inline void for_loaded(int32_t n, const Get& get, const F& f) {
  using T = decltype(get(0));
  for (int32_t j = 0; j < n; j += J) {
    T x[J];
#pragma unroll
    for (int u = 0; u < J; ++u)
      if (j + u < n) x[u] = get(j + u);
#pragma unroll
    for (int u = 0; u < J; ++u)
      if (j + u < n) f(j + u, x[u]);
  }
}

// Sum of a vertex's n parts get(0), ..., get(n-1) in that order.
template <class Get>
__host__ __device__ inline void sum_parts(int32_t n, const Get& get, double acc[4]) {
  for (int k = 0; k < 4; ++k) acc[k] = 0.0;
  for_loaded(n, get, [&](int32_t, const D4& c) {
    for (int k = 0; k < 4; ++k) acc[k] += c.v[k];
  });
}

// The update of Sections 3.3-3.4: out = in - (dt / V) acc.
__host__ __device__ inline void vertex_update(const double in[4], double f, const double acc[4], double out[4]) {
  for (int k = 0; k < 4; ++k) out[k] = in[k] - f * acc[k];
}

// phi^T of triangle t at the state st, into component-major arrays. The fluxes
// are bilinear in Z, so sum_i K_i dW_i is their differential at the mean of the
// corners' Z in the direction of sum_i n_i (Z_i - Z_0): no root and no matrix.
// Error against more than 64 bits (four quadrants, Sod, 800^2 points): 3.8e-16 and
// 1.7e-16; 1.2e-15 and 7.5e-16 by the step's symmetrising variables with the
// differences fused with the products in Z, which left 1e-19 on triangles of
// equal states.
__host__ __device__ inline void phi_body(int64_t t, const Dev& d, const State& st, double* soa) {
  D4 z[3];
  double2 xy[3];
  for (int i = 0; i < 3; ++i) {
    const int32_t v = d.tv[i * d.nt + t];
    const VertexDerived o = derive(d.gamma, st.at(v)->v);
    for (int k = 0; k < 4; ++k) z[i].v[k] = o.z[k];
    xy[i] = d.xy[v];
  }
  const TriDiff g = tri_diff(d, xy[0], xy[1], xy[2]);
  double s[4], x[4], y[4];
  for (int k = 0; k < 4; ++k) {
    double d1, d2;
    {
#pragma clang fp contract(off)  // not fused with the products in Z: equal states differ by 0
      d1 = z[1].v[k] - z[0].v[k];
      d2 = z[2].v[k] - z[0].v[k];
      s[k] = z[0].v[k] + z[1].v[k] + z[2].v[k];
    }
    x[k] = g.d2y * d1 - g.d1y * d2;
    y[k] = g.d1x * d2 - g.d2x * d1;
  }
  const double f = (d.gamma - 1.0) / d.gamma;
  const double px = f * (s[0] * x[3] + s[3] * x[0] - s[1] * x[1] - s[2] * x[2]);
  const double py = f * (s[0] * y[3] + s[3] * y[0] - s[1] * y[1] - s[2] * y[2]);
  const double phi[4] = {s[0] * (x[1] + y[2]) + s[1] * x[0] + s[2] * y[0],
                         2.0 * s[1] * x[1] + px + s[1] * y[2] + s[2] * y[1],
                         s[1] * x[2] + s[2] * x[1] + 2.0 * s[2] * y[2] + py,
                         s[3] * (x[1] + y[2]) + s[1] * x[3] + s[2] * y[3]};
  for (int k = 0; k < 4; ++k) soa[k * d.nt + t] = phi[k] / 6.0;
}

// Wall term (Section 3.5) of vertex v: the sum over its wall incidences
// went[e0, e1) of half the edge's length times the split flux of its two ends;
// state(i) gives the conserved state of vertex i.
template <class S>
__host__ __device__ inline void wall_term(const WallEnt* went, int32_t e0, int32_t e1, int64_t v, double gamma,
                                          const S& state, double acc[4]) {
  const double alpha = 0.75, g1 = gamma - 1.0;
  for (int k = 0; k < 4; ++k) acc[k] = 0.0;
  for (int32_t e = e0; e < e1; ++e) {
    const WallEnt we = went[e];
    double F[2][4];
    const int64_t ids[2] = {v, we.other};
    for (int s = 0; s < 2; ++s) {
      const D4 w = state(ids[s]);
      const double u = w.v[1] / w.v[0], vv = w.v[2] / w.v[0];
      const double p = g1 * (w.v[3] - 0.5 * w.v[0] * (u * u + vv * vv));
      const double vn = u * we.nx + vv * we.ny;
      F[s][0] = -vn * w.v[0];
      F[s][1] = -vn * w.v[1];
      F[s][2] = -vn * w.v[2];
      F[s][3] = -vn * (w.v[3] + p);
    }
    for (int k = 0; k < 4; ++k) {
      const double part = we.role == 0 ? alpha * F[0][k] + (1.0 - alpha) * F[1][k]
                                       : (1.0 - alpha) * F[1][k] + alpha * F[0][k];
      acc[k] += we.hl * part;
    }
  }
}

// The wall term of wall vertex b of the second view, at W or at Ws.
template <bool STAGE2>
__host__ __device__ inline void wall_body(int64_t b, const Dev& d) {
  const D4* W = STAGE2 ? d.Ws : d.W;
  D4 acc;
  wall_term(d.went, d.wptr[b], d.wptr[b + 1], d.wv[b], d.gamma, [&](int64_t i) { return W[i]; }, acc.v);
  (STAGE2 ? d.WCs : d.WCn)[b] = acc;
}

// 2 V_i / sum_{T ni i} l_max lambda_max of U vertices v[u] (terms of type R),
// each vertex's triangles taken in ascending order; out[u] is meaningful
// where in[u]. The triangles of the first J ranks of all U vertices are
// loaded before any term, and all those terms before any sum, so that the U
// chains of dependent loads (row bounds and slice base, triangle, term)
// overlap. Every load is in bounds whatever the degree, so none needs a
// branch: a vertex out of range reads vertex vsafe, a rank past the degree
// rereads the last rank (or slot 0 at degree 0) and its term is replaced by
// an exact zero. Ranks from J on follow one at a time.
template <typename R, int U, int J = 8>
__host__ __device__ inline void cfl_vertex_bounds(const int64_t v[U], const bool in[U], int64_t vsafe,
                                                  const Dev& d, double out[U]) {
  const R* lam = reinterpret_cast<const R*>(d.lam);
  int32_t deg[U];
  int64_t s0[U];
  double vol[U];
  for (int u = 0; u < U; ++u) {
    const int64_t w = in[u] ? v[u] : vsafe;
    deg[u] = d.row[w + 1] - d.row[w];
    s0[u] = vslot(d, w);
    vol[u] = d.V[w];
  }
  int32_t t[U][J];
  for (int u = 0; u < U; ++u)
    for (int j = 0; j < J; ++j) {
      const int64_t k = deg[u] > 0 ? s0[u] + 64 * (int64_t)(j < deg[u] ? j : deg[u] - 1) : 0;
      t[u][j] = d.vtri[k];
    }
  R term[U][J];
  for (int u = 0; u < U; ++u)
    for (int j = 0; j < J; ++j) {
      const R x = lam[t[u][j] > 0 ? t[u][j] : 0];
      term[u][j] = j < deg[u] ? x : R(0);
    }
  for (int u = 0; u < U; ++u) {
    double acc = 0.0;
    for (int j = 0; j < J; ++j) acc += (double)term[u][j];
    for (int32_t j = J; j < deg[u]; ++j) acc += (double)lam[d.vtri[s0[u] + 64 * (int64_t)j]];
    out[u] = 2.0 * vol[u] / acc;
  }
}

}  // namespace rd
