// The step with FP32 distribution (RD_FP32_ACC64): the triangle algebra in
// FP32 on the conserved variables (a pivoted 4x4 elimination), the vertex sums
// compensated in FP64, the state in FP64. It runs over the second view of the
// mesh (Dev, rd_device.h) in two passes, a triangle pass that writes every part
// to HBM and a vertex pass that sums them, or, with a tile size, tile by tile
// (rd_tiles.h). The FP64 step's algebra in symmetrising variables is not used:
// rounded to FP32 it lands 6e-8 (largest, of the rms) from these results on
// 2048^2 vertices after two steps, twice as far as a reordering of this
// algebra. The patch form with this algebra would give the same bits without
// the parts' way through HBM (the two gathers are 0.32 of the 0.87 ms of a
// 2048^2 step); it is not built.
#pragma once

#include "rd_device.h"

namespace rd {

enum { G_EULER = 0, G_STAGE1 = 1, G_STAGE2 = 2 };

// Buffers of the FP32 passes.
struct Dev32 {
  F4* Zf = nullptr;       // [nv] parameter vector
  F4* dW = nullptr;       // [nv] W* - W^n
  void* C = nullptr;      // [ns] distributed parts, sliced layout (one F4 per slot)
  void* keepN = nullptr;  // stage-1 N parts of corners 0 and 1 (2 nt records)
  void* keepT = nullptr;  // stage-1 triangle residual (nt records)
  int slump = 0;          // selective lumping in stage 2
  // tiled form
  D4* R1 = nullptr;       // [nv] stage-1 residual (sum of parts + wall term)
  double* cflv = nullptr; // [nv] CFL bound of each vertex
};

// Length with its reciprocal from one hardware reciprocal square root.
__host__ __device__ inline void len_rcp32(float e2, float& L, float& iL) {
#ifdef __HIP_DEVICE_COMPILE__
  iL = __builtin_amdgcn_rsqf(e2);
  L = e2 * iL;
#else
  L = sqrtf(e2);
  iL = 1.0f / L;
#endif
}

// Blend of Section 3.3.3: Theta_k = |res_k| / sum_i |N_{i,k}| (0 if the sum is
// 0, at most 1); BMAX / BMIN use the largest / smallest Theta_k for all k.
// den_k = sum_i |N_{i,k}| is accumulated by the caller in corner order.
// The quotient is a |res_k| times the reciprocal of den_k; where that product
// is not below 1 (the clamp, or a reciprocal that overflowed because den_k
// is below ~1/DBL_MAX, as happens at the edge of a uniform state at rest
// where the parts have decayed to subnormal values) the exact quotient
// decides.
template <int SCHEME>
__host__ __device__ inline void blend_theta32(const float res[4], const float den[4], float th[4]) {
  for (int k = 0; k < 4; ++k) {
    const float a = (float)fabs(res[k]);
    float q = 0.0f;
    if (den[k] > 0.0f && a > 0.0f) {
      q = a * rcp32(den[k]);
      if (!(q < 1.0f)) q = a < den[k] ? a / den[k] : 1.0f;
    }
    th[k] = q;
  }
  if (SCHEME == SCH_BMAX || SCHEME == SCH_BMIN) {
    float t = th[0];
    for (int k = 1; k < 4; ++k) {
      bool better = SCHEME == SCH_BMAX ? th[k] > t : th[k] < t;
      t = better ? th[k] : t;
    }
    for (int k = 0; k < 4; ++k) th[k] = t;
  }
}

// The loads of one triangle.
struct TriIn32 {
  int32_t iv[3], ip[3];
  uint32_t rk;
  double2 p[3];
  F4 Z[3];
  double sig[3];
};

__host__ __device__ inline void tri32_load_ids(int64_t t, const Dev& d, TriIn32& in) {
  const int64_t nt = d.nt;
  for (int i = 0; i < 3; ++i) in.iv[i] = d.tv[i * nt + t];
  in.rk = d.rk[t];
}

template <bool CFL>
__host__ __device__ inline void tri32_load_verts(const Dev& d, const Dev32& h, TriIn32& in) {
  const F4* Zp = h.Zf;
  for (int i = 0; i < 3; ++i) {
    in.p[i] = d.xy[in.iv[i]];
    in.Z[i] = Zp[in.iv[i]];
    if (CFL) in.sig[i] = d.sig[in.iv[i]];
    in.ip[i] = corner_slot(d, in.iv[i], in.rk, i);
  }
}

// What a triangle reads beside them, and where its results go (the tiled form
// has an LDS-staged one).
struct TriIO32 {
  const Dev& d;
  const Dev32& h;
  const int32_t* iv;
  const int32_t* ip;
  __host__ __device__ float idt(int64_t t) const { return (float)(1.0 / d.dt[d.tmesh ? d.tmesh[t] : 0]); }
  __host__ __device__ const double* vr(int64_t t) const { return d.vr + 3 * (d.tmesh ? d.tmesh[t] : 0); }
  __host__ __device__ F4 dw(int i) const { return h.dW[iv[i]]; }
  __host__ __device__ void part(int i, const float out[4]) const {
    plane_store<float, false>(h.C, d.ns, ip[i], 0, out);
  }
  __host__ __device__ void cfl(int64_t t, double x) const { reinterpret_cast<float*>(d.lam)[t] = (float)x; }
};

// One triangle, stage 1 (STAGE = 1) or stage 2 (STAGE = 2) of Section 3.4.
// Stage 1 writes the scheme's parts phi_i to C and, when SAVE, keeps phi^N_i
// and phi^T for stage 2. Stage 2 forms the total residuals
//   Phi^N_i = |T|/3 (W*_i - W^n_i)/dt + (phi^N_i(n) + phi^N_i(*))/2,
//   Phi^T   = |T|/3 sum_j (W*_j - W^n_j)/dt + (phi^T(n) + phi^T(*))/2,
//   Phi^LDA_i = K_i^+(*) A(*)^{-1} Phi^T,
// blends them and writes them to C.
// LUMP (stage 2 only): selective lumping of Section 3.4 instead of global lumping.
template <int SCHEME, int STAGE, bool SAVE, bool CFL, bool LUMP, class IO>
__host__ __device__ inline void tri32_compute(int64_t t, const TriIn32& in, const Dev& d, const Dev32& h,
                                              const IO& io) {
  using R = float;
  const double2 p0 = in.p[0], p1 = in.p[1], p2 = in.p[2];
  const double d1x = unwrap_select(p1.x - p0.x, d.px, d.hpx), d1y = unwrap_select(p1.y - p0.y, d.py, d.hpy);
  const double d2x = unwrap_select(p2.x - p0.x, d.px, d.hpx), d2y = unwrap_select(p2.y - p0.y, d.py, d.hpy);
  // inward normals scaled by edge length: rotate the opposite edge by +90 degrees
  const double nxd[3] = {-(d2y - d1y), d2y, -d1y};
  const double nyd[3] = {d2x - d1x, -d2x, d1x};

  const F4* Zc = in.Z;

  // Bx blend coefficient (Section 3.3.3): theta = min(1, s^2 h / L) with the
  // shock sensor s = (-L div v / (|v|max - |v|min))^+, div v that of the
  // linear interpolant of the corner velocities (u = Z_1 / Z_0, v = Z_2 / Z_0),
  // h = sqrt(2 |T|); |v|min, |v|max (at this stage's state) and the domain
  // size L of the triangle's mesh come from d.vr.
  R bx = R(0);
  if (SCHEME == SCH_BX) {
    const double* r = io.vr(t);
    R div = R(0);
    for (int i = 0; i < 3; ++i) div = div + (Zc[i].v[1] * (R)nxd[i] + Zc[i].v[2] * (R)nyd[i]) / Zc[i].v[0];
    const double a2 = d1x * d2y - d1y * d2x;  // 2 |T|
    const R range = (R)(r[1] - r[0]), L = (R)r[2];
    const R sn = range > R(0) ? rmax(-(L * div) / ((R)a2 * range), R(0)) : R(0);
    bx = rmin(sn * sn * (R)sqrt(a2) / L, R(1));
  }

  const R gam = (R)d.gamma;
  Roe<R> q;
  q.g1 = gam - R(1);
  const R third = R(1) / R(3);
  R zb[4];
  for (int k = 0; k < 4; ++k) zb[k] = (Zc[0].v[k] + Zc[1].v[k] + Zc[2].v[k]) * third;
  const R iz = rcp32(zb[0]);
  q.u = zb[1] * iz;
  q.v = zb[2] * iz;
  q.h = zb[3] * iz;
  const R q2 = q.u * q.u + q.v * q.v;
  len_rcp32(q.g1 * (q.h - R(0.5) * q2), q.c, q.ic);
  q.ac = R(0.5) * q.g1 * q2 * q.ic;
  q.uc = q.u * q.ic;
  q.vc = q.v * q.ic;

  // dW_i = M(Zbar)(Z_i - Z_0), M = dW/dZ
  R dWh[3][4];
  const R igam = (R)d.igamma;
  for (int k = 0; k < 4; ++k) dWh[0][k] = R(0);
  for (int i = 1; i < 3; ++i) {
    R dz[4];
    for (int k = 0; k < 4; ++k) dz[k] = Zc[i].v[k] - Zc[0].v[k];
    dWh[i][0] = R(2) * zb[0] * dz[0];
    dWh[i][1] = zb[1] * dz[0] + zb[0] * dz[1];
    dWh[i][2] = zb[2] * dz[0] + zb[0] * dz[2];
    dWh[i][3] = (zb[3] * dz[0] + q.g1 * (zb[1] * dz[1] + zb[2] * dz[2]) + zb[0] * dz[3]) * igam;
  }

  Corner<R> kc[3];
  const R hic = R(0.5) * q.ic;
  R lmax = R(0);
  for (int i = 0; i < 3; ++i) {
    // edge geometry in the algebra's precision, from FP64 coordinate differences
    const R ex = (R)nxd[i], ey = (R)nyd[i];
    R L, iL;
    len_rcp32(ex * ex + ey * ey, L, iL);
    lmax = rmax(lmax, L);
    Corner<R>& k = kc[i];
    k.nx = ex * iL;
    k.ny = ey * iL;
    k.s = R(0.5) * L;
    k.w = q.u * k.nx + q.v * k.ny;
    const R l1 = k.w + q.c, l2 = k.w - q.c, l3 = k.w;
    const R p1 = rmax(l1, R(0)), p2 = rmax(l2, R(0)), p3 = rmax(l3, R(0));
    const R m1 = rmin(l1, R(0)), m2 = rmin(l2, R(0)), m3 = rmin(l3, R(0));
    const R sh = k.s * hic;
    k.l3p = k.s * p3;
    k.h1p = sh * (p1 - p3);
    k.h2p = sh * (p2 - p3);
    k.l3m = k.s * m3;
    k.h1m = sh * (m1 - m3);
    k.h2m = sh * (m2 - m3);
  }

  if (CFL) {
    // CFL limit of Section 3.2: l_max^T max_j(|v_j| + c_j) of the triangle
    double lam = 0.0;
    for (int i = 0; i < 3; ++i) lam = rmax(lam, in.sig[i]);
    io.cfl(t, (double)lmax * lam);
  }

  // triangle residual and the N right-hand side
  R phiT[4], bN[4], t1[4], t2[4];
  apply_full(q, kc[1], dWh[1], t1);
  apply_full(q, kc[2], dWh[2], t2);
  for (int k = 0; k < 4; ++k) phiT[k] = t1[k] + t2[k];
  R A[4][4];
  build_A(q, kc, A);

  constexpr bool needN = SCHEME != SCH_LDA;
  constexpr bool needL = SCHEME != SCH_N;
  R pN[3][4];
  R rhs1[4];
  R mass = R(0), idt = R(0);
  if (needN) {
    apply_split(q, kc[1], kc[1].l3m, kc[1].h1m, kc[1].h2m, dWh[1], t1);
    apply_split(q, kc[2], kc[2].l3m, kc[2].h1m, kc[2].h2m, dWh[2], t2);
    for (int k = 0; k < 4; ++k) bN[k] = t1[k] + t2[k];
  } else {
    for (int k = 0; k < 4; ++k) bN[k] = R(0);
  }
  if (STAGE == 1) {
    for (int k = 0; k < 4; ++k) rhs1[k] = phiT[k];
  } else {
    idt = io.idt(t);
    mass = (R)((0.5 * (d1x * d2y - d1y * d2x)) * (1.0 / 3.0));
    if (needL) {
      R srate[4] = {R(0), R(0), R(0), R(0)};
      for (int i = 0; i < 3; ++i) {
        const Q4<R> dwv = io.dw(i);
        for (int k = 0; k < 4; ++k) srate[k] = srate[k] + dwv.v[k] * idt;
      }
      const Q4<R> kt = keep_load<R>(h.keepT, d.nt, t, 0);
      for (int k = 0; k < 4; ++k) rhs1[k] = mass * srate[k] + R(0.5) * (kt.v[k] + phiT[k]);
    } else {
      for (int k = 0; k < 4; ++k) rhs1[k] = R(0);
    }
  }
  R xN[4], xL[4], b0[4], b1[4];
  for (int k = 0; k < 4; ++k) {
    b0[k] = bN[k];
    b1[k] = rhs1[k];
  }
  solve2(A, b0, b1, xN, xL);
  // Corner parts. The parts of a distribution sum to the residual they
  // split (sum_i K_i^+ = A): sum_i K_i^+ (dW_i + xN) = phi^T and
  // sum_i K_i^+ xL = rhs1, so corner 2's parts are the residual minus those
  // of corners 0 and 1 (exact in exact arithmetic; saves two K^+ products).
  R pl[3][4];
  if (needL) {
    apply_split(q, kc[0], kc[0].l3p, kc[0].h1p, kc[0].h2p, xL, pl[0]);
    apply_split(q, kc[1], kc[1].l3p, kc[1].h1p, kc[1].h2p, xL, pl[1]);
    for (int k = 0; k < 4; ++k) pl[2][k] = rhs1[k] - pl[0][k] - pl[1][k];
  }
  // Selective lumping (Section 3.4, stage 2): the N and LDA total parts both
  // get sum_j (|T| delta_ij / 3 - m^G_ij) (W*_j - W^n_j) / dt with the
  // Galerkin mass m^G_ij = |T| (1 + delta_ij) / 12, that is
  // (|T| / 12) (3 r_i - r_0 - r_1 - r_2) with r = (W* - W^n) / dt.
  R sl[3][4];
  if (STAGE == 2 && LUMP) {
    R rs[4] = {R(0), R(0), R(0), R(0)};
    for (int i = 0; i < 3; ++i) {
      const Q4<R> dwv = io.dw(i);
      for (int k = 0; k < 4; ++k) {
        sl[i][k] = dwv.v[k] * idt;
        rs[k] = rs[k] + sl[i][k];
      }
    }
    const R m12 = mass * R(0.25);
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < 4; ++k) sl[i][k] = m12 * (R(3) * sl[i][k] - rs[k]);
    if (needL)
      for (int i = 0; i < 3; ++i)
        for (int k = 0; k < 4; ++k) pl[i][k] = pl[i][k] + sl[i][k];
  }
  R den[4] = {R(0), R(0), R(0), R(0)};
  if (needN) {
    for (int i = 0; i < 2; ++i) {
      R y[4];
      for (int k = 0; k < 4; ++k) y[k] = dWh[i][k] + xN[k];
      apply_split(q, kc[i], kc[i].l3p, kc[i].h1p, kc[i].h2p, y, pN[i]);
    }
    for (int k = 0; k < 4; ++k) pN[2][k] = phiT[k] - pN[0][k] - pN[1][k];
    // Only corners 0 and 1 of the N parts are kept: corner 2's is phi^T minus
    // those two, and stage 2 forms it again from the kept phi^T with the same
    // two subtractions, which gives back the identical value.
    if (STAGE == 1 && SAVE) {
      keep_store<R>(h.keepN, d.nt, t, 0, pN[0]);
      keep_store<R>(h.keepN, d.nt, t, 1, pN[1]);
    }
    if (STAGE == 2) {
      // Phi^N_i = |T|/3 (W*_i - W^n_i)/dt + (phi^N_i(n) + phi^N_i(*))/2; the
      // kept parts and per-vertex differences are loaded here (cached) to
      // keep them out of registers across the solve
      const Q4<R> k0 = keep_load<R>(h.keepN, d.nt, t, 0), k1 = keep_load<R>(h.keepN, d.nt, t, 1),
                  kt = keep_load<R>(h.keepT, d.nt, t, 0);
      R kn[3][4];
      for (int k = 0; k < 4; ++k) {
        kn[0][k] = k0.v[k];
        kn[1][k] = k1.v[k];
        kn[2][k] = kt.v[k] - k0.v[k] - k1.v[k];
      }
      for (int i = 0; i < 3; ++i) {
        const Q4<R> dwv = io.dw(i);
        for (int k = 0; k < 4; ++k) pN[i][k] = mass * (dwv.v[k] * idt) + R(0.5) * (kn[i][k] + pN[i][k]);
      }
      if (LUMP)
        for (int i = 0; i < 3; ++i)
          for (int k = 0; k < 4; ++k) pN[i][k] = pN[i][k] + sl[i][k];
    }
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < 4; ++k) den[k] = den[k] + (R)fabs(pN[i][k]);
  }
  if (STAGE == 1 && SAVE) keep_store<R>(h.keepT, d.nt, t, 0, phiT);
  // rhs1 is the residual being split (phi^T or Phi^T)
  R th[4] = {R(0), R(0), R(0), R(0)};
  if (SCHEME >= SCH_B && SCHEME <= SCH_BMIN) blend_theta32<SCHEME>(rhs1, den, th);
  if (SCHEME == SCH_BX)
    for (int k = 0; k < 4; ++k) th[k] = bx;
  for (int i = 0; i < 3; ++i) {
    R out[4];
    for (int k = 0; k < 4; ++k) {
      if (SCHEME == SCH_N) out[k] = pN[i][k];
      else if (SCHEME == SCH_LDA) out[k] = pl[i][k];
      else out[k] = pl[i][k] + th[k] * (pN[i][k] - pl[i][k]);
    }
    io.part(i, out);
  }
}

template <int SCHEME, int STAGE, bool SAVE, bool CFL, bool LUMP>
__host__ __device__ inline void tri32_body(int64_t t, const Dev& d, const Dev32& h) {
  TriIn32 in;
  tri32_load_ids(t, d, in);
  tri32_load_verts<CFL>(d, h, in);
  const TriIO32 io{d, h, in.iv, in.ip};
  tri32_compute<SCHEME, STAGE, SAVE, CFL, LUMP>(t, in, d, h, io);
}

// Sum of a vertex's n parts get(0), ..., get(n-1) in that order, in FP64,
// Neumaier-compensated.
template <class Get>
__host__ __device__ inline void sum_parts32(int32_t n, const Get& get, double acc[4]) {
  double cmp[4] = {0.0, 0.0, 0.0, 0.0};
  for (int k = 0; k < 4; ++k) acc[k] = 0.0;
  for_loaded(n, get, [&](int32_t, const F4& c) {
    for (int k = 0; k < 4; ++k) {
      const double x = (double)c.v[k];
      const double tsum = acc[k] + x;
      cmp[k] += fabs(acc[k]) >= fabs(x) ? (acc[k] - tsum) + x : (x - tsum) + acc[k];
      acc[k] = tsum;
    }
  });
  for (int k = 0; k < 4; ++k) acc[k] = acc[k] + cmp[k];
}

__host__ __device__ inline F4 zf_of(const VertexDerived& o) {
  F4 q;
  for (int k = 0; k < 4; ++k) q.v[k] = (float)o.z[k];
  return q;
}

// Parameter vector of vertex v at the state w; with_sig: also |v| + c (the CFL
// limit reads it at the start of a step; the first-stage state does not need it).
__host__ __device__ inline void vertex_epilogue32(const Dev& d, const Dev32& h, int64_t v, const double w[4],
                                                  bool with_sig) {
  const VertexDerived o = derive(d.gamma, w);
  h.Zf[v] = zf_of(o);
  if (with_sig) d.sig[v] = o.sig;
  if (!o.ok) d.flag[d.vmesh ? d.vmesh[v] : 0] = 1;
}

// One vertex of the vertex pass (MODE: G_EULER, G_STAGE1, G_STAGE2).
template <int MODE>
__host__ __device__ inline void gather32_body(int64_t v, const Dev& d, const Dev32& h) {
  D4* W = d.W;
  const int32_t code = d.bc ? d.bc[v] : -1;
  const int32_t b = is_ghost(code) ? -1 : wall_index(code);
  if (is_ghost(code)) {
    if (MODE == G_STAGE1) {
      d.Ws[v] = W[v];
      h.dW[v] = F4{{0.0f, 0.0f, 0.0f, 0.0f}};
    }
    return;
  }
  double acc[4];
  const int32_t deg = d.row[v + 1] - d.row[v];
  const int64_t s0 = vslot(d, v);
  sum_parts32(deg, [&](int32_t j) { return plane_load<float>(h.C, d.ns, s0 + 64 * (int64_t)j, 0); }, acc);
  if (b >= 0) {
    const D4 wn = d.WCn[b];
    if (MODE == G_STAGE2) {
      const D4 ws = d.WCs[b];
      for (int k = 0; k < 4; ++k) acc[k] = acc[k] + 0.5 * (wn.v[k] + ws.v[k]);
    } else {
      for (int k = 0; k < 4; ++k) acc[k] = acc[k] + wn.v[k];
    }
  }
  const int m = d.vmesh ? d.vmesh[v] : 0;
  const double f = d.dt[m] / d.V[v];
  const D4 win = MODE == G_STAGE2 ? d.Ws[v] : W[v];
  double wo[4];
  vertex_update(win.v, f, acc, wo);
  if (MODE == G_STAGE1) {
    st4<double>(d.Ws, v, wo);
    float dw[4];
    for (int k = 0; k < 4; ++k) dw[k] = (float)(wo[k] - win.v[k]);
    st4<float>(h.dW, v, dw);
  } else {
    st4<double>(W, v, wo);
  }
  vertex_epilogue32(d, h, v, wo, MODE != G_STAGE1);
}

}  // namespace rd
