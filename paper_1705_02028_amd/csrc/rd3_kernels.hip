// gfx950 kernels of the three-dimensional path (bodies in rd3_device.h): a
// tile pass over the tetrahedra and a pass over the vertices per stage, and
// the CFL limit. No float atomics: every sum has a fixed order. The time step
// is read on the device.
//
// A workgroup takes a tile of at most 256 tetrahedra cut compactly out of the
// mesh (rd3_tiling.h), one a thread. Its ~100 vertices go through LDS once;
// the parts are summed per vertex inside the tile, in LDS, and only these
// partial sums (about 0.35 of one per tetrahedron instead of 4 parts) reach
// HBM, one record for every tile a vertex lies in, which the vertex pass adds
// in tile order. Normals come from the vertices' positions and stage 2 works
// out the stage-1 N parts again from W^n: both cost less time than reading
// what they replace (96 and 160 bytes a tetrahedron).
//
// Measured on the 64^3 periodic box (1.57 M tetrahedra), B scheme: the tile
// passes take 82 us (stage 1) and 115 us (stage 2), where one thread per
// tetrahedron with a pivoted 5x5 elimination and every part through HBM took
// 233 and 304 us; a vertex pass 19 against 65 us, the CFL limit 15 against
// 61 us, a step 0.233 against 0.711 ms. The tile passes are bound by FP64
// instructions (about 1000 and 1600 a tetrahedron: 44 and 70 us if every
// cycle issued one) at two to three waves per SIMD. Tiles of 128 or 64
// tetrahedra: 0.243 and 0.255 ms a step. Three waves for stage 2 (168
// registers, 100 bytes spilled): 129 us.
#include "rd3_launch.h"

namespace rd3 {

// As rd::xcd_block: each XCD takes one contiguous range of tiles.
__device__ __forceinline__ int64_t xcd_tile() {
  const int64_t b = blockIdx.x, nb = gridDim.x;
  const int64_t x = b % 8, q = nb / 8, r = nb % 8;
  return x * q + (x < r ? x : r) + b / 8;
}

__global__ __launch_bounds__(kBlock) void k3_set(Dev3 d, const double* src) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v >= d.nv) return;
  const int64_t i = d.inv[v];
  double w[5], z[5], sg;
  for (int k = 0; k < 5; ++k) w[k] = src[k * d.nv + v];
  if (!to_z(w, d.gamma, z, sg)) d.flag[0] = 1;
  for (int k = 0; k < 5; ++k) d.W[k * d.nv + i] = w[k];
  d.r1[5 * i] = make_double2(z[0], z[1]);
  d.r1[5 * i + 1] = make_double2(z[2], z[3]);
  d.r1[5 * i + 2] = make_double2(z[4], sg);
}

__global__ __launch_bounds__(kBlock) void k3_get(Dev3 d, double* dst) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v >= d.nv) return;
  const int64_t i = d.inv[v];
  for (int k = 0; k < 5; ++k) dst[k * d.nv + v] = d.W[k * d.nv + i];
}

// STAGE 1, 2, or 0 (CFL terms alone).
template <int STAGE, int SCHEME, bool CFL>
__global__ __launch_bounds__(kBlock, 2) void k3_tile(Dev3 d) {
  extern __shared__ double2 lds[];
  const Tile3 T = d.tile[xcd_tile()];
  const int tid = threadIdx.x, nthr = blockDim.x, lvn = d.max_lv;
  double2* A = lds;            // [5][max_lv]
  double2* B = lds + 5 * lvn;  // [5][max_lv], stage 2
  for (int i = tid; i < 5 * T.nlv; i += nthr) {
    const int l = i / 5, c = i - 5 * l;
    const int64_t v = d.lv[T.l0 + l];
    A[c * lvn + l] = d.r1[5 * v + c];
    if (STAGE == 2) B[c * lvn + l] = d.r2[5 * v + c];
  }
  int32_t* jb = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(lds) + d.jb_at);
  for (int i = tid; i < T.nj; i += nthr) jb[i] = d.jb[T.j0 + i];
  __syncthreads();
  constexpr bool needN = SCHEME != S_LDA, needL = SCHEME != S_N;
  constexpr int NC = STAGE == 0 ? 1 : (CFL ? 6 : 5), K0 = STAGE == 0 ? 5 : 0;
  double out[4][5], term = 0.0;
  uint32_t sl[4];
  const bool mine = tid < T.nt;
  if (mine) {
    const uint4 q = d.tet[T.t0 + tid];
    const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
    int c[4];
    for (int i = 0; i < 4; ++i) {
      c[i] = w4[i] & 0xffff;
      sl[i] = w4[i] >> 16;
    }
    double p[3][3];
    {
      double x0[3];
      for (int i = 0; i < 4; ++i) {
        const double2 a = A[3 * lvn + c[i]], b = A[4 * lvn + c[i]];
        const double x[3] = {a.x, a.y, b.x};
        for (int k = 0; k < 3; ++k) {
          if (i == 0) x0[k] = x[k];
          else {
            const double dx = x[k] - x0[k], hi = dx - d.per[k], lo = dx + d.per[k];
            p[i - 1][k] = dx > d.half[k] ? hi : (dx < -d.half[k] ? lo : dx);
          }
        }
      }
    }
    double N[4][3];
    for (int k = 0; k < 3; ++k) {
      const int a = (k + 1) % 3, b = (k + 2) % 3;
      N[1][k] = p[1][a] * p[2][b] - p[1][b] * p[2][a];
      N[2][k] = p[2][a] * p[0][b] - p[2][b] * p[0][a];
      N[3][k] = p[0][a] * p[1][b] - p[0][b] * p[1][a];
      N[0][k] = -(N[1][k] + N[2][k] + N[3][k]);
    }
    if (CFL) {  // S_T lambda_T: the largest face area times the largest |u| + c
      double e2 = 0.0, lam = 0.0;
      for (int i = 0; i < 4; ++i) {
        e2 = rmax(e2, N[i][0] * N[i][0] + N[i][1] * N[i][1] + N[i][2] * N[i][2]);
        lam = rmax(lam, A[2 * lvn + c[i]].y);
      }
      double L, iL;
      len_rcp(e2, L, iL);
      term = 0.5 * L * lam;
    }
    auto zn = [&](int i, double z[5]) {
      const double2 a = A[c[i]], b = A[lvn + c[i]], e = A[2 * lvn + c[i]];
      z[0] = a.x; z[1] = a.y; z[2] = b.x; z[3] = b.y; z[4] = e.x;
    };
    double kN[3][5], res[5], xT[5];
    if (STAGE == 1) {
      Tet s;
      tet_eval<needN>(d, zn, N, s);
      to_conserved(s.f, s.phi, res);
      if (needN)
        for (int i = 0; i < 3; ++i) n_part(s, i, kN[i]);
      if (needL) solve(s.q, s.phi, xT);
      scheme_parts<SCHEME>(s, res, kN, xT, out);
    }
    if (STAGE == 2) {
      {
        Tet s;
        tet_eval<needN>(d, zn, N, s);
        to_conserved(s.f, s.phi, res);
        if (needN)
          for (int i = 0; i < 3; ++i) n_part(s, i, kN[i]);
      }
      fence();
      // the mass |T| / 4 times the first-stage rate of each corner
      const double m4 = 4.0 * (p[0][0] * N[1][0] + p[0][1] * N[1][1] + p[0][2] * N[1][2]);
      for (int i = 0; i < 4; ++i) {
        const double2 a = B[2 * lvn + c[i]], b = B[3 * lvn + c[i]], e = B[4 * lvn + c[i]];
        const double r[5] = {a.y, b.x, b.y, e.x, e.y};
        for (int k = 0; k < 5; ++k) {
          res[k] += m4 * r[k];
          if (needN && i < 3) kN[i][k] += m4 * r[k];
        }
      }
      fence();
      auto zs = [&](int i, double z[5]) {
        const double2 a = B[c[i]], b = B[lvn + c[i]], e = B[2 * lvn + c[i]];
        z[0] = a.x; z[1] = a.y; z[2] = b.x; z[3] = b.y; z[4] = e.x;
      };
      Tet s;
      tet_eval<needN>(d, zs, N, s);
      double x[5];
      to_conserved(s.f, s.phi, x);
      for (int k = 0; k < 5; ++k) res[k] += x[k];
      if (needN)
        for (int i = 0; i < 3; ++i) {
          n_part(s, i, x);
          for (int k = 0; k < 5; ++k) kN[i][k] += x[k];
        }
      if (needL) {
        from_conserved(s.f, res, x);
        solve(s.q, x, xT);
      }
      scheme_parts<SCHEME>(s, res, kN, xT, out);
    }
  }
  __syncthreads();
  // the parts over the vertex records
  double* P = reinterpret_cast<double*>(lds);
  const int ps = part_plane(d.max_tet);
  if (mine)
    for (int i = 0; i < 4; ++i) {
      if (STAGE != 0)
        for (int k = 0; k < 5; ++k) P[k * ps + sl[i]] = out[i][k];
      if (CFL) P[(NC - 1) * ps + sl[i]] = term;
    }
  __syncthreads();
  // four parts of a sum are loaded before the first is added
  for (int i = tid; i < NC * T.nlv; i += nthr) {
    const int l = i / NC, k = i - NC * l;
    const int n = d.deg[T.l0 + l];
    const double* q = P + k * ps + l;
    double acc = 0.0;
    for (int j0 = 0; j0 < n; j0 += 4) {
      double x[4];
      for (int u = 0; u < 4; ++u) x[u] = q[jb[j0 + u < n ? j0 + u : n - 1]];
      for (int u = 0; u < 4; ++u) acc = j0 + u < n ? acc + x[u] : acc;
    }
    if (K0 + k < 5) acc *= STAGE == 1 ? kScale1 : kScale2;
    d.rec[6 * (int64_t)d.rpos[T.l0 + l] + K0 + k] = acc;
  }
}

// mode 0: Euler (W <- W - dt/V R, then Z, sig of W); 1: first stage
// (Ws <- W - dt/V R, then Z of Ws and the rate); 2: second stage
// (W <- Ws - dt/V R, then Z, sig of W).
template <int MODE>
__global__ __launch_bounds__(kBlock) void k3_gather(Dev3 d) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v >= d.nv) return;
  const int64_t nv = d.nv;
  double r[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int32_t q = d.rbeg[v]; q < d.rbeg[v + 1]; ++q) {
    const double2* x = reinterpret_cast<const double2*>(d.rec + 6 * (int64_t)q);
    const double2 a = x[0], b = x[1];
    const double e = d.rec[6 * (int64_t)q + 4];
    r[0] += a.x;
    r[1] += a.y;
    r[2] += b.x;
    r[3] += b.y;
    r[4] += e;
  }
  const double dt = *d.dt, f = dt / d.V[v];
  const double* src = MODE == 2 ? d.Ws : d.W;
  double* dst = MODE == 1 ? d.Ws : d.W;
  double w[5], rate[5], z[5], sg;
  const double idt = 1.0 / dt;
  for (int k = 0; k < 5; ++k) {
    const double old = src[k * nv + v];
    w[k] = old - f * r[k];
    dst[k * nv + v] = w[k];
    rate[k] = (w[k] - old) * idt;
  }
  if (!to_z(w, d.gamma, z, sg)) d.flag[0] = 1;
  double2* o = (MODE == 1 ? d.r2 : d.r1) + 5 * v;
  o[0] = make_double2(z[0], z[1]);
  o[1] = make_double2(z[2], z[3]);
  if (MODE != 1) {
    o[2] = make_double2(z[4], sg);
  } else {
    o[2] = make_double2(z[4], rate[0]);
    o[3] = make_double2(rate[1], rate[2]);
    o[4] = make_double2(rate[3], rate[4]);
  }
}

// Per vertex 3 V / sum of its CFL terms; block minima.
__global__ __launch_bounds__(kBlock) void k3_cfl_vertex(Dev3 d) {
  __shared__ double red[kBlock];
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double best = INFINITY;
  if (v < d.nv) {
    double acc = 0.0;
    for (int32_t q = d.rbeg[v]; q < d.rbeg[v + 1]; ++q) acc += d.rec[6 * (int64_t)q + 5];
    best = 3.0 * d.V[v] / acc;
  }
  red[threadIdx.x] = best;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) d.bmin[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(kBlock) void k3_cfl_final(Dev3 d, int nblocks, double cfl) {
  __shared__ double red[kBlock];
  double best = INFINITY;
  for (int b = threadIdx.x; b < nblocks; b += kBlock) best = fmin(best, d.bmin[b]);
  red[threadIdx.x] = best;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *d.dt = cfl * red[0];
}

__global__ void k3_set_dt(double* p, double v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

static unsigned blocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

void tile3_lds(Dev3& d, int32_t max_jd) {
  const size_t vert = sizeof(double2) * 10 * (size_t)d.max_lv;
  const size_t parts = sizeof(double) * 6 * (size_t)part_plane(d.max_tet);
  d.jb_at = (int32_t)((vert > parts ? vert : parts) + 15) & ~15;
  d.lds = d.jb_at + (int32_t)sizeof(int32_t) * max_jd;
}

hipError_t launch3_set(const Dev3& d, const double* src, hipStream_t s) {
  hipLaunchKernelGGL(k3_set, dim3(blocks(d.nv)), dim3(kBlock), 0, s, d, src);
  return hipGetLastError();
}

hipError_t launch3_get(const Dev3& d, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k3_get, dim3(blocks(d.nv)), dim3(kBlock), 0, s, d, dst);
  return hipGetLastError();
}

template <int SCHEME>
static void tile_launch(const Dev3& d, int stage, bool cfl, hipStream_t s) {
  const dim3 g(d.ntiles), b(d.threads);
  const size_t lds = d.lds;
  if (stage == 2) hipLaunchKernelGGL((k3_tile<2, SCHEME, false>), g, b, lds, s, d);
  else if (cfl) hipLaunchKernelGGL((k3_tile<1, SCHEME, true>), g, b, lds, s, d);
  else hipLaunchKernelGGL((k3_tile<1, SCHEME, false>), g, b, lds, s, d);
}

hipError_t launch3_tile(const Dev3& d, int stage, int scheme, bool cfl, hipStream_t s) {
  if (stage == 0) {
    hipLaunchKernelGGL((k3_tile<0, S_N, true>), dim3(d.ntiles), dim3(d.threads), d.lds, s, d);
    return hipGetLastError();
  }
  switch (scheme) {
    case S_N: tile_launch<S_N>(d, stage, cfl, s); break;
    case S_LDA: tile_launch<S_LDA>(d, stage, cfl, s); break;
    case S_B: tile_launch<S_B>(d, stage, cfl, s); break;
    case S_BMAX: tile_launch<S_BMAX>(d, stage, cfl, s); break;
    case S_BMIN: tile_launch<S_BMIN>(d, stage, cfl, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch3_gather(const Dev3& d, int mode, hipStream_t s) {
  if (mode == 0)
    hipLaunchKernelGGL(k3_gather<0>, dim3(blocks(d.nv)), dim3(kBlock), 0, s, d);
  else if (mode == 1)
    hipLaunchKernelGGL(k3_gather<1>, dim3(blocks(d.nv)), dim3(kBlock), 0, s, d);
  else
    hipLaunchKernelGGL(k3_gather<2>, dim3(blocks(d.nv)), dim3(kBlock), 0, s, d);
  return hipGetLastError();
}

int cfl_blocks(int64_t nv) { return (int)blocks(nv); }

hipError_t launch3_cfl(const Dev3& d, double cfl, hipStream_t s) {
  hipLaunchKernelGGL(k3_cfl_vertex, dim3(blocks(d.nv)), dim3(kBlock), 0, s, d);
  hipLaunchKernelGGL(k3_cfl_final, dim3(1), dim3(kBlock), 0, s, d, (int)blocks(d.nv), cfl);
  return hipGetLastError();
}

hipError_t launch3_set_dt(const Dev3& d, double dt, hipStream_t s) {
  hipLaunchKernelGGL(k3_set_dt, dim3(1), dim3(64), 0, s, d.dt, dt);
  return hipGetLastError();
}

}  // namespace rd3
