// gfx950 kernels of the step with FP32 distribution (bodies in rd_fp32.h): one
// thread per triangle or per vertex, 256-thread workgroups.
#include "rd_fp32.h"
#include "rd_fp32_launch.h"
#include "rd_kcommon.h"

namespace rd {

// At least four waves per SIMD (at most 128 VGPRs; the instances use 75-113).
template <int SCHEME, int STAGE, bool SAVE, bool CFL, bool LUMP>
__global__ __launch_bounds__(kBlock, 4) void k_tri32(Dev d, Dev32 h) {
  const int64_t t = xcd_block() * kBlock + threadIdx.x;
  if (t < d.nt) tri32_body<SCHEME, STAGE, SAVE, CFL, LUMP>(t, d, h);
}

template <int MODE>
__global__ __launch_bounds__(kBlock) void k_gather32(Dev d, Dev32 h) {
  const int64_t v = xcd_block() * kBlock + threadIdx.x;
  if (v < d.nv) gather32_body<MODE>(v, d, h);
}

// Moves a state in a patch buffer to the FP32 form (d.W), with its Zf and
// |v| + c; nothing where the state is there already.
__global__ __launch_bounds__(kBlock) void k_enter32(Dev d, Dev32 h, State st) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v >= d.nv || *st.cur == kForm32) return;
  const D4 w = *st.at(v);
  d.W[v] = w;
  vertex_epilogue32(d, h, v, w.v, true);
}

// The state from the caller's [4][nv] arrays, as k_patch_set, with its Zf and |v| + c.
__global__ __launch_bounds__(kBlock) void k_set32(Dev d, Dev32 h, int* cur, const double* soa, const int* bad) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (bad && *bad < d.nv) return;
  if (v == 0) cur[0] = kForm32;
  if (v >= d.nv) return;
  const double w[4] = {soa[v], soa[d.nv + v], soa[2 * d.nv + v], soa[3 * d.nv + v]};
  st4<double>(d.W, v, w);
  vertex_epilogue32(d, h, v, w, true);
}

// Per-vertex CFL bounds 2 V_i / sum l_max lambda_max (summed over the terms of
// the vertex's triangles) and their block minima.
__global__ __launch_bounds__(kBlock) void k_cfl_vertex(Dev d, CflPlan p) {
  constexpr int U = kCflSpan / kBlock;
  const int b = blockIdx.x;
  double x = INFINITY;
  int64_t v[U];
  bool in[U];
  for (int u = 0; u < U; ++u) {
    v[u] = (int64_t)p.blk_v0[b] + u * kBlock + threadIdx.x;
    in[u] = v[u] < p.blk_v1[b];
  }
  double bound[U];
  cfl_vertex_bounds<float, U>(v, in, p.blk_v0[b], d, bound);
  for (int u = 0; u < U; ++u)
    if (in[u]) x = rmin(x, bound[u]);
  const double m = block_min(x);
  if (threadIdx.x == 0) p.part[b] = m;
}

// Per-mesh minimum over the mesh's blocks -> dt.
__global__ __launch_bounds__(kBlock) void k_cfl_final(Dev d, CflPlan p, double cfl) {
  const int m = blockIdx.x;
  double x = INFINITY;
  for (int b = p.mesh_b0[m] + threadIdx.x; b < p.mesh_b0[m + 1]; b += kBlock) x = rmin(x, p.part[b]);
  x = block_min(x);
  if (threadIdx.x == 0) d.dt[m] = cfl * x;
}

// Smallest and largest flow speed |v| over each CFL block's vertices (the Bx
// sensor's range) at W^n or at W*, then per mesh.
template <bool STAR>
__global__ __launch_bounds__(kBlock) void k_vrange32(Dev d, CflPlan p) {
  const int b = blockIdx.x;
  double lo = INFINITY, hi = 0.0;
#pragma unroll
  for (int u = 0; u < kCflSpan / kBlock; ++u) {
    const int64_t v = (int64_t)p.blk_v0[b] + u * kBlock + threadIdx.x;
    if (v < p.blk_v1[b]) {
      const double sp = flow_speed((STAR ? d.Ws : d.W)[v]);
      lo = rmin(lo, sp);
      hi = rmax(hi, sp);
    }
  }
  lo = block_min(lo);
  __syncthreads();
  hi = -block_min(-hi);
  if (threadIdx.x == 0) {
    p.vpart[2 * b] = lo;
    p.vpart[2 * b + 1] = hi;
  }
}

__global__ __launch_bounds__(kBlock) void k_vrange32_final(Dev d, CflPlan p) {
  const int m = blockIdx.x;
  double lo = INFINITY, hi = 0.0;
  for (int b = p.mesh_b0[m] + threadIdx.x; b < p.mesh_b0[m + 1]; b += kBlock) {
    lo = rmin(lo, p.vpart[2 * b]);
    hi = rmax(hi, p.vpart[2 * b + 1]);
  }
  lo = block_min(lo);
  __syncthreads();
  hi = -block_min(-hi);
  if (threadIdx.x == 0) {
    d.vr[3 * m] = lo;
    d.vr[3 * m + 1] = hi;
  }
}

template <int SCHEME>
static hipError_t tri32_go(const Dev& d, const Dev32& h, int stage, bool save, bool cfl, hipStream_t s) {
  const dim3 g(nblk(d.nt)), b(kBlock);
  if (stage == 1 && save && cfl) hipLaunchKernelGGL((k_tri32<SCHEME, 1, true, true, false>), g, b, 0, s, d, h);
  else if (stage == 1 && save) hipLaunchKernelGGL((k_tri32<SCHEME, 1, true, false, false>), g, b, 0, s, d, h);
  else if (stage == 1 && cfl) hipLaunchKernelGGL((k_tri32<SCHEME, 1, false, true, false>), g, b, 0, s, d, h);
  else if (stage == 1) hipLaunchKernelGGL((k_tri32<SCHEME, 1, false, false, false>), g, b, 0, s, d, h);
  else if (h.slump) hipLaunchKernelGGL((k_tri32<SCHEME, 2, false, false, true>), g, b, 0, s, d, h);
  else hipLaunchKernelGGL((k_tri32<SCHEME, 2, false, false, false>), g, b, 0, s, d, h);
  return hipGetLastError();
}

hipError_t launch_tri32(const Dev& d, const Dev32& h, int scheme, int stage, bool save, bool cfl, hipStream_t s) {
  switch (scheme) {
    case SCH_N: return tri32_go<SCH_N>(d, h, stage, save, cfl, s);
    case SCH_LDA: return tri32_go<SCH_LDA>(d, h, stage, save, cfl, s);
    case SCH_B: return tri32_go<SCH_B>(d, h, stage, save, cfl, s);
    case SCH_BMAX: return tri32_go<SCH_BMAX>(d, h, stage, save, cfl, s);
    case SCH_BMIN: return tri32_go<SCH_BMIN>(d, h, stage, save, cfl, s);
    case SCH_BX: return tri32_go<SCH_BX>(d, h, stage, save, cfl, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gather32(const Dev& d, const Dev32& h, int mode, hipStream_t s) {
  const dim3 g(nblk(d.nv)), b(kBlock);
  switch (mode) {
    case G_EULER: hipLaunchKernelGGL(k_gather32<G_EULER>, g, b, 0, s, d, h); break;
    case G_STAGE1: hipLaunchKernelGGL(k_gather32<G_STAGE1>, g, b, 0, s, d, h); break;
    case G_STAGE2: hipLaunchKernelGGL(k_gather32<G_STAGE2>, g, b, 0, s, d, h); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_enter32(const Dev& d, const Dev32& h, const State& st, hipStream_t s) {
  hipLaunchKernelGGL(k_enter32, dim3(nblk(d.nv)), dim3(kBlock), 0, s, d, h, st);
  return hipGetLastError();
}

hipError_t launch_set32(const Dev& d, const Dev32& h, int* cur, const double* soa, const int* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_set32, dim3(nblk(d.nv)), dim3(kBlock), 0, s, d, h, cur, soa, bad);
  return hipGetLastError();
}

hipError_t launch_cfl32(const Dev& d, const CflPlan& p, double cfl, hipStream_t s) {
  hipLaunchKernelGGL(k_cfl_vertex, dim3(p.nblocks), dim3(kBlock), 0, s, d, p);
  return launch_cfl_final(d, p, cfl, s);
}

hipError_t launch_cfl_final(const Dev& d, const CflPlan& p, double cfl, hipStream_t s) {
  hipLaunchKernelGGL(k_cfl_final, dim3(p.nmesh), dim3(kBlock), 0, s, d, p, cfl);
  return hipGetLastError();
}

hipError_t launch_vrange32(const Dev& d, const CflPlan& p, bool star, hipStream_t s) {
  if (star) hipLaunchKernelGGL(k_vrange32<true>, dim3(p.nblocks), dim3(kBlock), 0, s, d, p);
  else hipLaunchKernelGGL(k_vrange32<false>, dim3(p.nblocks), dim3(kBlock), 0, s, d, p);
  return launch_vrange_final(d, p, s);
}

hipError_t launch_vrange_final(const Dev& d, const CflPlan& p, hipStream_t s) {
  hipLaunchKernelGGL(k_vrange32_final, dim3(p.nmesh), dim3(kBlock), 0, s, d, p);
  return hipGetLastError();
}

}  // namespace rd
