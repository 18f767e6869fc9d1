// gfx950 kernels of the tiled form of the FP32 step: one workgroup per triangle tile, the
// tile's vertex data staged in LDS (see rd_tiles.h for the phases), then a
// vertex pass over the shared vertices.
#include "rd_fp32_launch.h"
#include "rd_kcommon.h"

namespace rd {

template <int SCHEME, bool SAVE, bool CFL>
__global__ __launch_bounds__(kBlock, 4) void k_tile1(Dev d, Dev32 h, Tiles tl) {
  extern __shared__ D4 lds_raw[];
  const int64_t tile = xcd_block();
  TileLds L;
  tile_lds(tl, 1, CFL, reinterpret_cast<char*>(lds_raw), &L);
  const int32_t nthr = blockDim.x, tid = threadIdx.x;
  const int32_t nlv = tl.vbeg[tile + 1] - tl.vbeg[tile];
  for (int32_t l = tid; l < nlv; l += nthr) tile_load1<CFL>(tile, l, d, h, tl, L);
  __syncthreads();
  const int32_t ntri = tl.tbeg[tile + 1] - tl.tbeg[tile];
  for (int32_t j = tid; j < ntri; j += nthr) tile_tri<SCHEME, 1, SAVE, CFL>(tile, j, d, h, tl, L);
  __syncthreads();
  const int32_t nvi = tl.nvi[tile];
  for (int32_t l = tid; l < nvi; l += nthr) tile_sum1<CFL>(tile, l, d, h, tl, L);
}

template <int SCHEME, bool LUMP>
__global__ __launch_bounds__(kBlock, 4) void k_tile2(Dev d, Dev32 h, Tiles tl) {
  extern __shared__ D4 lds_raw[];
  const int64_t tile = xcd_block();
  TileLds L;
  tile_lds(tl, 2, false, reinterpret_cast<char*>(lds_raw), &L);
  const int32_t nthr = blockDim.x, tid = threadIdx.x;
  const int32_t nlv = tl.vbeg[tile + 1] - tl.vbeg[tile];
  for (int32_t l = tid; l < nlv; l += nthr) tile_load2(tile, l, d, h, tl, L);
  __syncthreads();
  const int32_t ntri = tl.tbeg[tile + 1] - tl.tbeg[tile];
  for (int32_t j = tid; j < ntri; j += nthr) tile_tri<SCHEME, 2, false, false, LUMP>(tile, j, d, h, tl, L);
  __syncthreads();
  const int32_t nvi = tl.nvi[tile];
  for (int32_t l = tid; l < nvi; l += nthr) tile_sum2(tile, l, d, h, tl, L);
}

template <bool CFL>
__global__ __launch_bounds__(kBlock) void k_shared1(Dev d, Dev32 h, Tiles tl) {
  const int64_t k = xcd_block() * kBlock + threadIdx.x;
  if (k < tl.nsv) shared_sum1<CFL>(k, d, h, tl);
}

__global__ __launch_bounds__(kBlock) void k_shared2(Dev d, Dev32 h, Tiles tl) {
  const int64_t k = xcd_block() * kBlock + threadIdx.x;
  if (k < tl.nsv) shared_sum2(k, d, h, tl);
}

__global__ __launch_bounds__(kBlock) void k_euler_apply(Dev d, Dev32 h) {
  const int64_t v = xcd_block() * kBlock + threadIdx.x;
  if (v < d.nv) euler_apply(v, d, h);
}

__global__ __launch_bounds__(kBlock) void k_tile_wall2(Dev d, Dev32 h) {
  const int64_t b = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (b < d.nwv) tile_wall2(b, d, h);
}

// Block minima of the vertex CFL bounds the passes store.
__global__ __launch_bounds__(kBlock) void k_tile_cfl(Dev32 h, CflPlan p) {
  const int b = blockIdx.x;
  double x = INFINITY;
  for (int u = 0; u < kCflSpan / kBlock; ++u) {
    const int64_t v = (int64_t)p.blk_v0[b] + u * kBlock + threadIdx.x;
    if (v < p.blk_v1[b]) x = rmin(x, h.cflv[v]);
  }
  const double m = block_min(x);
  if (threadIdx.x == 0) p.part[b] = m;
}

// Smallest and largest flow speed over each block's vertices at W*.
__global__ __launch_bounds__(kBlock) void k_tile_vrange(Dev d, Dev32 h, CflPlan p) {
  const int b = blockIdx.x;
  double lo = INFINITY, hi = 0.0;
  for (int u = 0; u < kCflSpan / kBlock; ++u) {
    const int64_t v = (int64_t)p.blk_v0[b] + u * kBlock + threadIdx.x;
    if (v < p.blk_v1[b]) {
      const double sp = flow_speed(star_state(d, h, v, d.bc ? d.bc[v] : -1, d.vmesh ? d.vmesh[v] : 0));
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

size_t tile_lds_bytes(const Tiles& tl, int stage, bool cfl, size_t size) {
  return tile_lds(tl, stage, cfl, nullptr, nullptr, size);
}

// Threads of a tile workgroup: one triangle each in stage 1, two in stage 2.
static int tile_threads(const Tiles& tl, int stage) {
  const int t = stage == 2 ? tl.tt / 2 : tl.tt;
  return t < 64 ? 64 : (t < kBlock ? t : kBlock);
}

template <int SCHEME>
static hipError_t tile_go(const Dev& d, const Dev32& h, const Tiles& tl, int stage, bool save, bool cfl, hipStream_t s) {
  const dim3 g(tl.ntiles), b(tile_threads(tl, stage));
  const size_t lds = tile_lds(tl, stage, cfl, nullptr, nullptr);
  if (stage == 2 && h.slump) hipLaunchKernelGGL((k_tile2<SCHEME, true>), g, b, lds, s, d, h, tl);
  else if (stage == 2) hipLaunchKernelGGL((k_tile2<SCHEME, false>), g, b, lds, s, d, h, tl);
  else if (save && cfl) hipLaunchKernelGGL((k_tile1<SCHEME, true, true>), g, b, lds, s, d, h, tl);
  else if (save) hipLaunchKernelGGL((k_tile1<SCHEME, true, false>), g, b, lds, s, d, h, tl);
  else if (cfl) hipLaunchKernelGGL((k_tile1<SCHEME, false, true>), g, b, lds, s, d, h, tl);
  else hipLaunchKernelGGL((k_tile1<SCHEME, false, false>), g, b, lds, s, d, h, tl);
  return hipGetLastError();
}

hipError_t launch_tile(const Dev& d, const Dev32& h, const Tiles& tl, int scheme, int stage, bool save, bool cfl,
                       hipStream_t s) {
  switch (scheme) {
    case SCH_N: return tile_go<SCH_N>(d, h, tl, stage, save, cfl, s);
    case SCH_LDA: return tile_go<SCH_LDA>(d, h, tl, stage, save, cfl, s);
    case SCH_B: return tile_go<SCH_B>(d, h, tl, stage, save, cfl, s);
    case SCH_BMAX: return tile_go<SCH_BMAX>(d, h, tl, stage, save, cfl, s);
    case SCH_BMIN: return tile_go<SCH_BMIN>(d, h, tl, stage, save, cfl, s);
    case SCH_BX: return tile_go<SCH_BX>(d, h, tl, stage, save, cfl, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_shared(const Dev& d, const Dev32& h, const Tiles& tl, int stage, bool cfl, hipStream_t s) {
  if (tl.nsv == 0) return hipSuccess;
  const dim3 g(nblk(tl.nsv)), b(kBlock);
  if (stage == 2) hipLaunchKernelGGL(k_shared2, g, b, 0, s, d, h, tl);
  else if (cfl) hipLaunchKernelGGL(k_shared1<true>, g, b, 0, s, d, h, tl);
  else hipLaunchKernelGGL(k_shared1<false>, g, b, 0, s, d, h, tl);
  return hipGetLastError();
}

hipError_t launch_euler_apply(const Dev& d, const Dev32& h, hipStream_t s) {
  hipLaunchKernelGGL(k_euler_apply, dim3(nblk(d.nv)), dim3(kBlock), 0, s, d, h);
  return hipGetLastError();
}

hipError_t launch_tile_wall2(const Dev& d, const Dev32& h, hipStream_t s) {
  if (d.nwv == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_wall2, dim3(nblk(d.nwv)), dim3(kBlock), 0, s, d, h);
  return hipGetLastError();
}

hipError_t launch_tile_cfl(const Dev& d, const Dev32& h, const CflPlan& p, double cfl, hipStream_t s) {
  hipLaunchKernelGGL(k_tile_cfl, dim3(p.nblocks), dim3(kBlock), 0, s, h, p);
  return launch_cfl_final(d, p, cfl, s);
}

hipError_t launch_tile_vrange(const Dev& d, const Dev32& h, const CflPlan& p, hipStream_t s) {
  hipLaunchKernelGGL(k_tile_vrange, dim3(p.nblocks), dim3(kBlock), 0, s, d, h, p);
  return launch_vrange_final(d, p, s);
}

}  // namespace rd
