// Host-side launchers of the step with FP32 distribution (rd_fp32.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "rd_fp32.h"
#include "rd_launch.h"
#include "rd_tiles.h"
#include "rd_patch.h"

namespace rd {

constexpr int kCflSpan = 4 * kBlock;  // vertices per block of the CFL reduction

// Segmented min-reduction layout for the CFL limit: vertex block b covers
// vertices [blk_v0[b], blk_v1[b]) (at most kCflSpan) of one mesh; mesh m owns blocks
// [mesh_b0[m], mesh_b0[m+1]).
struct CflPlan {
  int32_t nblocks = 0, nmesh = 0;
  const int32_t* blk_v0 = nullptr;
  const int32_t* blk_v1 = nullptr;
  const int32_t* mesh_b0 = nullptr;
  double* part = nullptr;
  double* vpart = nullptr;  // [2 nblocks] Bx speed range per block
};

// One triangle pass; cfl: also l_max lambda_max per triangle (stage 1).
hipError_t launch_tri32(const Dev& d, const Dev32& h, int scheme, int stage, bool save, bool cfl, hipStream_t s);
// One vertex pass (G_EULER, G_STAGE1, G_STAGE2).
hipError_t launch_gather32(const Dev& d, const Dev32& h, int mode, hipStream_t s);
// A state in a patch buffer into d.W, parameter vectors and signal speeds with
// it; the caller marks where the state is now.
hipError_t launch_enter32(const Dev& d, const Dev32& h, const State& st, hipStream_t s);
// The same from the caller's arrays, and cur[0] set to the FP32 form; nothing
// with a `bad` that names a vertex (launch_check_state).
hipError_t launch_set32(const Dev& d, const Dev32& h, int* cur, const double* soa, const int* bad, hipStream_t s);
// d.dt from the terms of the stage-1 pass.
hipError_t launch_cfl32(const Dev& d, const CflPlan& p, double cfl, hipStream_t s);
// Bx sensor range at W, or (star) at Ws -> d.vr
hipError_t launch_vrange32(const Dev& d, const CflPlan& p, bool star, hipStream_t s);

// Their second halves: the per-mesh results of the block ones.
hipError_t launch_cfl_final(const Dev& d, const CflPlan& p, double cfl, hipStream_t s);
hipError_t launch_vrange_final(const Dev& d, const CflPlan& p, hipStream_t s);

// Tiled form. Stage 1 (also Euler): R1 and, with cfl, the CFL bounds of
// interior vertices; stage 2: their new state.
hipError_t launch_tile(const Dev& d, const Dev32& h, const Tiles& tl, int scheme, int stage, bool save, bool cfl,
                       hipStream_t s);
// The same for the shared vertices.
hipError_t launch_shared(const Dev& d, const Dev32& h, const Tiles& tl, int stage, bool cfl, hipStream_t s);
// Forward-Euler update from R1.
hipError_t launch_euler_apply(const Dev& d, const Dev32& h, hipStream_t s);
// Wall terms at W*, dt from the vertex bounds, Bx sensor range at W*.
hipError_t launch_tile_wall2(const Dev& d, const Dev32& h, hipStream_t s);
hipError_t launch_tile_cfl(const Dev& d, const Dev32& h, const CflPlan& p, double cfl, hipStream_t s);
hipError_t launch_tile_vrange(const Dev& d, const Dev32& h, const CflPlan& p, hipStream_t s);
// Dynamic LDS bytes of a tile workgroup with values of `size` bytes.
size_t tile_lds_bytes(const Tiles& tl, int stage, bool cfl, size_t size);

}  // namespace rd
