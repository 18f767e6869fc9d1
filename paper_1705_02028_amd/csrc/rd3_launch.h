// Host-side launchers of the three-dimensional kernels (rd3_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "rd3_device.h"

namespace rd3 {

// The state from / to the caller's [5][nv] arrays; set makes Z and |u| + c.
hipError_t launch3_set(const Dev3& d, const double* src, hipStream_t s);
hipError_t launch3_get(const Dev3& d, double* dst, hipStream_t s);
// One tile pass: stage 1 (or Euler) at W, with the CFL terms where cfl, or
// stage 2 at W*; stage 0: the CFL terms alone.
hipError_t launch3_tile(const Dev3& d, int stage, int scheme, bool cfl, hipStream_t s);
// Vertex sums and update: mode 0 Euler, 1 first stage, 2 second stage.
hipError_t launch3_gather(const Dev3& d, int mode, hipStream_t s);
// CFL limit from the tiles' terms, times cfl -> *d.dt (d.bmin holds
// cfl_blocks(nv) values).
int cfl_blocks(int64_t nv);
hipError_t launch3_cfl(const Dev3& d, double cfl, hipStream_t s);
hipError_t launch3_set_dt(const Dev3& d, double dt, hipStream_t s);
// Sets the layout of a tile workgroup's LDS (max_jd: most diagonals of a tile).
void tile3_lds(Dev3& d, int32_t max_jd);

}  // namespace rd3
