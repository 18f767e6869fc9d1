// Host-side launchers of the gfx950 kernels (defined in rd_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "rd_adjoint.h"
#include "rd_device.h"

namespace rd {

constexpr int kBlock = 256;

// Stage-1 parts of every triangle, N parts and residual kept.
hipError_t launch_tri(const Dev& d, int scheme, hipStream_t s);
// wall term at W, or (stage2) at Ws
hipError_t launch_wall(const Dev& d, bool stage2, hipStream_t s);
// d.W and d.Z from the caller's [4][nv], and d.dt[0]; flag[0] where non-physical
hipError_t launch_set_state(const Dev& d, const double* soa, double dt, hipStream_t s);
// Vertex residuals (r) -> R [4][nv]; phi^T of every triangle at the state st
// -> phi [4][nt] (may be null).
hipError_t launch_residual(const Dev& d, const State& r, double* R, const State& st, double* phi, hipStream_t s);
// First vertex of a state [2 + momenta][nv] that is not physical -> *bad
// (INT_MAX: none).
hipError_t launch_check_state(const double* W, int64_t nv, int momenta, double gamma, int* bad, hipStream_t s);
hipError_t launch_set_scalar(double* p, double v, hipStream_t s);
hipError_t launch_set_int(int* p, int v, hipStream_t s);
// *p = 0 unless *bad names one of nv vertices
hipError_t launch_clear_unless(int* p, const int* bad, int64_t nv, hipStream_t s);
// p[0..n) = v
hipError_t launch_fill_int(int* p, int v, int64_t n, hipStream_t s);

// The adjoint's first-stage vertex pass: W* from the stage-1 parts and the
// stage-2 reverse records (Z at W*, W* - W^n, mu2) of every vertex.
hipError_t launch_adj_star(const Dev& d, const AdjDev& a, hipStream_t s);
// Reverse of one step (FP64): stage-2 triangles and gather (rk2), then
// stage-1 triangles and gather; dL/dW^n goes to out [4][nv].
hipError_t launch_adjoint(const Dev& d, const AdjDev& a, int scheme, int rk2, double* out, hipStream_t s);

}  // namespace rd
