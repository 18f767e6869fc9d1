// Host-side launchers of the patch form (rd_patch.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "rd_patch.h"

namespace rd {

// One member of a batch as its copy kernel sees it.
struct PatchMember {
  State st;
  int* cur;
  int* flag;
  int32_t nv, v0;      // vertices; the member's first vertex in the batch (caller's order)
};

// Dynamic LDS bytes of a patch workgroup.
size_t patch_lds_bytes(const Patches& p, int stage, bool cfl, bool wide = false);
// stage 1 (also Euler): p.D and, with cfl, the patch bounds p.pmin; stage 2:
// the new state (in the other buffer).
hipError_t launch_patch(const Patches& p, int scheme, int stage, bool cfl, hipStream_t s);
// The residual of every vertex into p.D (p.vr set for Bx).
hipError_t launch_patch_residual(const Patches& p, int scheme, hipStream_t s);
// Stage 1 with CFL bounds of a state that is one Euler step back (p.Dp,
// p.pminp of the pass before; not for Bx, whose sensor needs the state first).
hipError_t launch_patch_after(const Patches& p, int scheme, hipStream_t s);
// Forward Euler: the state in cur[p.ci]'s buffer by -dt p.D.
hipError_t launch_patch_euler(const Patches& p, hipStream_t s);
// The patch bounds alone (a state in the FP32 form is read from its copy in the
// first patch buffer, see launch_patch_copy), with `done` also their minimum times cfl -> p.dt[0]
// and *host (one mesh).
hipError_t launch_patch_cfl(const Patches& p, double cfl, unsigned* done, double* host, hipStream_t s);
// Per mesh cfl times the minimum of its patches' bounds -> p.dt (and host).
hipError_t launch_patch_dt(const Patches& p, double cfl, hipStream_t s, double* host = nullptr);
// Bx sensor range at W^n, or at W* (after stage 1, with p.dt set) -> p.vr
hipError_t launch_patch_vrange(const Patches& p, bool star, hipStream_t s);
// The state from the caller's [4][nv] arrays into the first patch buffer
// (p.cur[0] with it; nothing with a `bad` that names a vertex, see
// launch_check_state), and from where it is to the caller's arrays or records.
hipError_t launch_patch_set(const Patches& p, const int32_t* inv, const double* soa, const int* bad, hipStream_t s);
hipError_t launch_state_get(const State& st, int64_t nv, double* soa, hipStream_t s);
hipError_t launch_state_get4(const State& st, int64_t nv, D4* out, hipStream_t s);
// Records of the caller's order into the first patch buffer; the state is
// there once p.cur[0] is set (launch_set_int).
hipError_t launch_patch_set4(const Patches& p, const int32_t* inv, const D4* in, hipStream_t s);
// A copy of a state in the FP32 form in the first patch buffer, which holds
// nothing then; nothing where the state is in a patch buffer.
hipError_t launch_patch_copy(const Patches& p, const State& st, hipStream_t s);
// The same, and the state is there from now on.
hipError_t launch_patch_enter(const Patches& p, const State& st, hipStream_t s);
// The members' states into the batch's first patch buffer (batch latches
// cleared), or the batch's state and latches out into the members' first ones.
hipError_t launch_patch_members(const State& st, int* cur, int* flags, int64_t nv,
                                const PatchMember* mem, const int32_t* mb, const int32_t* vb, int nblocks, bool out,
                                hipStream_t s);

}  // namespace rd
