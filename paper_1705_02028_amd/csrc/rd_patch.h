// Bodies of the patch form of the step.
//
// One workgroup takes one patch of vertices (rd_patching.h): the vertices it
// owns, all triangles with an owned corner, and the other corners of those
// triangles (its halo). It forms the parameter vectors of its vertices in
// LDS, runs one triangle per thread, passes the parts of owned corners
// through LDS (over the vertex records, which are no longer needed), and sums
// each owned vertex's parts in ascending triangle id. Nothing per triangle is
// stored in HBM: a pass reads each vertex's state (and the halo's again,
// about 0.3 nv) and the patch's 12 bytes per triangle of local ids, and
// writes 32 bytes per vertex. Triangles on patch borders are computed by each
// of their patches (about 1.14 nt in all), with the same arithmetic on the
// same inputs, so results do not depend on how the mesh is cut.
//
//   stage 1 (or Euler)  D = (sum of parts + wall term) / V of W^n, and the
//                       patch's smallest CFL bound;
//   stage 2             W* = W^n - dt D in LDS; the triangle's stage-1 N parts
//                       and residual are formed again from W^n (about 250
//                       instructions, against 192 bytes written and read per
//                       triangle to keep them), and the new state goes to the
//                       other of two state buffers.
//
// Measured at 2048^2 (8.4 M triangles, B, RK2, FP64): stage 1 with the CFL
// terms 0.31 ms, stage 2 0.40, a step 0.72 ms, FP64 issue-bound (1.52 ms with
// the parts through HBM, in two passes a stage).
#pragma once

#include "rd_device.h"

namespace rd {

// One patch as its workgroup finds it: 64 bytes, read at once, since every
// other load of the patch waits for them.
struct alignas(64) PatchDesc {
  int32_t v0, own, nlv;  // owned vertices v0 .. v0 + own - 1, local vertices
  int32_t h0;            // halo ids
  int32_t t0, nt;        // patch triangles
  int32_t xy0;           // coordinates of the local vertices
  int32_t mesh;
  int32_t seam;          // 1: some triangle's corner differences are unwrapped
  int32_t jb;            // part slots: the j-th parts (ascending triangle) of the vertices that have one
                         // stand at jb[j] + local vertex; the first eight bases are in jb8
  uint16_t jb8[8];
  int32_t pad[2];
};

// Device view of one mesh (or of a batch laid end to end), vertices in
// internal order.
struct Patches {
  int64_t nv = 0, ptn = 0;  // vertices, patch triangles
  int32_t npatch = 0, threads = 0;
  int32_t max_lv = 0, max_slots = 0, max_tri = 0;
  const PatchDesc* desc = nullptr; // [npatch] wide patches (below) empty
  const int32_t* halo = nullptr;   // internal ids
  const uint32_t* tri = nullptr;   // [3][ptn] local corner id, part slot << 16 (0xffff: not owned)
  const uint16_t* deg = nullptr;   // [nv]
  const int32_t* jb = nullptr;
  const int32_t* mbeg = nullptr;   // [nmesh + 1] patches of each mesh
  int32_t nmesh = 1;
  double gamma = 1.4;
  SymGas gas;
  double px = 0.0, py = 0.0, hpx = 0.0, hpy = 0.0;
  const double2* xy = nullptr;     // coordinates of every patch's local vertices, patch by patch
  const double* V = nullptr;       // [nv] vertex volume, negative on ghosts
  const int32_t* wb = nullptr;     // [nv] wall vertex of each vertex or -1; null without walls
  const int32_t* wptr = nullptr;   // wall incidences of wall vertex b: [wptr[b], wptr[b + 1])
  const WallEnt* went = nullptr;   // their other vertex in internal ids
  D4* W[2] = {nullptr, nullptr};   // state buffers
  int* cur = nullptr;              // cur[0]: where the state is; cur[1]: its copy for stage 2 (see State)
  D4* D = nullptr;                 // [nv] (W^n - W*) / dt, 0 on ghosts
  double* pmin = nullptr;          // [npatch] smallest CFL bound of each patch's vertices
  double* vpart = nullptr;         // [2 npatch] smallest and largest |v| (Bx)
  double* vr = nullptr;            // [3 nmesh] Bx sensor: range of |v|, domain size
  double* dt = nullptr;            // [nmesh]
  int* flag = nullptr;             // [nmesh] non-physical state latch
  double dt_val = 0.0;             // > 0: the step's dt
  double cfl = 0.0;                // > 0: the workgroup takes dt = cfl * min of its mesh's pmin itself
  // a stage-1 pass that first takes the Euler step whose D the pass before it left
  const D4* Dp = nullptr;
  const double* pminp = nullptr;
  int ci = 1;                      // where it (and the Euler update) finds the state's buffer: cur[ci]
  int32_t slump = 0;
  const PatchDesc* all = nullptr;  // [npatch] wide patches as they are
  // Wide patches: those whose vertex records would not fit a workgroup's LDS
  // beside the parts of any one vertex (1166 local vertices or more of 160 KiB:
  // 583 triangles or more around a vertex that share no other corner). They keep
  // them in memory ([3][nloc] records of all patches' local vertices, patch by
  // patch, and in stage 1 |v| + c), and a launch of their own takes them after
  // the others'; so a vertex's bits do not depend on the mesh or batch around
  // it. max_lv does not count them, all_lv does.
  int32_t nwide = 0, all_lv = 0;
  const int32_t* wide = nullptr;   // [nwide] patches
  D4* rec = nullptr;
  double* rsig = nullptr;
  int64_t nloc = 0;
};


constexpr int kPatchThreads = 512;

// Records of four reals in LDS: two planes of n 16-byte units, so that lanes
// that read (or write) consecutive records touch consecutive banks.
struct Lds4 {
  double2* a;
  int32_t n;
  __host__ __device__ D4 get(int32_t i) const {
    const double2 lo = a[i], hi = a[n + i];
    return D4{{lo.x, lo.y, hi.x, hi.y}};
  }
  __host__ __device__ void set(int32_t i, const double v[4]) const {
    a[i] = make_double2(v[0], v[1]);
    a[n + i] = make_double2(v[2], v[3]);
  }
};

// The same in memory.
struct Mem4 {
  D4* a;
  __host__ __device__ D4 get(int32_t i) const { return a[i]; }
  __host__ __device__ void set(int32_t i, const double v[4]) const {
    for (int k = 0; k < 4; ++k) a[i].v[k] = v[k];
  }
};

// Z of a state (and |v| + c), as derive.
__host__ __device__ inline D4 patch_z(const Patches& p, const D4& w, double* sig, bool* ok) {
  const VertexDerived o = derive(p.gamma, w.v);
  D4 z;
  for (int k = 0; k < 4; ++k) z.v[k] = o.z[k];
  if (sig) *sig = o.sig;
  if (ok) *ok = o.ok;
  return z;
}

// W* = W^n - dt D.
__host__ __device__ inline D4 patch_star(const D4& w, const D4& dd, double dt) {
  D4 o;
  for (int k = 0; k < 4; ++k) o.v[k] = w.v[k] - dt * dd.v[k];
  return o;
}

// (W^n - W*) / dt of the W* in hand. Not D itself: the mass term then takes
// the rounding of W* back out of the new state, which D would leave in it (the
// error against 64 bits of two steps at 2048^2 is 6.8e-17 this way, 9.6e-17
// with D).
__host__ __device__ inline D4 patch_rate(const D4& w, const D4& ws, double idt) {
  D4 o;
  for (int k = 0; k < 4; ++k) o.v[k] = (w.v[k] - ws.v[k]) * idt;
  return o;
}

// Stage 2: the stage-1 N parts and residual from Z^n, the total residuals
//   Phi^N_i = |T|/3 r_i + (phi^N_i(n) + phi^N_i(*))/2,  r = (W* - W^n)/dt,
//   Phi^T   = |T|/3 sum_j r_j + (phi^T(n) + phi^T(*))/2,
// and the scheme's parts. zn(i), zs(i), dd(i): Z^n, Z*, -r of corner i, read
// where they are used.
template <int SCHEME, bool LUMP, class ZN, class ZS, class DD>
__host__ __device__ inline void patch_tri2(const Patches& p, const TriDiff& g, const ZN& zn, const ZS& zs, const DD& dd,
                                           const double* vr, double out[3][4]) {
  constexpr bool needN = SCHEME != SCH_LDA, needL = SCHEME != SCH_N;
  double bx = 0.0;
  if (SCHEME == SCH_BX) {
    const D4 z[3] = {zs(0), zs(1), zs(2)};
    bx = bx_theta(g, z, vr);
    sched_fence();
  }
  SymEdge<double> e[3];
  sym_edges(g.d1x, g.d1y, g.d2x, g.d2y, e);
  const double mass = (0.5 * (g.d1x * g.d2y - g.d1y * g.d2x)) * (1.0 / 3.0);
  // what the total parts of corners 0 and 1 and the total residual take from
  // W^n: half the stage-1 value plus the mass term (corner 2's parts are the
  // total residual minus those of corners 0 and 1)
  double b0[4], b1[4], bt[4];
  {
    const D4 z0 = zn(0), z1 = zn(1), z2 = zn(2);
    SymTri<double> s;
    sym_triangle<double, needN>(z0.v, z1.v, z2.v, e, p.gas, s);
    sym_to_conserved(s.f, s.phi, bt);
    if (needN) sym_n_parts(s, e, b0, b1);
  }
  sched_fence();
  {
    const D4 r0 = dd(0), r1 = dd(1), r2 = dd(2);
    for (int k = 0; k < 4; ++k) {
      const double rs = r0.v[k] + r1.v[k] + r2.v[k];
      bt[k] = 0.5 * kSymScale * bt[k] - mass * rs;
      if (needN) {
        b0[k] = 0.5 * kSymScale * b0[k] - mass * r0.v[k];
        b1[k] = 0.5 * kSymScale * b1[k] - mass * r1.v[k];
      }
      if (LUMP && needN) {
        b0[k] = b0[k] + mass * 0.25 * (rs - 3.0 * r0.v[k]);
        b1[k] = b1[k] + mass * 0.25 * (rs - 3.0 * r1.v[k]);
      }
    }
  }
  sched_fence();
  double rhs[4], pN[2][4], pl[2][4];
  {
    SymTri<double> s;
    {
      const D4 z[3] = {zs(0), zs(1), zs(2)};
      sym_triangle<double, needN>(z[0].v, z[1].v, z[2].v, e, p.gas, s);
    }
    sym_to_conserved(s.f, s.phi, rhs);
    for (int k = 0; k < 4; ++k) rhs[k] = 0.5 * kSymScale * rhs[k] + bt[k];
    if (needN) {
      sym_n_parts(s, e, pN[0], pN[1]);
      for (int k = 0; k < 4; ++k) {
        pN[0][k] = 0.5 * kSymScale * pN[0][k] + b0[k];
        pN[1][k] = 0.5 * kSymScale * pN[1][k] + b1[k];
      }
    }
    if (needL) {
      double y[4];
      sym_from_conserved(s.f, rhs, y);
      sym_lda_parts(s, e, y, pl[0], pl[1]);
    }
  }
  if (LUMP && needL) {
    // selective lumping: sum_j (|T| delta_ij / 3 - |T| (1 + delta_ij) / 12) r_j
    // to the N and the LDA parts (it sums to zero over the corners)
    const D4 r0 = dd(0), r1 = dd(1), r2 = dd(2);
    for (int k = 0; k < 4; ++k) {
      const double rs = r0.v[k] + r1.v[k] + r2.v[k];
      pl[0][k] = pl[0][k] + mass * 0.25 * (rs - 3.0 * r0.v[k]);
      pl[1][k] = pl[1][k] + mass * 0.25 * (rs - 3.0 * r1.v[k]);
    }
  }
  blend_parts<SCHEME>(rhs, pN[0], pN[1], pl[0], pl[1], bx, out);
}

}  // namespace rd
