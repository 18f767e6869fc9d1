// Mesh generation on the GPU: launchers of the flip and refinement passes
// (kernels in rd_delaunay.hip, per-element bodies in rd_delaunay_kern.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rd_delaunay_kern.h"

namespace rd {
namespace dl {

// Account of a run of flip rounds, kept on the device.
struct Control {
  int32_t done = 0;    // a round found no illegal edge
  int32_t rounds = 0;  // rounds that flipped
  int32_t stuck = 0;   // a round with illegal edges flipped none
  int32_t starved = 0; // the exact pass had work and no scratch: done, but unfinished
  int32_t need = 0;    // most edges the exact pass had to test in a round
  int64_t flips = 0;
};

// What the host reads after a batch of launches.
struct Report {
  Control c;
  int32_t count[3];  // candidates, not located, cavities too large
  int32_t nwin, nadd;
};

// Scratch doubles of the exact in-circle pass (m.work) on that many workgroups.
int64_t exact_scratch(int blocks);

// One flip round (start: the first of a run, or the one to try again after it
// starved): reset the claims (and the three
// ints at `also`, if any); test in FP64 the interior edges of the triangles
// marked for test pass `pass`, and exactly those left undecided; flip the
// edges that hold both claims (marking triangles with an illegal edge, and
// flipped ones, for pass + 1); repoint neighbours at flipped pairs. Does
// nothing once the run is done.
enum { kGoOn = 0, kFresh = 1, kResume = 2 };
hipError_t launch_round(const Mesh& m, Control* c, int start, int32_t round, int32_t pass, int* also, int exact_blocks,
                        hipStream_t s);

// One refinement iteration over the m.nt triangles in use, once the flips are
// done (nothing before): candidates (quality and encroachment), their location
// and encroachment test, cavity locks, winners (win, tnew); then, after the
// prefix sums, the insertion and the neighbour repair over the nt_after
// triangles.
hipError_t launch_candidates(const Mesh& m, const Refine& r, const Control* c, hipStream_t s);
hipError_t launch_report(const Mesh& m, const Refine& r, const Control* c, Report* h, hipStream_t s);
hipError_t launch_insert(const Mesh& m, const Refine& r, int32_t it, int32_t pass, hipStream_t s);
hipError_t launch_fixsplit(const Mesh& m, const Refine& r, int32_t it, int64_t nt_after, hipStream_t s);

// Morton ordering passes: keys of n vertices or triangles (with o.idx =
// 0..n-1), the stable sort of (key, idx) into (skey, perm), the inverse
// permutation, and the moves (into o's buffers; the caller swaps them in).
hipError_t launch_vkeys(const Mesh& m, const Order& o, int64_t nv, hipStream_t s);
hipError_t launch_tkeys(const Mesh& m, const Order& o, hipStream_t s);
size_t sort_tmp_bytes(int64_t n);
hipError_t launch_sort(const Order& o, int64_t n, void* tmp, size_t tmp_bytes, hipStream_t s);
hipError_t launch_invert(const Order& o, int64_t n, hipStream_t s);
hipError_t launch_vapply(const Mesh& m, const Order& o, int64_t nv, hipStream_t s);
hipError_t launch_vrename(const Mesh& m, const Order& o, hipStream_t s);
hipError_t launch_tapply(const Mesh& m, const Order& o, hipStream_t s);

// Exclusive prefix sum of n ints (dst may not alias src); tmp of at least
// scan_tmp_bytes(n) bytes.
size_t scan_tmp_bytes(int64_t n);
hipError_t launch_scan(const int32_t* src, int32_t* dst, int64_t n, void* tmp, size_t tmp_bytes, hipStream_t s);

}  // namespace dl
}  // namespace rd
