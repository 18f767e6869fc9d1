// Host side of the librd C ABI: mesh validation and precompute, device
// buffers, and the order of kernel launches for one step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "rd.h"
#include "rd3_launch.h"
#include "rd3_tiling.h"
#include "rd_delaunay.h"
#include "rd_fp32_launch.h"
#include "rd_launch.h"
#include "rd_noalloc.h"
#include "rd_patch_launch.h"
#include "rd_patching.h"
#include "rd_tiling.h"

#define RD_API extern "C" __attribute__((visibility("default")))

namespace {

thread_local std::string g_last_error;

rd_status fail(rd_status st, const std::string& msg) {
  g_last_error = msg;
  return st;
}

#define HIPCHK(call)                                                                        \
  do {                                                                                      \
    hipError_t e_ = (call);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return fail(RD_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_));          \
  } while (0)

double unwrap_h(double d, double period) {
  if (period > 0.0) {
    if (d > 0.5 * period) d -= period;
    else if (d < -0.5 * period) d += period;
  }
  return d;
}

// Largest vertex degree (triangles per vertex) a mesh may have: the rank of
// a triangle among the triangles of each of its corner vertices is packed in
// 10 bits.
constexpr int32_t kMaxDegree = 1023;

// Host states of up to this many vertices are checked on the host, larger ones
// on the device (launch_check_state), whose two launches and copy take 16 us
// whatever the size (rd_set_state, us, host / device: 20 / 36 at 64 vertices,
// 39 / 41 at 6400, 48 / 44 at 10000; rd3_set_state: 22 / 36 at 125, 40 / 51 at
// 8000, 52 / 56 at 13824, 72 / 65 at 21952, but with an RK2 step and the state
// out after it 164 / 192 at 19683 and 233 / 260 at 27000, 388 / 385 at 54872).
constexpr int64_t kHostCheck2 = 8192, kHostCheck3 = 32768;

// First vertex of a state [2 + momenta][nv] that is not physical, nv if none:
// the check of launch_check_state.
int64_t first_unphysical(const double* W, int64_t nv, int momenta, double gamma) {
  for (int64_t i = 0; i < nv; ++i) {
    const double rho = W[i], e = W[(1 + momenta) * nv + i];
    bool ok = rho > 0.0 && std::isfinite(e) && (momenta == 3 || std::isfinite(rho));
    double q = 0.0;
    for (int k = 1; k <= momenta; ++k) {
      const double m = W[k * nv + i];
      q += m * m;
      ok = ok && (momenta == 3 || std::isfinite(m));
    }
    if (!ok || !((gamma - 1.0) * (e - 0.5 * q / rho) > 0.0)) return i;
  }
  return nv;
}

int host_threads() {
  const unsigned n = std::thread::hardware_concurrency();
  return (int)std::min(8u, std::max(1u, n));
}

// The host side of a call may run out of memory (or of threads): no C++
// exception crosses the ABI.
template <class F>
rd_status guarded(F f) {
  try {
    return f();
  } catch (const std::bad_alloc&) {
    return fail(RD_ENOMEM, "host allocation failed");
  } catch (const std::exception& e) {
    return fail(RD_ENOMEM, std::string("host: ") + e.what());
  }
}

// What check_desc works out: the vertex -> corner lists (corner 3 t + i,
// ascending t in each row) and the vertex volumes (median dual).
struct HostGeom {
  rd::UVec<int32_t> row, slot;
  rd::UVec<double> V;
};

// Workers for the host side of a mesh of n triangles: small ones are done
// sooner than the threads would start, medium ones before eight would (mesh
// creation, us, by one / four / eight: 620 / 590 / 700 at 64^2, 1400 / 900 /
// 1000 at 93^2, 2800 / 1600 / 1500 at 144^2).
int workers_for(int64_t nt) { return nt < 10000 ? 1 : nt < 30000 ? std::min(4, host_threads()) : host_threads(); }

// The checks of rd_mesh_validate, and (out) the lists. Each worker takes a
// range of triangles, then a range of vertices, whose corners it finds by
// reading the triangles in blocks, those blocks that have none left out.
rd_status check_desc(const rd_mesh_desc* d, HostGeom* out, rd::Workers& pool) {
  if (!d) return fail(RD_EINVAL, "null mesh description");
  if (d->n_vertices <= 0 || d->n_triangles <= 0) return fail(RD_EINVAL, "empty mesh");
  if (d->n_vertices >= (int64_t(1) << 31) || 3 * d->n_triangles >= (int64_t(1) << 31))
    return fail(RD_EINVAL, "mesh too large for 32-bit indices");
  if (!d->x || !d->y || !d->tri) return fail(RD_EINVAL, "null coordinate or triangle array");
  if (!(d->gamma > 1.0)) return fail(RD_EINVAL, "gamma must exceed 1");
  if (d->period_x < 0.0 || d->period_y < 0.0) return fail(RD_EINVAL, "negative period");
  if (d->n_wall_edges < 0 || (d->n_wall_edges > 0 && !d->wall_edges))
    return fail(RD_EINVAL, "bad wall edge list");
  const int64_t nv = d->n_vertices, nt = d->n_triangles;
  const int w = pool.size();
  constexpr int64_t kBlockTri = 1024;
  const int64_t nb = (nt + kBlockTri - 1) / kBlockTri;
  struct Span {
    int32_t lo, hi;  // vertices of a block's corners
  };
  rd::UVec<Span> span(nb);
  rd::UVec<double> third(out ? nt : 0);  // a third of each triangle's area
  std::vector<int64_t> bad(w, nt);       // first bad triangle of each worker
  pool.run([&](int q) {
    for (int64_t k = nb * q / w; k < nb * (q + 1) / w; ++k) {
      int32_t lo = INT32_MAX, hi = -1;
      for (int64_t t = k * kBlockTri; t < std::min(nt, (k + 1) * kBlockTri); ++t) {
        const int32_t* v = d->tri + 3 * t;
        if (t + 16 < nt)  // the coordinates of one ahead: without locality each is a miss
          for (int c = 0; c < 3; ++c) {
            __builtin_prefetch(d->x + v[48 + c]);
            __builtin_prefetch(d->y + v[48 + c]);
          }
        const int32_t v0 = std::min(v[0], std::min(v[1], v[2])), v1 = std::max(v[0], std::max(v[1], v[2]));
        lo = std::min(lo, v0);
        hi = std::max(hi, v1);
        double area = 0.0;
        if (v0 >= 0 && v1 < nv) {
          double px[3] = {0.0, 0.0, 0.0}, py[3] = {0.0, 0.0, 0.0};
          for (int c = 1; c < 3; ++c) {
            px[c] = unwrap_h(d->x[v[c]] - d->x[v[0]], d->period_x);
            py[c] = unwrap_h(d->y[v[c]] - d->y[v[0]], d->period_y);
          }
          area = 0.5 * (px[1] * py[2] - py[1] * px[2]);
        }
        if (!(area > 0.0)) {
          bad[q] = t;
          return;
        }
        if (out) third[t] = area / 3.0;
      }
      span[k] = Span{lo, hi};
    }
  });
  for (int64_t t : bad)
    if (t < nt) {
      for (int k = 0; k < 3; ++k)
        if (d->tri[3 * t + k] < 0 || d->tri[3 * t + k] >= nv)
          return fail(RD_EINVAL, "triangle " + std::to_string(t) + " has a vertex index out of range");
      return fail(RD_EINVAL, "triangle " + std::to_string(t) + " is not counter-clockwise with positive area");
    }
  // f(s, v) for the corners s of the vertices v in [a, b), ascending; collected
  // block by block first, without a branch on each
  auto corners = [&](int64_t a, int64_t b, const auto& f) {
    int32_t mine[3 * kBlockTri];
    for (int64_t k = 0; k < nb; ++k) {
      if (span[k].hi < a || span[k].lo >= b) continue;
      const int64_t s0 = 3 * k * kBlockTri, s1 = 3 * std::min(nt, (k + 1) * kBlockTri);
      int32_t n = 0;
      for (int64_t s = s0; s < s1; ++s) {
        mine[n] = (int32_t)s;
        n += (uint64_t)(d->tri[s] - a) < (uint64_t)(b - a);
      }
      for (int32_t i = 0; i < n; ++i) f(mine[i], d->tri[mine[i]]);
    }
  };
  auto share = [&](int q) { return nv * q / w; };
  HostGeom geo;
  rd::UVec<int32_t>&row = geo.row, &slot = geo.slot;
  row.resize(nv + 1);
  std::vector<int64_t> first(w + 1, 0), lost(w, nv);  // corners before each worker's vertices; first bad vertex
  pool.run([&](int q) {
    const int64_t a = share(q), b = share(q + 1);
    std::fill(row.begin() + a + 1, row.begin() + b + 1, 0);
    corners(a, b, [&](int64_t, int32_t v) { ++row[v + 1]; });
    int64_t n = 0;
    for (int64_t i = b; i-- > a;) {
      n += row[i + 1];
      if (row[i + 1] == 0 || row[i + 1] > kMaxDegree) lost[q] = i;
    }
    first[q + 1] = n;
  });
  for (int64_t i : lost)
    if (i < nv) {
      const int32_t deg = row[i + 1];
      if (deg == 0) return fail(RD_EINVAL, "vertex " + std::to_string(i) + " belongs to no triangle");
      // a triangle's rank among the triangles of each corner vertex is packed in 10 bits
      return fail(RD_EINVAL, "vertex " + std::to_string(i) + " belongs to " + std::to_string(deg) +
                                 " triangles; at most " + std::to_string(kMaxDegree) + " are supported");
    }
  for (int64_t e = 0; e < d->n_wall_edges; ++e) {
    const int32_t a = d->wall_edges[2 * e], b = d->wall_edges[2 * e + 1];
    if (a < 0 || a >= nv || b < 0 || b >= nv || a == b)
      return fail(RD_EINVAL, "wall edge " + std::to_string(e) + " is invalid");
  }
  if (!out) return RD_OK;
  for (int q = 0; q < w; ++q) first[q + 1] += first[q];
  slot.resize(3 * nt);
  geo.V.resize(nv);
  row[0] = 0;
  pool.run([&](int q) {
    const int64_t a = share(q), b = share(q + 1);
    rd::UVec<int32_t> next(b - a);  // where each vertex's next corner goes
    int32_t at = (int32_t)first[q];
    for (int64_t i = a; i < b; ++i) {
      next[i - a] = at;
      at += row[i + 1];
      row[i + 1] = at;
      geo.V[i] = 0.0;
    }
    corners(a, b, [&](int64_t s, int32_t v) {
      slot[next[v - a]++] = (int32_t)s;
      geo.V[v] += third[s / 3];
    });
  });
  *out = std::move(geo);
  return RD_OK;
}

}  // namespace

constexpr size_t kSlab = size_t(1) << 19;

struct rd_mesh {
  rd::Patches p;             // the step's view, vertices in internal order (patch by patch)
  rd::Dev d;                 // the second view (the caller's order): residual, adjoint
  rd::CflPlan cfl;           // its vertex reductions
  // the FP32 step (its state is d.W): buffers allocated on first use, and its tiles
  rd::Dev32 d32;
  rd::Tiles tiles;
  std::vector<void*> tile_allocs;
  // Where the state is by the host's account: in the FP32 form after FP32
  // steps (d32.Zf and d.sig belong to it then), else in a patch buffer. Once a
  // call of this mesh was captured only the device's word (p.cur[0]) counts,
  // since a replay moves the state without the host's knowledge.
  bool form32 = false;
  bool captured = false;
  hipStream_t stream = nullptr;
  int device = 0;
  int ncu = 0;      // compute units of the device
  int lds_max = 0;  // bytes of LDS one workgroup may use on the device
  // host copies, kept for batches, for other patches and for the second view
  rd::UVec<double> x, y, V;
  rd::UVec<int32_t> tri, row, slot;
  rd::UVec<int32_t> bc;
  std::vector<int32_t> wall, wv, wptr;
  rd::UVec<uint8_t> ghost;
  std::vector<rd::WallEnt> went;
  double px = 0.0, py = 0.0, gamma = 1.4;
  double Ldom = 0.0;  // domain size of the Bx sensor
  // device buffers
  std::vector<void*> allocs;
  // the newest shared allocations (of buffers, and of tables from the host), and
  // their bytes that are free
  struct Slab {
    char* at = nullptr;
    size_t left = 0;
  } slab, tables;
  // during creation: what goes to the tables, in one copy
  rd::UVec<char> stage;
  bool staging = false;
  double* scratch = nullptr;      // [4 nv] host states pass through it
  int* bad = nullptr;             // first vertex of a host state that is not physical
  unsigned* done = nullptr;       // workgroups of the CFL pass that have finished
  double* host_dt = nullptr;      // host memory it writes its result to, from the second rd_max_dt on
  bool asked = false;             // rd_max_dt has been called
  double* phi_scratch = nullptr;  // [4 nt] triangle residuals to a host caller
  // adjoint buffers, allocated on first use
  rd::AdjDev adj;
  rd::D4* adjW = nullptr;     // W^n of the step being reversed
  double* adjIn = nullptr;    // [4 nv] host staging: W^n in, then dL/dW^n out
  double* adjOut = nullptr;   // [4 nv] host staging: dL/dW^{n+1} in
  hipEvent_t events[RD_NKERNELS + 1] = {};
  // patches
  int tile = 0;                     // triangles per tile of the FP32 step, 0: its two-pass form
  int32_t max_mesh_patches = 0;     // patches of the mesh (of a batch: the member) that has most
  int64_t tile_info[4] = {0, 0, 0, 0};
  const int32_t* inv = nullptr;     // [nv] device: internal vertex of each of the caller's
  std::vector<int64_t> voff, toff;  // vertex / triangle ranges of the meshes laid end to end
};

namespace {

template <class T>
rd_status dalloc_in(std::vector<void*>& list, T** p, size_t n) {
  void* q = nullptr;
  if (n == 0) n = 1;
  hipError_t e = hipMalloc(&q, n * sizeof(T));
  if (e != hipSuccess) {
    *p = nullptr;
    return fail(RD_ENOMEM, "hipMalloc of " + std::to_string(n * sizeof(T)) + " bytes failed");
  }
  list.push_back(q);
  *p = static_cast<T*>(q);
  return RD_OK;
}

// Brings what is staged to the device.
rd_status flush_stage(rd_mesh* m) {
  const size_t n = kSlab - m->tables.left;
  if (m->staging && m->tables.at) HIPCHK(hipMemcpy(m->tables.at, m->stage.data(), n, hipMemcpyHostToDevice));
  return RD_OK;
}

// Buffers that live as long as the mesh: small ones (a small mesh has some
// sixty) share allocations of half a megabyte, at 256-byte boundaries.
template <class T>
rd_status dalloc(rd_mesh* m, T** p, size_t n, rd_mesh::Slab rd_mesh::*from = &rd_mesh::slab) {
  rd_mesh::Slab& s = m->*from;
  const size_t bytes = (std::max<size_t>(n, 1) * sizeof(T) + 255) & ~size_t(255);
  if (bytes > kSlab / 4) return dalloc_in(m->allocs, p, n);
  if (bytes > s.left) {
    const bool tables = &s == &m->tables;
    rd_status st = tables ? flush_stage(m) : RD_OK;
    if (st != RD_OK || (st = dalloc_in(m->allocs, &s.at, kSlab)) != RD_OK) return st;
    s.left = kSlab;
    if (tables && m->staging) m->stage.resize(kSlab);
  }
  *p = reinterpret_cast<T*>(s.at + (kSlab - s.left));
  s.left -= bytes;
  return RD_OK;
}

// Several buffers of a mesh in one allocation: the runtime keeps about 64 MB of
// freed blocks, and an allocation that makes it give one of them back takes 250
// us, so a dozen of a first call's own could take milliseconds.
class Block {
 public:
  template <class T>
  Block& add(T** p, size_t n) {
    at_[n_++] = {reinterpret_cast<void**>(p), bytes_};
    bytes_ += (std::max<size_t>(n, 1) * sizeof(T) + 255) & ~size_t(255);
    return *this;
  }
  rd_status take(rd_mesh* m) {
    char* q;
    rd_status st = dalloc(m, &q, bytes_);
    for (int k = 0; st == RD_OK && k < n_; ++k) *at_[k].first = q + at_[k].second;
    return st;
  }

 private:
  std::pair<void**, size_t> at_[16];
  int n_ = 0;
  size_t bytes_ = 0;
};

template <class T, class A>
rd_status upload_in(std::vector<void*>& list, T** p, const std::vector<T, A>& h) {
  rd_status st = dalloc_in(list, p, h.size());
  if (st != RD_OK) return st;
  if (!h.empty()) HIPCHK(hipMemcpy(*p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice));
  return RD_OK;
}

template <class T, class A>
rd_status upload(rd_mesh* m, T** p, const std::vector<T, A>& h) {
  rd_status st = dalloc(m, p, h.size(), &rd_mesh::tables);
  if (st != RD_OK || h.empty()) return st;
  const ptrdiff_t at = m->tables.at ? reinterpret_cast<char*>(*p) - m->tables.at : -1;
  const size_t bytes = h.size() * sizeof(T);
  if (m->staging && at >= 0 && at + bytes <= kSlab) std::memcpy(&m->stage[at], h.data(), bytes);
  else HIPCHK(hipMemcpy(*p, h.data(), bytes, hipMemcpyHostToDevice));
  return RD_OK;
}

void free_list(std::vector<void*>& list) {
  for (void* p : list) (void)hipFree(p);
  list.clear();
}

void free_all(rd_mesh* m) {
  if (m->host_dt) (void)hipHostFree(m->host_dt);
  m->host_dt = nullptr;
  free_list(m->tile_allocs);
  free_list(m->allocs);
}

struct DeviceGuard {
  int prev = -1;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) (void)hipSetDevice(dev);
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

// One step of Sections 3.2-3.4. With cfl > 0 the time step is computed on
// the device from the state at the start of the step: the stage-1 pass leaves
// every patch's smallest bound, and the pass that needs dt takes their
// minimum itself where no mesh has more than kDirectPatches patches (one load
// per thread of the workgroup), else one workgroup per mesh reduces them
// first (one more launch, against more than kDirectPatches loads by every
// workgroup). Otherwise dt is given. With `ev` (RD_NKERNELS + 1 events) an
// event is recorded before every kernel slot and after the last.
constexpr int32_t kDirectPatches = rd::kPatchThreads;

rd_status run_step32(rd_mesh* m, int scheme, int time, double cfl, double dt, hipEvent_t* ev);

rd_status run_step(rd_mesh* m, int scheme, int time, int fp32, double cfl, double dt, hipEvent_t* ev = nullptr) {
  if (fp32) return run_step32(m, scheme, time, cfl, dt, ev);
  rd::Patches p = m->p;
  hipStream_t s = m->stream;
  auto mark = [&](int k) -> hipError_t { return ev ? hipEventRecord(ev[k], s) : hipSuccess; };
  const bool with_cfl = cfl > 0.0, bx = scheme == RD_BX;
  p.dt_val = with_cfl ? 0.0 : dt;
  HIPCHK(mark(RD_K_WALL1));
  HIPCHK(mark(RD_K_TRI1));
  if (bx) HIPCHK(rd::launch_patch_vrange(p, false, s));
  HIPCHK(rd::launch_patch(p, scheme, 1, with_cfl, s));
  HIPCHK(mark(RD_K_SHARED1));
  HIPCHK(mark(RD_K_CFL));
  if (with_cfl) {
    if (m->max_mesh_patches <= kDirectPatches && !bx) p.cfl = cfl;
    else HIPCHK(rd::launch_patch_dt(p, cfl, s));
  }
  HIPCHK(mark(RD_K_GATHER1));
  if (time != RD_RK2) HIPCHK(rd::launch_patch_euler(p, s));
  HIPCHK(mark(RD_K_WALL2));
  HIPCHK(mark(RD_K_TRI2));
  if (time == RD_RK2) {
    if (bx) HIPCHK(rd::launch_patch_vrange(p, true, s));
    HIPCHK(rd::launch_patch(p, scheme, 2, false, s));
  }
  HIPCHK(mark(RD_K_GATHER2));
  HIPCHK(mark(RD_NKERNELS));
  return RD_OK;
}

// n CFL-limited steps. FP64 Euler steps of one call run into each other (a
// pass brings the state forward by the step before it); D and the bounds
// alternate between two buffers, the second lent by the second view and the
// speed ranges.
rd_status run_steps(rd_mesh* m, int n, int scheme, int time, int fp32, double cfl) {
  rd_status st;
  if (fp32 || time == RD_RK2 || scheme == RD_BX || n < 2) {
    for (int k = 0; k < n; ++k)
      if ((st = run_step(m, scheme, time, fp32, cfl, 0.0)) != RD_OK) return st;
    return RD_OK;
  }
  rd::Patches p = m->p;
  hipStream_t s = m->stream;
  rd::D4* D[2] = {p.D, m->d.Ws};
  double* pmin[2] = {p.pmin, p.vpart};
  const bool direct = m->max_mesh_patches <= kDirectPatches;
  for (int k = 0; k < n; ++k) {
    p.ci = k & 1;
    p.D = D[k & 1];
    p.Dp = D[~k & 1];
    p.pmin = pmin[k & 1];
    p.pminp = pmin[~k & 1];
    HIPCHK(k ? rd::launch_patch_after(p, scheme, s) : rd::launch_patch(p, scheme, 1, true, s));
    if (direct) p.cfl = cfl;
    else HIPCHK(rd::launch_patch_dt(p, cfl, s));
  }
  p.ci = n & 1;
  HIPCHK(rd::launch_patch_euler(p, s));
  return RD_OK;
}

// The tiled form of the FP32 step: the tile pass finishes interior vertices
// (stage 1: their residual R1 and CFL bound; stage 2: their new state), the
// shared pass the rest. Stage 1 stores R1 only; W* is rebuilt from it where
// needed, after dt is known.
rd_status run_step32_tiled(rd_mesh* m, int scheme, int time, double cfl, double dt, hipEvent_t* ev) {
  const rd::Dev d = m->d;
  const rd::Tiles& tl = m->tiles;
  rd::Dev32 h = m->d32;
  h.slump = m->p.slump;
  hipStream_t s = m->stream;
  auto mark = [&](int k) -> hipError_t { return ev ? hipEventRecord(ev[k], s) : hipSuccess; };
  const bool with_cfl = cfl > 0.0, rk2 = time == RD_RK2, bx = scheme == RD_BX;
  HIPCHK(mark(RD_K_WALL1));
  if (!with_cfl) HIPCHK(rd::launch_set_scalar(d.dt, dt, s));
  HIPCHK(rd::launch_wall(d, false, s));
  HIPCHK(mark(RD_K_TRI1));
  if (bx) HIPCHK(rd::launch_vrange32(d, m->cfl, false, s));
  HIPCHK(rd::launch_tile(d, h, tl, scheme, 1, rk2, with_cfl, s));
  HIPCHK(mark(RD_K_SHARED1));
  HIPCHK(rd::launch_shared(d, h, tl, 1, with_cfl, s));
  HIPCHK(mark(RD_K_CFL));
  if (with_cfl) HIPCHK(rd::launch_tile_cfl(d, h, m->cfl, cfl, s));
  HIPCHK(mark(RD_K_GATHER1));
  if (!rk2) HIPCHK(rd::launch_euler_apply(d, h, s));
  HIPCHK(mark(RD_K_WALL2));
  if (rk2) HIPCHK(rd::launch_tile_wall2(d, h, s));
  HIPCHK(mark(RD_K_TRI2));
  if (rk2 && bx) HIPCHK(rd::launch_tile_vrange(d, h, m->cfl, s));
  if (rk2) HIPCHK(rd::launch_tile(d, h, tl, scheme, 2, false, false, s));
  HIPCHK(mark(RD_K_GATHER2));
  if (rk2) HIPCHK(rd::launch_shared(d, h, tl, 2, false, s));
  HIPCHK(mark(RD_NKERNELS));
  return RD_OK;
}

// The step with FP32 distribution, two passes over the second view.
rd_status run_step32(rd_mesh* m, int scheme, int time, double cfl, double dt, hipEvent_t* ev) {
  if (m->tiles.ntiles > 0) return run_step32_tiled(m, scheme, time, cfl, dt, ev);
  const rd::Dev d = m->d;
  rd::Dev32 h = m->d32;
  h.slump = m->p.slump;
  hipStream_t s = m->stream;
  auto mark = [&](int k) -> hipError_t { return ev ? hipEventRecord(ev[k], s) : hipSuccess; };
  const bool with_cfl = cfl > 0.0, bx = scheme == RD_BX, rk2 = time == RD_RK2;
  HIPCHK(mark(RD_K_WALL1));
  if (!with_cfl) HIPCHK(rd::launch_set_scalar(d.dt, dt, s));
  HIPCHK(rd::launch_wall(d, false, s));
  HIPCHK(mark(RD_K_TRI1));
  if (bx) HIPCHK(rd::launch_vrange32(d, m->cfl, false, s));
  HIPCHK(rd::launch_tri32(d, h, scheme, 1, rk2, with_cfl, s));
  HIPCHK(mark(RD_K_SHARED1));
  HIPCHK(mark(RD_K_CFL));
  if (with_cfl) HIPCHK(rd::launch_cfl32(d, m->cfl, cfl, s));
  HIPCHK(mark(RD_K_GATHER1));
  HIPCHK(rd::launch_gather32(d, h, rk2 ? rd::G_STAGE1 : rd::G_EULER, s));
  HIPCHK(mark(RD_K_WALL2));
  if (rk2) HIPCHK(rd::launch_wall(d, true, s));
  HIPCHK(mark(RD_K_TRI2));
  if (rk2) {
    if (bx) HIPCHK(rd::launch_vrange32(d, m->cfl, true, s));
    HIPCHK(rd::launch_tri32(d, h, scheme, 2, false, false, s));
  }
  HIPCHK(mark(RD_K_GATHER2));
  if (rk2) HIPCHK(rd::launch_gather32(d, h, rd::G_STAGE2, s));
  HIPCHK(mark(RD_NKERNELS));
  return RD_OK;
}

rd::State state_of(const rd_mesh* m) {
  return rd::State{{m->p.W[0], m->p.W[1]}, m->p.cur, m->inv, m->d.W};
}

// The tables of the second view of the mesh and the blocks of its vertex
// reductions.
rd_status build_view(rd_mesh* m, rd::Workers& pool) {
  rd::Dev& d = m->d;
  rd::CflPlan& c = m->cfl;
  const int64_t nv = m->d.nv, nt = m->d.nt;
  d.flag = m->p.flag;
  d.dt = m->p.dt;
  d.vr = m->p.vr;
  d.gamma = m->gamma;
  d.igamma = 1.0 / m->gamma;
  d.gas = m->p.gas;
  d.px = m->px;
  d.py = m->py;
  d.hpx = m->p.hpx;
  d.hpy = m->p.hpy;
  d.nwv = (int32_t)m->wv.size();
  // sliced part layout: 64-vertex slices, each as wide as its largest
  // degree; the j-th part of vertex v sits at sbase[v / 64] + v % 64 + 64 j
  std::vector<int32_t> sbase((nv + 63) / 64);
  int64_t base = 0;
  for (int64_t g0 = 0; g0 < nv; g0 += 64) {
    int32_t width = 0;
    for (int64_t v = g0; v < std::min<int64_t>(g0 + 64, nv); ++v) width = std::max(width, m->row[v + 1] - m->row[v]);
    sbase[g0 / 64] = (int32_t)base;
    base += 64 * (int64_t)width;
    if (base >= (int64_t(1) << 31)) return fail(RD_EINVAL, "mesh too large for 32-bit part slots");
  }
  d.ns = base;
  rd::UVec<double2> xy(nv);
  rd::UVec<int32_t> tv(3 * nt), vtri(base);
  std::vector<int32_t> vmesh, tmesh;
  rd::UVec<uint32_t> rk(nt);
  // the triangle of every part slot (none: -1)
  pool.each((int64_t)sbase.size(), [&](int64_t g) {
    const int64_t end = g + 1 < (int64_t)sbase.size() ? sbase[g + 1] : base;
    for (int64_t l = 0; l < 64; ++l) {
      const int64_t v = 64 * g + l;
      const int32_t n = v < nv ? m->row[v + 1] - m->row[v] : 0;
      if (v < nv) xy[v] = make_double2(m->x[v], m->y[v]);
      for (int64_t j = 0; sbase[g] + 64 * j < end; ++j)
        vtri[sbase[g] + l + 64 * j] = j < n ? m->slot[m->row[v] + j] / 3 : -1;
    }
  });
  // corners, and the rank of each triangle among the triangles of each of its
  // corner vertices (10 bits per corner)
  pool.each(nt, [&](int64_t t) {
    uint32_t r = 0;
    for (int k = 0; k < 3; ++k) {  // the lists ahead: without locality each is two misses
      if (t + 24 < nt) __builtin_prefetch(&m->row[m->tri[3 * (t + 24) + k]]);
      if (t + 12 < nt) __builtin_prefetch(&m->slot[m->row[m->tri[3 * (t + 12) + k]]]);
    }
    for (int k = 0; k < 3; ++k) {
      const int32_t v = m->tri[3 * t + k];
      tv[k * nt + t] = v;
      const int32_t* b = &m->slot[m->row[v]];
      uint32_t j = 0;
      while (b[j] != 3 * t + k) ++j;
      r |= j << (10 * k);
    }
    rk[t] = r;
  });
  const size_t nmesh = m->voff.size() - 1;
  if (nmesh > 1) {
    vmesh.resize(nv);
    tmesh.resize(nt);
    for (size_t k = 0; k < nmesh; ++k) {
      std::fill(vmesh.begin() + m->voff[k], vmesh.begin() + m->voff[k + 1], (int32_t)k);
      std::fill(tmesh.begin() + m->toff[k], tmesh.begin() + m->toff[k + 1], (int32_t)k);
    }
  }
  // blocks of the CFL reduction, none straddling two meshes
  std::vector<int32_t> v0, v1, b0{0};
  for (size_t k = 0; k < nmesh; ++k) {
    for (int64_t v = m->voff[k]; v < m->voff[k + 1]; v += rd::kCflSpan) {
      v0.push_back((int32_t)v);
      v1.push_back((int32_t)std::min<int64_t>(v + rd::kCflSpan, m->voff[k + 1]));
    }
    b0.push_back((int32_t)v0.size());
  }
  double2* pxy;
  double *pV, *part, *vpart;
  int32_t *prow, *ptv, *psbase, *pvtri, *pbc, *pwv, *pwptr, *pvm, *ptm, *pv0, *pv1, *pb0;
  uint32_t* prk;
  rd::WallEnt* pwent;
  rd_status st;
  if ((st = upload(m, &pxy, xy)) || (st = upload(m, &pV, m->V)) || (st = upload(m, &prow, m->row)) ||
      (st = upload(m, &ptv, tv)) || (st = upload(m, &prk, rk)) || (st = upload(m, &psbase, sbase)) ||
      (st = upload(m, &pvtri, vtri)) || (st = upload(m, &pbc, m->bc)) || (st = upload(m, &pwv, m->wv)) ||
      (st = upload(m, &pwptr, m->wptr)) || (st = upload(m, &pwent, m->went)) ||
      (st = upload(m, &pvm, vmesh)) || (st = upload(m, &ptm, tmesh)) || (st = upload(m, &pv0, v0)) ||
      (st = upload(m, &pv1, v1)) || (st = upload(m, &pb0, b0)) ||
      (st = dalloc(m, &part, v0.size())) || (st = dalloc(m, &vpart, 2 * v0.size())))
    return st;
  d.xy = pxy;
  d.V = pV;
  d.row = prow;
  d.tv = ptv;
  d.rk = prk;
  d.sbase = psbase;
  d.vtri = pvtri;
  d.bc = m->bc.empty() ? nullptr : pbc;
  d.wv = pwv;
  d.wptr = pwptr;
  d.went = pwent;
  d.vmesh = vmesh.empty() ? nullptr : pvm;
  d.tmesh = tmesh.empty() ? nullptr : ptm;
  c.nblocks = (int32_t)v0.size();
  c.nmesh = (int32_t)nmesh;
  c.blk_v0 = pv0;
  c.blk_v1 = pv1;
  c.mesh_b0 = pb0;
  c.part = part;
  c.vpart = vpart;
  return RD_OK;
}

void note_capture(rd_mesh* m) {
  hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(m->stream, &c) != hipSuccess) (void)hipGetLastError();
  else m->captured = m->captured || c != hipStreamCaptureStatusNone;
}

// Builds the tiles of tt triangles (0: drops them). Sizes whose tiles would
// not fit a workgroup's LDS with 8-byte values are refused.
rd_status build_tiles(rd_mesh* m, int tt) {
  const rd::Dev& d = m->d;
  rd::TilePlan P;
  auto replace = [&](std::vector<void*> list, const rd::Tiles& tl) {
    // a captured graph may still read the old tables
    if (m->captured) m->allocs.insert(m->allocs.end(), m->tile_allocs.begin(), m->tile_allocs.end());
    else free_list(m->tile_allocs);
    m->tile_allocs = std::move(list);
    m->tiles = tl;
    m->tile = tt;
    const int64_t info[4] = {P.ntiles, (int64_t)P.tvl.size(), (int64_t)P.sv.size(), 0};
    for (int k = 0; k < 4; ++k) m->tile_info[k] = info[k];
    for (int32_t v : P.sv) m->tile_info[3] += m->row[v + 1] - m->row[v];
  };
  if (tt == 0) {
    replace({}, rd::Tiles());
    return RD_OK;
  }
  const std::string why = rd::build_tile_plan(d.nv, d.nt, m->tri.data(), m->x.data(), m->y.data(), m->px, m->py,
                                              m->row.data(), m->slot.data(), m->voff, m->toff, tt, P);
  if (!why.empty()) return fail(RD_EINVAL, why);
  rd::Tiles tl;
  tl.ntiles = P.ntiles;
  tl.tt = P.tt;
  tl.max_lv = P.max_lv;
  tl.max_lvi = P.max_lvi;
  tl.max_slots = P.max_slots;
  tl.nsv = (int64_t)P.sv.size();
  tl.nss = P.nss;
  const size_t need = std::max(rd::tile_lds_bytes(tl, 1, true, sizeof(double)),
                               rd::tile_lds_bytes(tl, 2, false, sizeof(double)));
  if (need > (size_t)m->lds_max)
    return fail(RD_EUNSUPPORTED, "tiles of " + std::to_string(tt) + " triangles need " + std::to_string(need) +
                                     " bytes of LDS");
  std::vector<void*> list;
  int32_t *tbeg, *vbeg, *nvi, *lpb, *lp, *tvl, *dst, *tm, *sv, *ssbeg;
  uint16_t* lv;
  rd::F4* cs;
  double* lams;
  rd_status st;
  if ((st = upload_in(list, &tbeg, P.tbeg)) || (st = upload_in(list, &vbeg, P.vbeg)) ||
      (st = upload_in(list, &nvi, P.nvi)) || (st = upload_in(list, &lpb, P.lpb)) ||
      (st = upload_in(list, &lp, P.lp)) || (st = upload_in(list, &tvl, P.tvl)) ||
      (st = upload_in(list, &lv, P.lv)) || (st = upload_in(list, &dst, P.dst)) ||
      (st = upload_in(list, &tm, P.tmesh)) || (st = upload_in(list, &sv, P.sv)) ||
      (st = upload_in(list, &ssbeg, P.ssbeg)) || (st = dalloc_in(list, &cs, (size_t)P.nss)) ||
      (st = dalloc_in(list, &lams, (size_t)P.nss))) {
    free_list(list);
    return st;
  }
  if (!m->d32.R1) {
    rd::D4* r1;
    double* cv;
    if ((st = dalloc(m, &r1, d.nv)) || (st = dalloc(m, &cv, d.nv))) {
      free_list(list);
      return st;
    }
    m->d32.R1 = r1;
    m->d32.cflv = cv;
  }
  tl.tbeg = tbeg;
  tl.vbeg = vbeg;
  tl.nvi = nvi;
  tl.lpb = lpb;
  tl.lp = lp;
  tl.tvl = tvl;
  tl.lv = lv;
  tl.dst = dst;
  tl.tmesh = m->voff.size() > 2 ? tm : nullptr;
  tl.sv = sv;
  tl.ssbeg = ssbeg;
  tl.Cs = cs;
  tl.lams = lams;
  replace(std::move(list), tl);
  return RD_OK;
}

// The FP32 step's own buffers, on first use (its state, signal speeds and CFL
// terms are the second view's, there from creation).
rd_status buffers32(rd_mesh* m) {
  rd::Dev32& h = m->d32;
  const int64_t nv = m->d.nv, nt = m->d.nt;
  rd_status st;
  if (!h.Zf) {
    rd::Dev32 n = h;  // the tiled form's buffers may be there
    rd::F4 *c, *kn, *kt;
    st = Block().add(&n.Zf, nv).add(&n.dW, nv).add(&kn, 2 * nt).add(&kt, nt).add(&c, m->d.ns).take(m);
    if (st != RD_OK) return st;
    n.C = c;
    n.keepN = kn;
    n.keepT = kt;
    h = n;
  }
  return RD_OK;
}

// The state into the form the steps about to run use: the FP32 form with its
// parameter vectors, or a patch buffer. One pass, where the last
// steps were of the other precision; after a capture the device decides.
rd_status enter(rd_mesh* m, int fp32) {
  rd_status st;
  note_capture(m);
  if (fp32 && (st = guarded([&] { return buffers32(m); })) != RD_OK) return st;
  if (!m->captured && (fp32 != 0) == m->form32) return RD_OK;
  hipStream_t s = m->stream;
  if (fp32) {
    HIPCHK(rd::launch_enter32(m->d, m->d32, state_of(m), s));
    HIPCHK(rd::launch_set_int(m->p.cur, rd::kForm32, s));
  } else {
    HIPCHK(rd::launch_patch_enter(m->p, state_of(m), s));
  }
  m->form32 = fp32 != 0;
  return RD_OK;
}

// Owned vertices per patch the library asks for: 215 (about 490 triangles, the
// 512 threads of a workgroup nearly full) on meshes with enough vertices to
// give every compute unit a patch, fewer on smaller ones so that the step is
// spread over the device, down to 48: below, the triangles shared with
// neighbouring patches outnumber the patch's own, and a pass is the latency of
// one patch anyway (RK2 step, us, with a least size of 16 / 32 / 48 / 64 / 128:
// 14.0 / 13.4 / 13.5 / 13.5 / 16.5 at 64^2, 15.3 / 15.3 / 13.8 / 13.7 / 16.5 at
// 100^2, 16.4 / 16.5 / 16.5 / 16.5 / 16.4 at 160^2).
int patch_own(int64_t nv, int ncu) {
  return (int)std::min<int64_t>(215, std::max<int64_t>(48, nv / std::max(1, ncu)));
}

constexpr int kPatchVertexBytes = 112;  // of LDS in the second stage

rd_status build_patches(rd_mesh* m, rd::Workers& pool) {
  rd::Patches& q = m->p;
  const int64_t nv = q.nv, nt = m->d.nt;
  rd::PatchPlan P;
  rd::PatchInput in;
  in.nv = nv;
  in.nt = nt;
  in.tri = m->tri.data();
  in.x = m->x.data();
  in.y = m->y.data();
  in.hpx = q.hpx;
  in.hpy = q.hpy;
  in.row = m->row.data();
  in.slot = m->slot.data();
  in.voff = &m->voff;
  in.toff = &m->toff;
  in.own = patch_own(nv, m->ncu);
  in.workers = &pool;
  std::string why = rd::build_patch_plan(in, P);
  // a vertex in more triangles than a workgroup has threads: its patch keeps
  // vertex records and parts apart in LDS, so the other patches are kept small
  if (why.empty() && P.max_tri > rd::kPatchThreads) {
    in.max_tri = rd::kPatchThreads / 2;
    why = rd::build_patch_plan(in, P);
  }
  if (!why.empty()) return fail(RD_EINVAL, why);
  rd::Patches p = q;
  p.ptn = (int64_t)P.tid.size();
  p.npatch = P.npatch;
  p.max_lv = P.max_lv;
  p.max_slots = P.max_slots;
  p.max_tri = P.max_tri;
  p.threads = std::min(rd::kPatchThreads, (P.max_tri + 63) / 64 * 64);
  // wide patches: the kernels' own shared words take less than 512 bytes, the
  // largest vertex's parts 32 bytes each
  const int32_t room = (m->lds_max - 512 - 32 * (kMaxDegree + 1)) / kPatchVertexBytes;
  p.all_lv = P.max_lv;
  std::vector<int32_t> wide;
  rd_status st;
  if (P.max_lv > room) {
    p.max_lv = 0;
    for (int32_t k = 0; k < P.npatch; ++k) {
      const int32_t lv = P.vbeg[k + 1] - P.vbeg[k] + P.hbeg[k + 1] - P.hbeg[k];
      if (lv > room) wide.push_back(k);
      else p.max_lv = std::max(p.max_lv, lv);
    }
    p.nloc = nv + (int64_t)P.halo.size();
    if ((st = dalloc(m, &p.rec, 3 * p.nloc)) || (st = dalloc(m, &p.rsig, p.nloc))) return st;
  }
  const size_t need = std::max(rd::patch_lds_bytes(p, 1, true), rd::patch_lds_bytes(p, 2, false));
  if (need > (size_t)m->lds_max)
    return fail(RD_EUNSUPPORTED, "patches of this mesh need " + std::to_string(need) + " bytes of LDS");
  // descriptors, geometry and boundary lists in internal order
  const rd::UVec<int32_t>& inv = P.inv;
  std::vector<rd::PatchDesc> desc(P.npatch);
  rd::UVec<double2> xy(nv + P.halo.size());
  rd::UVec<double> V(nv);
  pool.each(P.npatch, [&](int64_t k) {
    int64_t at = (int64_t)P.vbeg[k] + P.hbeg[k];
    rd::PatchDesc& d = desc[k];
    d = rd::PatchDesc();
    d.v0 = P.vbeg[k];
    d.own = P.vbeg[k + 1] - d.v0;
    d.h0 = P.hbeg[k];
    d.nlv = d.own + P.hbeg[k + 1] - d.h0;
    d.t0 = P.tbeg[k];
    d.nt = P.tbeg[k + 1] - d.t0;
    d.xy0 = (int32_t)at;
    d.mesh = P.pmesh[k];
    d.seam = P.seam[k];
    d.jb = P.jbeg[k];
    for (int j = 0; j < 8; ++j) d.jb8[j] = (uint16_t)(j < P.jbeg[k + 1] - P.jbeg[k] ? P.jb[P.jbeg[k] + j] : 0);
    for (int32_t l = 0; l < d.nlv; ++l) {
      const int32_t v = P.order[l < d.own ? d.v0 + l : P.halo[d.h0 + l - d.own]];
      xy[at++] = make_double2(m->x[v], m->y[v]);
    }
  });
  pool.each(nv, [&](int64_t i) { V[i] = m->ghost[P.order[i]] ? -m->V[P.order[i]] : m->V[P.order[i]]; });
  std::vector<int32_t> wb;
  std::vector<rd::WallEnt> went = m->went;
  if (!m->wv.empty()) {
    wb.assign(nv, -1);
    for (size_t b = 0; b < m->wv.size(); ++b)
      if (!m->ghost[m->wv[b]]) wb[inv[m->wv[b]]] = (int32_t)b;
    for (auto& e : went) e.other = inv[e.other];
  }
  int32_t *halo, *mbeg, *dinv, *dwb, *dwptr, *jb;
  rd::PatchDesc* ddesc;
  uint32_t* tri;
  uint16_t* deg;
  double2* dxy;
  double *dV, *pmin, *vpart;
  rd::WallEnt* dwent;
  if ((st = upload(m, &ddesc, desc)) || (st = upload(m, &halo, P.halo)) ||
      (st = upload(m, &mbeg, P.mbeg)) ||
      (st = upload(m, &dinv, inv)) || (st = upload(m, &tri, P.tri)) ||
      (st = upload(m, &deg, P.deg)) || (st = upload(m, &jb, P.jb)) || (st = upload(m, &dxy, xy)) ||
      (st = upload(m, &dV, V)) || (st = dalloc(m, &pmin, P.npatch)) ||
      (st = dalloc(m, &vpart, 2 * (size_t)P.npatch)) || (st = upload(m, &dwb, wb)) ||
      (st = upload(m, &dwptr, m->wptr)) || (st = upload(m, &dwent, went)))
    return st;
  p.desc = p.all = ddesc;
  if (!wide.empty()) {
    for (int32_t k : wide) desc[k].own = desc[k].nlv = desc[k].nt = 0;
    int32_t* dwide;
    rd::PatchDesc* rest;
    if ((st = upload(m, &dwide, wide)) || (st = upload(m, &rest, desc))) return st;
    p.nwide = (int32_t)wide.size();
    p.wide = dwide;
    p.desc = rest;
  }
  p.halo = halo;
  p.mbeg = mbeg;
  p.nmesh = (int32_t)m->voff.size() - 1;
  p.tri = tri;
  p.deg = deg;
  p.jb = jb;
  p.xy = dxy;
  p.V = dV;
  p.wb = wb.empty() ? nullptr : dwb;
  p.wptr = dwptr;
  p.went = dwent;
  p.pmin = pmin;
  p.vpart = vpart;
  m->p = p;
  m->inv = dinv;
  m->max_mesh_patches = 0;
  for (size_t k = 0; k + 1 < P.mbeg.size(); ++k)
    m->max_mesh_patches = std::max(m->max_mesh_patches, P.mbeg[k + 1] - P.mbeg[k]);
  return RD_OK;
}

// The tile size of the FP32 step. (The FP64 step always takes the patches,
// whose size the library chooses: cut to half the triangles of a 512-triangle
// tile they left the last of a workgroup's eight wavefronts empty, 2.36
// against 1.53 ms for two steps at 2048^2, state in and out.)
bool tile_in_range(int tt) { return tt == 0 || (tt >= 32 && tt <= 1024); }

rd_status set_tile(rd_mesh* m, int tt) {
  if (tt == m->tile) return RD_OK;
  if (!tile_in_range(tt)) return fail(RD_EINVAL, "tile size must be 0 or in [32, 1024]");
  DeviceGuard g(m->device);
  HIPCHK(hipStreamSynchronize(m->stream));
  return guarded([&] { return build_tiles(m, tt); });
}

rd_status check_step_args(int scheme, int time, int precision) {
  if (scheme < RD_N || scheme > RD_BX) return fail(RD_EINVAL, "unknown scheme");
  if (time != RD_EULER1 && time != RD_RK2) return fail(RD_EINVAL, "unknown time integration");
  if (precision != RD_FP64 && precision != RD_FP32_ACC64) return fail(RD_EINVAL, "unknown precision");
  return RD_OK;
}

}  // namespace

RD_API rd_status rd_mesh_validate(const rd_mesh_desc* desc) {
  return guarded([&] {
    rd::Workers pool(desc ? workers_for(desc->n_triangles) : 1);
    return check_desc(desc, nullptr, pool);
  });
}

namespace {

// A mesh of `voff.size() - 1` meshes laid end to end (vertex and triangle
// ranges voff, toff; empty: one mesh), with the domain size of each for the
// Bx sensor (empty: from the description).
rd_status create_mesh(const rd_mesh_desc* desc, hipStream_t stream, const std::vector<int64_t>& voff,
                      const std::vector<int64_t>& toff, const std::vector<double>& Ldom, rd_mesh** out) {
  HostGeom geo;
  rd::Workers pool(desc ? workers_for(desc->n_triangles) : 1);
  rd_status st = check_desc(desc, &geo, pool);
  if (st != RD_OK) return st;
  struct Drop {
    void operator()(rd_mesh* m) const {
      free_all(m);
      delete m;
    }
  };
  std::unique_ptr<rd_mesh, Drop> owner(new rd_mesh());
  rd_mesh* m = owner.get();
  m->stream = stream;
  if (hipGetDevice(&m->device) != hipSuccess ||
      hipDeviceGetAttribute(&m->ncu, hipDeviceAttributeMultiprocessorCount, m->device) != hipSuccess ||
      hipDeviceGetAttribute(&m->lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, m->device) != hipSuccess ||
      m->ncu <= 0 || m->lds_max <= 0)
    return fail(RD_EDEVICE, "no HIP device");
  const int64_t nv = desc->n_vertices, nt = desc->n_triangles;
  m->x.resize(nv);
  m->y.resize(nv);
  m->tri.resize(3 * nt);
  m->ghost.resize(nv);
  // copies of the description, its extent, and whether it has ghosts
  struct Seen {
    double x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    bool ghosts = false;
  };
  std::vector<Seen> seen(pool.size());
  pool.run([&](int q) {
    Seen s;
    const int64_t w = pool.size();
    for (int64_t i = nv * q / w; i < nv * (q + 1) / w; ++i) {
      const double x = m->x[i] = desc->x[i], y = m->y[i] = desc->y[i];
      s.x0 = std::min(s.x0, x);
      s.x1 = std::max(s.x1, x);
      s.y0 = std::min(s.y0, y);
      s.y1 = std::max(s.y1, y);
      m->ghost[i] = desc->ghost && desc->ghost[i] ? 1 : 0;
      s.ghosts = s.ghosts || m->ghost[i];
    }
    std::copy(desc->tri + 3 * (nt * q / w), desc->tri + 3 * (nt * (q + 1) / w), m->tri.begin() + 3 * (nt * q / w));
    seen[q] = s;
  });
  Seen all;
  for (const Seen& s : seen) {
    all.x0 = std::min(all.x0, s.x0);
    all.x1 = std::max(all.x1, s.x1);
    all.y0 = std::min(all.y0, s.y0);
    all.y1 = std::max(all.y1, s.y1);
    all.ghosts = all.ghosts || s.ghosts;
  }
  if (desc->n_wall_edges > 0) m->wall.assign(desc->wall_edges, desc->wall_edges + 2 * desc->n_wall_edges);
  m->px = desc->period_x;
  m->py = desc->period_y;
  m->gamma = desc->gamma;
  m->V.swap(geo.V);
  m->voff = voff.empty() ? std::vector<int64_t>{0, nv} : voff;
  m->toff = toff.empty() ? std::vector<int64_t>{0, nt} : toff;

  m->row.swap(geo.row);
  m->slot.swap(geo.slot);
  // boundary kinds and wall incidences (ascending edge id per vertex)
  if (m->wall.empty() && all.ghosts) {
    m->bc.resize(nv);
    pool.each(nv, [&](int64_t i) { m->bc[i] = m->ghost[i] ? -2 : -1; });
    m->wptr.push_back(0);
  } else if (!m->wall.empty()) {
    m->bc.resize(nv);
    // incidences per vertex, ascending edge id
    const int64_t nw = (int64_t)m->wall.size() / 2;
    std::vector<int32_t> wrow(nv + 1, 0);
    for (int32_t v : m->wall) wrow[v + 1]++;
    for (int64_t i = 0; i < nv; ++i) wrow[i + 1] += wrow[i];
    std::vector<rd::WallEnt> ents(2 * nw);
    {
      std::vector<int32_t> fill(wrow.begin(), wrow.end() - 1);
      for (int64_t e = 0; e < nw; ++e) {
        const int32_t a = m->wall[2 * e], b = m->wall[2 * e + 1];
        const double dx = unwrap_h(m->x[b] - m->x[a], m->px), dy = unwrap_h(m->y[b] - m->y[a], m->py);
        const double len = std::sqrt(dx * dx + dy * dy);
        ents[fill[a]++] = rd::WallEnt{b, 0, len / 2.0, dy / len, -dx / len};
        ents[fill[b]++] = rd::WallEnt{a, 1, len / 2.0, dy / len, -dx / len};
      }
    }
    m->wptr.push_back(0);
    for (int64_t i = 0; i < nv; ++i) {
      int32_t b = -1;
      if (wrow[i + 1] > wrow[i]) {
        b = (int32_t)m->wv.size();
        m->wv.push_back((int32_t)i);
        m->went.insert(m->went.end(), ents.begin() + wrow[i], ents.begin() + wrow[i + 1]);
        m->wptr.push_back((int32_t)m->went.size());
      }
      if (m->ghost[i]) m->bc[i] = b >= 0 ? -3 - b : -2;
      else m->bc[i] = b;
    }
  }

  rd::Patches& p = m->p;
  p.nv = nv;
  m->d.nv = nv;
  m->d.nt = nt;
  p.gamma = m->gamma;
  p.gas = rd::SymGas(m->gamma);
  p.px = m->px;
  p.py = m->py;
  p.hpx = m->px > 0.0 ? 0.5 * m->px : HUGE_VAL;
  p.hpy = m->py > 0.0 ? 0.5 * m->py : HUGE_VAL;
  // domain size L of the Bx sensor: the period on a periodic axis, else the coordinate extent
  {
    const double lx = m->px > 0.0 ? m->px : all.x1 - all.x0;
    const double ly = m->py > 0.0 ? m->py : all.y1 - all.y0;
    m->Ldom = std::max(lx, ly);
  }
  const size_t nmesh = m->voff.size() - 1;
  std::vector<double> vr0(3 * nmesh, 0.0);
  for (size_t k = 0; k < nmesh; ++k) vr0[3 * k + 2] = Ldom.empty() ? m->Ldom : Ldom[k];
  DeviceGuard g(m->device);
  rd::Dev& d = m->d;
  rd::D4 *W0, *W1, *D;
  int *cur, *flag;
  double *dt, *vr;
  m->staging = true;
  if ((st = Block().add(&W0, nv).add(&W1, nv).add(&D, nv).add(&m->scratch, 4 * nv).take(m)) ||
      (st = upload(m, &cur, std::vector<int>{0, 0})) || (st = upload(m, &m->done, std::vector<unsigned>{0})) ||
      (st = dalloc(m, &m->bad, 1)) || (st = upload(m, &flag, std::vector<int>(nmesh, 0))) || (st = dalloc(m, &dt, nmesh)) || (st = upload(m, &vr, vr0)))
    return st;
  p.W[0] = W0;
  p.W[1] = W1;
  p.D = D;
  p.cur = cur;
  p.flag = d.flag = flag;
  p.dt = d.dt = dt;
  p.vr = d.vr = vr;
  if ((st = build_view(m, pool)) != RD_OK) return st;
  rd::D4 *W, *Ws, *Z, *C, *kN, *kT, *wcn, *wcs;
  float* lam;
  st = Block().add(&W, nv).add(&Ws, nv).add(&Z, nv).add(&d.sig, nv).add(&lam, nt).add(&C, d.ns).add(&kN, 2 * nt)
           .add(&kT, nt).add(&wcn, m->wv.size()).add(&wcs, m->wv.size()).take(m);
  if (st != RD_OK) return st;
  d.W = W;
  d.lam = lam;
  d.Ws = Ws;
  d.Z = Z;
  d.C = C;
  d.keepN = kN;
  d.keepT = kT;
  d.WCn = wcn;
  d.WCs = wcs;
  if ((st = build_patches(m, pool)) != RD_OK || (st = flush_stage(m)) != RD_OK) return st;
  m->staging = false;
  rd::UVec<char>().swap(m->stage);
  hipError_t e = hipMemset(W0, 0, sizeof(rd::D4) * nv);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) return fail(RD_EDEVICE, std::string("initialising buffers: ") + hipGetErrorString(e));
  *out = owner.release();
  return RD_OK;
}

// Workspace of the allocation-free adjoint: every buffer starts on a 256-byte
// boundary.
struct NoallocLayout {
  size_t bytes = 0;
  size_t R2, R1, LamS, LamN, Zn, Wa, CZ, CZW, KN, KT;
  NoallocLayout(int64_t nv, int64_t nt, int64_t ns) {
    auto take = [&](size_t n) {
      const size_t at = bytes;
      bytes += (n + 255) & ~size_t(255);
      return at;
    };
    R2 = take(sizeof(rd::AdjRec2) * nv);
    R1 = take(sizeof(rd::AdjRec1) * nv);
    LamS = take(sizeof(rd::D4) * nv);
    LamN = take(sizeof(rd::D4) * nv);
    Zn = take(sizeof(rd::D4) * nv);
    Wa = take(sizeof(rd::D4) * nv);
    CZ = take(sizeof(rd::D4) * ns);
    CZW = take(sizeof(rd::ZW) * ns);
    KN = take(sizeof(rd::D4) * 2 * nt);
    KT = take(sizeof(rd::D4) * nt);
  }
};

}  // namespace

RD_API rd_status rd_mesh_create(const rd_mesh_desc* desc, void* stream, rd_mesh** out) {
  if (!out) return fail(RD_EINVAL, "null output pointer");
  *out = nullptr;
  return guarded([&] { return create_mesh(desc, static_cast<hipStream_t>(stream), {}, {}, {}, out); });
}

RD_API rd_status rd_mesh_destroy(rd_mesh* m) {
  if (!m) return RD_OK;
  DeviceGuard g(m->device);
  (void)hipStreamSynchronize(m->stream);
  for (hipEvent_t e : m->events)
    if (e) (void)hipEventDestroy(e);
  free_all(m);
  delete m;
  return RD_OK;
}

RD_API rd_status rd_mesh_info(const rd_mesh* m, int64_t* nv, int64_t* nt) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  if (nv) *nv = m->d.nv;
  if (nt) *nt = m->d.nt;
  return RD_OK;
}

RD_API rd_status rd_set_stream(rd_mesh* m, void* stream) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  m->stream = static_cast<hipStream_t>(stream);
  return RD_OK;
}

RD_API rd_status rd_set_state(rd_mesh* m, const double* W, int on_device) {
  if (!m || !W) return fail(RD_EINVAL, "null argument");
  DeviceGuard g(m->device);
  const int64_t nv = m->d.nv;
  hipStream_t s = m->stream;
  const double* src = W;
  const int* bad = nullptr;
  int64_t first = nv;
  auto status = [&] {
    return first == nv ? RD_OK
                       : fail(RD_ENONPHYS, "vertex " + std::to_string(first) +
                                               " has rho <= 0, p <= 0 or a non-finite value");
  };
  if (!on_device) {
    if (nv <= kHostCheck2 && (first = first_unphysical(W, nv, 2, m->gamma)) < nv) return status();
    HIPCHK(hipMemcpyAsync(m->scratch, W, sizeof(double) * 4 * nv, hipMemcpyHostToDevice, s));
    src = m->scratch;
  }
  if (!on_device && nv > kHostCheck2) {
    bad = m->bad;
    HIPCHK(rd::launch_check_state(src, nv, 2, m->gamma, m->bad, s));
    HIPCHK(rd::launch_clear_unless(m->p.flag, bad, nv, s));
  } else {
    HIPCHK(rd::launch_set_int(m->p.flag, 0, s));
  }
  // into the form of the last steps
  note_capture(m);
  if (m->form32) HIPCHK(rd::launch_set32(m->d, m->d32, m->p.cur, src, bad, s));
  else HIPCHK(rd::launch_patch_set(m->p, m->inv, src, bad, s));
  if (on_device) return RD_OK;
  // a host state is in place when the call returns
  int named = INT_MAX;
  if (bad) HIPCHK(hipMemcpyAsync(&named, bad, sizeof(int), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  first = std::min<int64_t>(named, nv);
  return status();
}

RD_API rd_status rd_get_state(rd_mesh* m, double* W, int on_device) {
  if (!m || !W) return fail(RD_EINVAL, "null argument");
  DeviceGuard g(m->device);
  const int64_t nv = m->d.nv;
  if (on_device) {
    HIPCHK(rd::launch_state_get(state_of(m), nv, W, m->stream));
    return RD_OK;
  }
  HIPCHK(rd::launch_state_get(state_of(m), nv, m->scratch, m->stream));
  HIPCHK(hipMemcpyAsync(W, m->scratch, sizeof(double) * 4 * nv, hipMemcpyDeviceToHost, m->stream));
  int flag = 0;
  HIPCHK(hipMemcpyAsync(&flag, m->p.flag, sizeof(int), hipMemcpyDeviceToHost, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  if (flag) return fail(RD_ENONPHYS, "a non-physical state was produced");
  return RD_OK;
}

RD_API rd_status rd_max_dt(rd_mesh* m, double cfl, double* dt_out) {
  if (!m || !dt_out) return fail(RD_EINVAL, "null argument");
  if (!(cfl > 0.0)) return fail(RD_EINVAL, "cfl must be positive");
  DeviceGuard g(m->device);
  // The bounds are those of the FP64 passes whatever steps ran before. A state
  // in the FP32 form stays there, for the steps that follow: a copy is read.
  note_capture(m);
  if (m->form32 || m->captured) HIPCHK(rd::launch_patch_copy(m->p, state_of(m), m->stream));
  // The device writes the result into host memory: a wait then gives it, where
  // a copy behind the kernels costs 10 us more at 49^2. A mesh's first call takes
  // the copy, since to allocate that memory costs 30 us. Up to kDirectPatches
  // patches the last workgroup takes the minimum itself (their count goes
  // through one word, which many more would queue for).
  if (m->asked && !m->host_dt) {
    void* q = nullptr;
    HIPCHK(hipHostMalloc(&q, sizeof(double), hipHostMallocDefault));
    m->host_dt = static_cast<double*>(q);
  }
  m->asked = true;
  double* const to = m->host_dt ? m->host_dt : m->scratch;
  const bool one = m->p.npatch <= kDirectPatches;
  HIPCHK(rd::launch_patch_cfl(m->p, cfl, one ? m->done : nullptr, to, m->stream));
  if (!one) HIPCHK(rd::launch_patch_dt(m->p, cfl, m->stream, to));
  if (!m->host_dt) HIPCHK(hipMemcpyAsync(dt_out, to, sizeof(double), hipMemcpyDeviceToHost, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  if (m->host_dt) *dt_out = *const_cast<volatile double*>(m->host_dt);
  return RD_OK;
}

RD_API rd_status rd_step(rd_mesh* m, double dt, int scheme, int time, int precision) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  if (!(dt > 0.0) || !std::isfinite(dt)) return fail(RD_EINVAL, "dt must be positive and finite");
  rd_status st = check_step_args(scheme, time, precision);
  if (st != RD_OK) return st;
  DeviceGuard g(m->device);
  if ((st = enter(m, precision == RD_FP32_ACC64)) != RD_OK) return st;
  return run_step(m, scheme, time, precision == RD_FP32_ACC64, 0.0, dt);
}

RD_API rd_status rd_step_cfl(rd_mesh* m, int n_steps, double cfl, int scheme, int time, int precision) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  if (n_steps < 0) return fail(RD_EINVAL, "negative step count");
  if (!(cfl > 0.0)) return fail(RD_EINVAL, "cfl must be positive");
  rd_status st = check_step_args(scheme, time, precision);
  if (st != RD_OK) return st;
  DeviceGuard g(m->device);
  if ((st = enter(m, precision == RD_FP32_ACC64)) != RD_OK) return st;
  return run_steps(m, n_steps, scheme, time, precision == RD_FP32_ACC64, cfl);
}

RD_API rd_status rd_step_timed(rd_mesh* m, double cfl, int scheme, int time, int precision, double* ms) {
  if (!m || !ms) return fail(RD_EINVAL, "null argument");
  if (!(cfl > 0.0)) return fail(RD_EINVAL, "cfl must be positive");
  rd_status st = check_step_args(scheme, time, precision);
  if (st != RD_OK) return st;
  DeviceGuard g(m->device);
  const int fp32 = precision == RD_FP32_ACC64;
  if ((st = enter(m, fp32)) != RD_OK) return st;
  if (!m->events[0])
    for (int k = 0; k <= RD_NKERNELS; ++k) HIPCHK(hipEventCreate(&m->events[k]));
  hipEvent_t* ev = m->events;
  if ((st = run_step(m, scheme, time, fp32, cfl, 0.0, ev)) != RD_OK) return st;
  HIPCHK(hipEventSynchronize(ev[RD_NKERNELS]));
  for (int k = 0; k < RD_NKERNELS; ++k) {
    float t = 0.0f;
    HIPCHK(hipEventElapsedTime(&t, ev[k], ev[k + 1]));
    ms[k] = t;
  }
  return RD_OK;
}

RD_API rd_status rd_mesh_set_tile(rd_mesh* m, int tile_triangles) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  return set_tile(m, tile_triangles);
}

RD_API rd_status rd_mesh_get_tile(const rd_mesh* m, int* tile_triangles) {
  if (!m || !tile_triangles) return fail(RD_EINVAL, "null argument");
  *tile_triangles = m->tile;
  return RD_OK;
}

RD_API rd_status rd_mesh_set_lumping(rd_mesh* m, int lumping) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  if (lumping != RD_LUMP_GLOBAL && lumping != RD_LUMP_SELECTIVE) return fail(RD_EINVAL, "unknown lumping");
  m->p.slump = lumping == RD_LUMP_SELECTIVE;
  return RD_OK;
}

RD_API rd_status rd_mesh_get_lumping(const rd_mesh* m, int* lumping) {
  if (!m || !lumping) return fail(RD_EINVAL, "null argument");
  *lumping = m->p.slump ? RD_LUMP_SELECTIVE : RD_LUMP_GLOBAL;
  return RD_OK;
}

RD_API rd_status rd_mesh_tile_info(const rd_mesh* m, int64_t* info) {
  if (!m || !info) return fail(RD_EINVAL, "null argument");
  for (int k = 0; k < 4; ++k) info[k] = m->tile_info[k];
  return RD_OK;
}

namespace {

const int kTuneDefault[] = {0, 64, 128, 256, 512};
// A later candidate replaces the one kept so far only when it is faster by
// more than this fraction (the run-to-run spread of one timing is about 1-2%),
// so the tuner does not switch forms on noise.
constexpr float kTuneMargin = 0.02f;

rd_status tune_args(double cfl, int scheme, int time, int precision, int n_steps, const int*& cand, int& nc,
                    int* best) {
  if (!best) return fail(RD_EINVAL, "null argument");
  if (!(cfl > 0.0)) return fail(RD_EINVAL, "cfl must be positive");
  if (n_steps < 1) return fail(RD_EINVAL, "n_steps must be at least 1");
  if (!cand) {
    cand = kTuneDefault;
    nc = (int)(sizeof(kTuneDefault) / sizeof(kTuneDefault[0]));
  }
  if (nc < 1) return fail(RD_EINVAL, "no candidates");
  return check_step_args(scheme, time, precision);
}

// Times `body` (enqueued on s) with two events; returns milliseconds.
template <class F>
rd_status time_on(hipStream_t s, F body, float* ms) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HIPCHK(hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return fail(RD_EDEVICE, "hipEventCreate failed");
  }
  rd_status st = RD_OK;
  hipError_t e = hipEventRecord(e0, s);
  if (e == hipSuccess) st = body();
  if (e == hipSuccess && st == RD_OK) e = hipEventRecord(e1, s);
  if (e == hipSuccess && st == RD_OK) e = hipEventSynchronize(e1);
  if (e == hipSuccess && st == RD_OK) e = hipEventElapsedTime(ms, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (st != RD_OK) return st;
  if (e != hipSuccess) return fail(RD_EDEVICE, std::string("timing: ") + hipGetErrorString(e));
  return RD_OK;
}

}  // namespace

RD_API rd_status rd_tune(rd_mesh* m, double cfl, int scheme, int time, int precision, int n_steps,
                         const int* candidates, int n_candidates, double* ms_per_step, int* best) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  rd_status st = tune_args(cfl, scheme, time, precision, n_steps, candidates, n_candidates, best);
  if (st != RD_OK) return st;
  DeviceGuard g(m->device);
  const int fp32 = precision == RD_FP32_ACC64;
  hipStream_t s = m->stream;
  // the state (in the caller's order) and the flag are saved
  rd::D4* saveW = reinterpret_cast<rd::D4*>(m->scratch);
  HIPCHK(rd::launch_state_get4(state_of(m), m->p.nv, saveW, s));
  int flag0 = 0;
  HIPCHK(hipMemcpyAsync(&flag0, m->p.flag, sizeof(int), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  auto restore = [&]() -> rd_status {
    HIPCHK(rd::launch_patch_set4(m->p, m->inv, saveW, s));
    HIPCHK(rd::launch_set_int(m->p.cur, 0, s));
    HIPCHK(rd::launch_set_int(m->p.flag, flag0, s));
    m->form32 = false;
    return RD_OK;
  };
  const int prev = m->tile;
  int pick = -1;
  float pick_ms = 0.0f;
  for (int i = 0; i < n_candidates; ++i) {
    if (ms_per_step) ms_per_step[i] = -1.0;
    if (!fp32 && pick >= 0) {  // the FP64 step has one form: its time stands for every size
      if (ms_per_step && tile_in_range(candidates[i])) ms_per_step[i] = pick_ms / n_steps;
      continue;
    }
    st = set_tile(m, candidates[i]);
    if (st == RD_EUNSUPPORTED || st == RD_EINVAL) continue;
    if (st != RD_OK) break;
    if ((st = enter(m, fp32)) != RD_OK || (st = run_step(m, scheme, time, fp32, cfl, 0.0)) != RD_OK) break;
    float t = 0.0f;
    st = time_on(s, [&]() -> rd_status {
      for (int k = 0; k < n_steps; ++k) {
        rd_status r = run_step(m, scheme, time, fp32, cfl, 0.0);
        if (r != RD_OK) return r;
      }
      return RD_OK;
    }, &t);
    if (st != RD_OK) break;
    if ((st = restore()) != RD_OK) break;
    if (ms_per_step) ms_per_step[i] = t / n_steps;
    if (pick < 0 || t < pick_ms * (1.0f - kTuneMargin)) {
      pick = candidates[i];
      pick_ms = t;
    }
  }
  if (st == RD_EUNSUPPORTED || st == RD_EINVAL) st = RD_OK;
  rd_status st2 = set_tile(m, pick >= 0 ? pick : prev);
  rd_status st3 = restore();
  HIPCHK(hipStreamSynchronize(s));
  if (st != RD_OK) return st;
  if (st2 != RD_OK) return st2;
  if (st3 != RD_OK) return st3;
  if (pick < 0) return fail(RD_EUNSUPPORTED, "no candidate tile size is usable");
  *best = pick;
  return RD_OK;
}

RD_API rd_status rd_residual(rd_mesh* m, int scheme, double* R, double* phiT, int on_device) {
  if (!m || !R) return fail(RD_EINVAL, "null argument");
  if (scheme < RD_N || scheme > RD_BX) return fail(RD_EINVAL, "unknown scheme");
  DeviceGuard g(m->device);
  rd_status st;
  if ((st = enter(m, 0)) != RD_OK) return st;
  const rd::Dev& d = m->d;
  hipStream_t s = m->stream;
  const int64_t nv = d.nv, nt = d.nt;
  if (!on_device && phiT && !m->phi_scratch && (st = dalloc(m, &m->phi_scratch, 4 * nt)) != RD_OK) return st;
  if (scheme == RD_BX) HIPCHK(rd::launch_patch_vrange(m->p, false, s));
  HIPCHK(rd::launch_patch_residual(m->p, scheme, s));
  const rd::State res{{m->p.D, m->p.D}, m->p.cur, m->inv, nullptr};
  double* phi = !phiT || on_device ? phiT : m->phi_scratch;
  HIPCHK(rd::launch_residual(d, res, on_device ? R : m->scratch, state_of(m), phi, s));
  if (on_device) return RD_OK;
  HIPCHK(hipMemcpyAsync(R, m->scratch, sizeof(double) * 4 * nv, hipMemcpyDeviceToHost, s));
  if (phiT) HIPCHK(hipMemcpyAsync(phiT, m->phi_scratch, sizeof(double) * 4 * nt, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  return RD_OK;
}

namespace {

// Waits for the mesh's stream and reports (then clears) the adjoint's latches:
// a non-physical recomputed step, or a triangle whose solve skipped a column.
rd_status adjoint_status(rd_mesh* m) {
  int flag[2] = {0, 0};
  if (m->adj.flag) HIPCHK(hipMemcpyAsync(flag, m->adj.flag, sizeof(flag), hipMemcpyDeviceToHost, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  if (!flag[0] && !flag[1]) return RD_OK;
  HIPCHK(rd::launch_set_int(m->adj.flag, 0, m->stream));
  HIPCHK(rd::launch_set_int(m->adj.flag + 1, 0, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  if (flag[0]) return fail(RD_ENONPHYS, "the adjoint's input state W_n or its recomputed first stage is non-physical");
  return fail(RD_EUNSUPPORTED,
              "the adjoint met a triangle whose pivoted solve skipped a column (exact stagnation, Section 3.3.1); "
              "the gradient of that branch is not computed");
}

}  // namespace

namespace {

rd_status adjoint_args(rd_mesh* m, double dt, int scheme, int time) {
  if (!(dt > 0.0) || !std::isfinite(dt)) return fail(RD_EINVAL, "dt must be positive and finite");
  rd_status st = check_step_args(scheme, time, RD_FP64);
  if (st != RD_OK) return st;
  if (scheme == RD_BX) return fail(RD_EUNSUPPORTED, "the adjoint does not cover the Bx scheme");
  if (m->p.slump && time == RD_RK2)
    return fail(RD_EUNSUPPORTED, "the adjoint does not cover selective lumping");
  return RD_OK;
}

// Enqueues the reverse of one step on the mesh's stream, all pointers on the
// device: the step from W_n is recomputed on the buffers of `a` (W^n copy Wa,
// latches a.flag) and the mesh's stage buffers; the mesh's own state, signal
// speeds and latch are not touched.
rd_status adjoint_enqueue(rd_mesh* m, const rd::AdjDev& a, rd::D4* Wa, const double* W_n, double dt, int scheme,
                          int time, const double* lam_np1, double* lam_n) {
  hipStream_t s = m->stream;
  rd::Dev d = m->d;
  d.W = Wa;
  d.flag = a.flag;
  // parameter vectors at W^n go straight to Zn (read by the stage-1 passes and
  // the adjoint); the first-stage vertex pass writes W* and the stage-2
  // reverse records
  rd::Dev dn = d;
  dn.Z = a.Zn;
  rd::AdjDev ad = a;
  ad.lam = rd::LamSoA{lam_np1, m->d.nv};  // read in the caller's layout
  ad.idt = 1.0 / dt;
  ad.waves = rd::kAdjWavesPerCu * m->ncu;
  HIPCHK(rd::launch_set_state(dn, W_n, dt, s));
  const bool rk2 = time == RD_RK2;
  if (rk2) {
    HIPCHK(rd::launch_wall(dn, false, s));
    HIPCHK(rd::launch_tri(dn, scheme, s));
    HIPCHK(rd::launch_adj_star(d, ad, s));
  }
  HIPCHK(rd::launch_adjoint(d, ad, scheme, rk2 ? 1 : 0, lam_n, s));
  return RD_OK;
}

}  // namespace

RD_API rd_status rd_adjoint_step(rd_mesh* m, const double* W_n, double dt, int scheme, int time,
                                 const double* lam_np1, double* lam_n, int on_device) {
  if (!m || !W_n || !lam_np1 || !lam_n) return fail(RD_EINVAL, "null argument");
  rd_status st = adjoint_args(m, dt, scheme, time);
  if (st != RD_OK) return st;
  DeviceGuard g(m->device);
  const int64_t nv = m->d.nv, nt = m->d.nt;
  if (!m->adjW) {
    rd::AdjDev& a = m->adj;
    rd::D4 *lamS, *lamN, *Zn, *cZ, *kN, *kT, *Wa;
    rd::ZW* cZW;
    rd::AdjRec2* r2;
    rd::AdjRec1* r1;
    double *in, *out;
    int* flag;
    st = Block().add(&lamS, nv).add(&lamN, nv).add(&r2, nv).add(&r1, nv).add(&Zn, nv).add(&cZ, m->d.ns)
             .add(&cZW, m->d.ns).add(&kN, 2 * nt).add(&kT, nt).add(&Wa, nv).add(&in, 4 * nv).add(&out, 4 * nv)
             .add(&flag, 2).take(m);
    if (st != RD_OK) return st;
    HIPCHK(rd::launch_set_int(flag, 0, m->stream));
    HIPCHK(rd::launch_set_int(flag + 1, 0, m->stream));
    a.flag = flag;
    a.lamS = lamS;
    a.lamN = lamN;
    a.r2 = r2;
    a.r1 = r1;
    a.Zn = Zn;
    a.cZ = cZ;
    a.cZW = cZW;
    a.kN = kN;
    a.kT = kT;
    m->adjW = Wa;
    m->adjIn = in;
    m->adjOut = out;
  }
  hipStream_t s = m->stream;
  const double* src = W_n;
  if (!on_device) {
    HIPCHK(hipMemcpyAsync(m->adjIn, W_n, sizeof(double) * 4 * nv, hipMemcpyHostToDevice, s));
    src = m->adjIn;
  }
  // dL/dW^n is written back to adjIn: its copy of W^n is consumed by the first
  // kernel of the recomputation, which runs before (stream order)
  const double* lsrc = lam_np1;
  if (!on_device) {
    HIPCHK(hipMemcpyAsync(m->adjOut, lam_np1, sizeof(double) * 4 * nv, hipMemcpyHostToDevice, s));
    lsrc = m->adjOut;
  }
  double* out = on_device ? lam_n : m->adjIn;
  if ((st = adjoint_enqueue(m, m->adj, m->adjW, src, dt, scheme, time, lsrc, out)) != RD_OK) return st;
  if (!on_device) {
    HIPCHK(hipMemcpyAsync(lam_n, m->adjIn, sizeof(double) * 4 * nv, hipMemcpyDeviceToHost, s));
    return adjoint_status(m);
  }
  return RD_OK;
}

RD_API rd_status rd_adjoint_step_noalloc(rd_mesh* m, const double* W_n, double dt, int scheme, int time,
                                         const double* lam_np1, double* lam_n, int* flags) {
  if (!m || !W_n || !lam_np1 || !lam_n || !flags) return fail(RD_EINVAL, "null argument");
  rd_status st = adjoint_args(m, dt, scheme, time);
  if (st != RD_OK) return st;
  const int64_t nv = m->p.nv, nt = m->d.nt, ns = m->d.ns;
  const NoallocLayout o(nv, nt, ns);
  if (o.bytes > rd::kNoallocScratchBytes)
    return fail(RD_EINVAL, "mesh too large for the allocation-free adjoint: it needs " + std::to_string(o.bytes) +
                               " bytes of workspace, the fixed workspace holds " +
                               std::to_string(rd::kNoallocScratchBytes));
  DeviceGuard g(m->device);
  void* base = nullptr;
  HIPCHK(rd::noalloc_scratch(&base));
  char* p = static_cast<char*>(base);
  rd::AdjDev a;
  a.r2 = reinterpret_cast<rd::AdjRec2*>(p + o.R2);
  a.r1 = reinterpret_cast<rd::AdjRec1*>(p + o.R1);
  a.lamS = reinterpret_cast<rd::D4*>(p + o.LamS);
  a.lamN = reinterpret_cast<rd::D4*>(p + o.LamN);
  a.Zn = reinterpret_cast<rd::D4*>(p + o.Zn);
  a.cZ = reinterpret_cast<rd::D4*>(p + o.CZ);
  a.cZW = reinterpret_cast<rd::ZW*>(p + o.CZW);
  a.kN = reinterpret_cast<rd::D4*>(p + o.KN);
  a.kT = reinterpret_cast<rd::D4*>(p + o.KT);
  a.flag = flags;
  // the latches start cleared on every call (a fill kernel, so the call can be captured)
  HIPCHK(rd::launch_fill_int(flags, 0, 2, m->stream));
  return adjoint_enqueue(m, a, reinterpret_cast<rd::D4*>(p + o.Wa), W_n, dt,
                         scheme, time, lam_np1, lam_n);
}

// ------------------------------------------------------------- batches --
//
// A batch lays its meshes end to end as one disjoint mesh (vertex and
// triangle ids offset in order), adds a mesh id per vertex and per triangle so
// every kernel reads its own mesh's time step, and reduces the CFL limit per
// mesh over vertex blocks that never straddle two meshes. n steps are
// captured once into a HIP graph and replayed; the members' states are
// copied in before and out after.

struct rd_batch {
  rd_mesh* flat = nullptr;
  std::vector<rd_mesh*> members;
  std::vector<int64_t> voff, toff;
  // the copy of the members' states in and out: one launch over blocks of one member's vertices
  rd::PatchMember* mem = nullptr;
  int32_t *mb = nullptr, *vb = nullptr;
  int nblocks = 0;
  hipStream_t stream = nullptr;  // the caller's stream
  hipStream_t own = nullptr;     // the batch's own stream (a null stream cannot be captured)
  hipEvent_t ev_in = nullptr, ev_out = nullptr;
  struct Graph {
    int n_steps, scheme, time, fp32, slump;
    double cfl;
    hipGraph_t graph;
    hipGraphExec_t exec;
  };
  std::vector<Graph> graphs;
};

namespace {

void destroy_graphs(rd_batch* b) {
  for (auto& g : b->graphs) {
    (void)hipGraphExecDestroy(g.exec);
    (void)hipGraphDestroy(g.graph);
  }
  b->graphs.clear();
}

}  // namespace

static rd_status batch_create(rd_mesh* const* meshes, int n, void* stream, rd_batch** out) {
  if (!meshes || n <= 0) return fail(RD_EINVAL, "empty batch");
  const double gamma = meshes[0] ? meshes[0]->gamma : 0.0;
  // The batch unwraps triangles with one period per axis: the members that
  // are periodic on an axis must share their period there. A member that is
  // not periodic on that axis is laid out as it is; unwrapping leaves its
  // triangles and wall edges alone when every coordinate difference along
  // them is at most half the period, and its tiles' centroids (strictly
  // inside its extent) stay put when that extent is at most the period (both
  // checked).
  double bp[2] = {0.0, 0.0};
  for (int k = 0; k < n; ++k) {
    const rd_mesh* m = meshes[k];
    if (!m) return fail(RD_EINVAL, "null mesh in batch");
    const double mp[2] = {m->px, m->py};
    for (int a = 0; a < 2; ++a)
      if (mp[a] > 0.0) {
        if (bp[a] == 0.0) bp[a] = mp[a];
        else if (mp[a] != bp[a])
          return fail(RD_EINVAL, "batched meshes periodic on the same axis must share the period");
      }
  }
  for (int k = 0; k < n; ++k) {
    const rd_mesh* m = meshes[k];
    const double mp[2] = {m->px, m->py};
    const rd::UVec<double>* c[2] = {&m->x, &m->y};
    for (int a = 0; a < 2; ++a) {
      if (bp[a] == 0.0 || mp[a] > 0.0) continue;
      const rd::UVec<double>& q = *c[a];
      const auto r = std::minmax_element(q.begin(), q.end());
      bool ok = *r.second - *r.first <= bp[a];
      for (size_t t = 0; ok && t < m->tri.size(); t += 3)
        for (int i = 1; i < 3; ++i) ok = ok && std::fabs(q[m->tri[t + i]] - q[m->tri[t]]) <= 0.5 * bp[a];
      for (size_t e = 0; ok && e < m->wall.size(); e += 2)
        ok = std::fabs(q[m->wall[e + 1]] - q[m->wall[e]]) <= 0.5 * bp[a];
      if (!ok)
        return fail(RD_EINVAL, "batched mesh " + std::to_string(k) + " is not periodic on an axis where others are, "
                               "and its extent or a triangle's extent along that axis is too large for their period");
    }
  }
  std::vector<double> x, y;
  std::vector<int32_t> tri, wall;
  std::vector<uint8_t> ghost;
  std::vector<int64_t> voff{0}, toff{0};
  for (int k = 0; k < n; ++k) {
    const rd_mesh* m = meshes[k];
    if (m->gamma != gamma) return fail(RD_EINVAL, "batched meshes must share gamma");
    if (m->device != meshes[0]->device) return fail(RD_EINVAL, "batched meshes must live on one device");
    const int32_t vo = (int32_t)voff.back();
    x.insert(x.end(), m->x.begin(), m->x.end());
    y.insert(y.end(), m->y.begin(), m->y.end());
    for (int32_t v : m->tri) tri.push_back(v + vo);
    for (int32_t v : m->wall) wall.push_back(v + vo);
    ghost.insert(ghost.end(), m->ghost.begin(), m->ghost.end());
    voff.push_back(voff.back() + m->d.nv);
    toff.push_back(toff.back() + m->d.nt);
  }
  if (voff.back() >= (int64_t(1) << 31) || 3 * toff.back() >= (int64_t(1) << 31))
    return fail(RD_EINVAL, "batch too large for 32-bit indices");
  rd_mesh_desc desc{};
  desc.n_vertices = voff.back();
  desc.n_triangles = toff.back();
  desc.x = x.data();
  desc.y = y.data();
  desc.tri = tri.data();
  desc.period_x = bp[0];
  desc.period_y = bp[1];
  desc.ghost = ghost.data();
  desc.n_wall_edges = (int64_t)wall.size() / 2;
  desc.wall_edges = wall.empty() ? nullptr : wall.data();
  desc.gamma = gamma;
  // blocks of the member copies
  std::vector<int32_t> mb, vb;
  for (int k = 0; k < n; ++k)
    for (int64_t v = 0; v < meshes[k]->p.nv; v += rd::kBlock) {
      mb.push_back(k);
      vb.push_back((int32_t)v);
    }
  std::unique_ptr<rd_batch> owner(new rd_batch());
  rd_batch* b = owner.get();
  b->members.assign(meshes, meshes + n);
  b->voff = voff;
  b->toff = toff;
  std::vector<double> Ldom(n);
  for (int k = 0; k < n; ++k) Ldom[k] = meshes[k]->Ldom;  // each member's own domain size
  DeviceGuard g(meshes[0]->device);
  hipStream_t own = nullptr;
  hipEvent_t ev_in = nullptr, ev_out = nullptr;
  HIPCHK(hipStreamCreateWithFlags(&own, hipStreamNonBlocking));
  if (hipEventCreateWithFlags(&ev_in, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&ev_out, hipEventDisableTiming) != hipSuccess) {
    (void)hipStreamDestroy(own);
    return fail(RD_EDEVICE, "hipEventCreate failed");
  }
  rd_mesh* flat = nullptr;
  rd_status st = guarded([&] { return create_mesh(&desc, own, voff, toff, Ldom, &flat); });
  if (st != RD_OK) {
    (void)hipEventDestroy(ev_in);
    (void)hipEventDestroy(ev_out);
    (void)hipStreamDestroy(own);
    return st;
  }
  std::vector<rd::PatchMember> mem;
  for (int k = 0; k < n; ++k) {
    const rd_mesh* m = meshes[k];
    mem.push_back(rd::PatchMember{state_of(m), m->p.cur, m->p.flag, (int32_t)m->p.nv, (int32_t)voff[k]});
  }
  if ((st = upload(flat, &b->mem, mem)) || (st = upload(flat, &b->mb, mb)) || (st = upload(flat, &b->vb, vb))) {
    rd_mesh_destroy(flat);
    (void)hipEventDestroy(ev_in);
    (void)hipEventDestroy(ev_out);
    (void)hipStreamDestroy(own);
    return st;
  }
  b->nblocks = (int)mb.size();
  b->flat = flat;
  b->stream = static_cast<hipStream_t>(stream);
  b->own = own;
  b->ev_in = ev_in;
  b->ev_out = ev_out;
  (void)owner.release();
  *out = b;
  return RD_OK;
}

RD_API rd_status rd_batch_create(rd_mesh* const* meshes, int n, void* stream, rd_batch** out) {
  if (!out) return fail(RD_EINVAL, "null output pointer");
  *out = nullptr;
  return guarded([&] { return batch_create(meshes, n, stream, out); });
}

namespace {

// Orders the batch's stream after the caller's and the members' pending work
// and copies the members' states in.
rd_status batch_begin(rd_batch* b, int fp32, std::vector<hipStream_t>& outer) {
  rd_mesh* f = b->flat;
  // the members' lumping, which must agree
  for (rd_mesh* m : b->members)
    if (m->p.slump != b->members[0]->p.slump)
      return fail(RD_EINVAL, "the meshes of a batch use different lumpings");
  f->p.slump = b->members[0]->p.slump;
  hipStream_t s = f->stream;  // the batch's own stream
  outer.assign(1, b->stream);
  for (rd_mesh* m : b->members)
    if (std::find(outer.begin(), outer.end(), m->stream) == outer.end()) outer.push_back(m->stream);
  for (hipStream_t o : outer) {
    HIPCHK(hipEventRecord(b->ev_in, o));
    HIPCHK(hipStreamWaitEvent(s, b->ev_in, 0));
  }
  HIPCHK(rd::launch_patch_members(state_of(f), f->p.cur, f->p.flag, f->p.nv, b->mem, b->mb, b->vb, b->nblocks, false,
                                  s));
  f->form32 = false;
  return enter(f, fp32);
}

// The captured graph of n_steps steps (cached per configuration; the cache
// is dropped whenever the tile size changes).
rd_status batch_graph(rd_batch* b, int n_steps, double cfl, int scheme, int time, int fp32,
                      hipGraphExec_t* exec) {
  rd_mesh* f = b->flat;
  hipStream_t s = f->stream;
  for (auto& c : b->graphs)
    if (c.n_steps == n_steps && c.scheme == scheme && c.time == time && c.fp32 == fp32 && c.cfl == cfl &&
        c.slump == f->p.slump) {
      *exec = c.exec;
      return RD_OK;
    }
  rd_batch::Graph c{n_steps, scheme, time, fp32, f->p.slump, cfl, nullptr, nullptr};
  HIPCHK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  rd_status rs = RD_OK;
  rs = run_steps(f, n_steps, scheme, time, fp32, cfl);
  hipError_t ce = hipStreamEndCapture(s, &c.graph);
  if (rs != RD_OK) {
    if (ce == hipSuccess) (void)hipGraphDestroy(c.graph);
    return rs;
  }
  if (ce != hipSuccess) return fail(RD_EDEVICE, std::string("graph capture: ") + hipGetErrorString(ce));
  hipError_t ie = hipGraphInstantiate(&c.exec, c.graph, nullptr, nullptr, 0);
  if (ie != hipSuccess) {
    (void)hipGraphDestroy(c.graph);
    return fail(RD_EDEVICE, std::string("graph instantiate: ") + hipGetErrorString(ie));
  }
  b->graphs.push_back(c);
  *exec = c.exec;
  return RD_OK;
}

rd_status batch_set_tile(rd_batch* b, int tt) {
  if (tt == b->flat->tile) return RD_OK;
  DeviceGuard g(b->flat->device);
  (void)hipStreamSynchronize(b->own);
  destroy_graphs(b);
  return set_tile(b->flat, tt);
}

}  // namespace

RD_API rd_status rd_batch_run(rd_batch* b, int n_steps, double cfl, int scheme, int time, int precision) {
  if (!b) return fail(RD_EINVAL, "null batch");
  if (n_steps < 0) return fail(RD_EINVAL, "negative step count");
  if (!(cfl > 0.0)) return fail(RD_EINVAL, "cfl must be positive");
  rd_status st = check_step_args(scheme, time, precision);
  if (st != RD_OK) return st;
  rd_mesh* f = b->flat;
  DeviceGuard g(f->device);
  const int fp32 = precision == RD_FP32_ACC64;
  hipStream_t s = f->stream;
  std::vector<hipStream_t> outer;
  if ((st = batch_begin(b, fp32, outer)) != RD_OK) return st;
  if (n_steps > 0) {
    hipGraphExec_t exec = nullptr;
    if ((st = batch_graph(b, n_steps, cfl, scheme, time, fp32, &exec)) != RD_OK) return st;
    HIPCHK(hipGraphLaunch(exec, s));
  }
  // states and latches out
  HIPCHK(rd::launch_patch_members(state_of(f), f->p.cur, f->p.flag, f->p.nv, b->mem, b->mb, b->vb, b->nblocks, true,
                                  s));
  for (rd_mesh* m : b->members) {
    note_capture(m);
    m->form32 = false;
  }
  HIPCHK(hipEventRecord(b->ev_out, s));
  for (hipStream_t o : outer) HIPCHK(hipStreamWaitEvent(o, b->ev_out, 0));
  return RD_OK;
}

RD_API rd_status rd_batch_set_tile(rd_batch* b, int tile_triangles) {
  if (!b) return fail(RD_EINVAL, "null batch");
  return batch_set_tile(b, tile_triangles);
}

RD_API rd_status rd_batch_tune(rd_batch* b, double cfl, int scheme, int time, int precision, int n_steps,
                               const int* candidates, int n_candidates, double* ms_per_step, int* best) {
  if (!b) return fail(RD_EINVAL, "null batch");
  rd_status st = tune_args(cfl, scheme, time, precision, n_steps, candidates, n_candidates, best);
  if (st != RD_OK) return st;
  rd_mesh* f = b->flat;
  DeviceGuard g(f->device);
  const int fp32 = precision == RD_FP32_ACC64;
  hipStream_t s = f->stream;
  const int prev = f->tile;
  int pick = -1;
  float pick_ms = 0.0f;
  std::vector<hipStream_t> outer;
  for (int i = 0; i < n_candidates; ++i) {
    if (ms_per_step) ms_per_step[i] = -1.0;
    if (!fp32 && pick >= 0) {  // as rd_tune
      if (ms_per_step && tile_in_range(candidates[i])) ms_per_step[i] = pick_ms / n_steps;
      continue;
    }
    st = batch_set_tile(b, candidates[i]);
    if (st == RD_EUNSUPPORTED || st == RD_EINVAL) continue;
    if (st != RD_OK) break;
    hipGraphExec_t exec = nullptr;
    if ((st = batch_begin(b, fp32, outer)) != RD_OK) break;
    if ((st = batch_graph(b, n_steps, cfl, scheme, time, fp32, &exec)) != RD_OK) break;
    HIPCHK(hipGraphLaunch(exec, s));  // warm-up replay
    if ((st = batch_begin(b, fp32, outer)) != RD_OK) break;
    float t = 0.0f;
    st = time_on(s, [&]() -> rd_status {
      HIPCHK(hipGraphLaunch(exec, s));
      return RD_OK;
    }, &t);
    if (st != RD_OK) break;
    if (ms_per_step) ms_per_step[i] = t / n_steps;
    if (pick < 0 || t < pick_ms * (1.0f - kTuneMargin)) {
      pick = candidates[i];
      pick_ms = t;
    }
  }
  if (st == RD_EUNSUPPORTED || st == RD_EINVAL) st = RD_OK;
  rd_status st2 = batch_set_tile(b, pick >= 0 ? pick : prev);
  HIPCHK(hipStreamSynchronize(s));
  if (st != RD_OK) return st;
  if (st2 != RD_OK) return st2;
  if (pick < 0) return fail(RD_EUNSUPPORTED, "no candidate tile size is usable");
  *best = pick;
  return RD_OK;
}

RD_API rd_status rd_batch_destroy(rd_batch* b) {
  if (!b) return RD_OK;
  DeviceGuard g(b->flat->device);
  (void)hipStreamSynchronize(b->own);
  destroy_graphs(b);
  rd_mesh_destroy(b->flat);
  (void)hipEventDestroy(b->ev_in);
  (void)hipEventDestroy(b->ev_out);
  (void)hipStreamDestroy(b->own);
  delete b;
  return RD_OK;
}

RD_API rd_status rd_sync(rd_mesh* m) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  DeviceGuard g(m->device);
  int flag = 0;
  HIPCHK(hipMemcpyAsync(&flag, m->p.flag, sizeof(int), hipMemcpyDeviceToHost, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  if (flag) return fail(RD_ENONPHYS, "a non-physical state was produced");
  return adjoint_status(m);
}

RD_API const char* rd_last_error(void) { return g_last_error.c_str(); }

// ---------------------------------------------------- mesh generation --
//
// A triangulation is checked as a mesh is (indices, counter-clockwise
// triangles after unwrapping); the neighbour table is built on the host from
// the triangles around each vertex; the flip rounds and refinement iterations
// run on the current device (rd_delaunay.hip), which keeps their account
// (Control): the host enqueues rounds ahead, and an iteration's candidates
// behind them, and waits once for all.

namespace {

// Buffers of one mesh-generation call, freed together: device memory, cut
// from few allocations, and the host's report, which the device writes.
// Allocations of up to 1 MiB take 1 us with their release, larger ones 25 (beyond
// 64 MiB 250), so the arrays of a small mesh's flips come from pieces of 1 MiB,
// others from 16: a refinement's passes take 5 to 9 % longer in many small pieces
// (12 x 12 points to 3e-2 3.4 ms against 3.1, 32 x 32 to 4e-3 14.9 against 14.2).
constexpr int64_t kSmallDl = 80000;  // triangles whose arrays take less than 1 MiB each
struct DlBuffers {
  std::vector<void*> p;
  char* at = nullptr;
  size_t left = 0, piece = size_t(16) << 20;
  rd::dl::Control* control = nullptr;
  // Workgroups the exact pass has scratch for, and how many times those that a
  // run had use for a new block gives: a refinement's runs come to have use for
  // more of them, and a thread that takes a second edge doubles the pass (32 x 32
  // points to 4e-3 14.2 ms without the spare, 13.6 with it).
  int exact_blocks = 0, exact_spare = 1;
  // the report, in pinned memory that the device writes (`mapped`, 24 us to
  // take and give back) or in `own`, the control words copied at each wait
  rd::dl::Report own;
  rd::dl::Report* mapped = nullptr;
  DlBuffers() = default;
  DlBuffers(const DlBuffers&) = delete;
  DlBuffers& operator=(const DlBuffers&) = delete;
  ~DlBuffers() {
    for (void* q : p) (void)hipFree(q);
    if (mapped) (void)hipHostFree(mapped);
  }
  template <class T>
  bool get(T** out, size_t n) {
    const size_t bytes = (std::max<size_t>(n, 1) * sizeof(T) + 255) & ~size_t(255);
    if (bytes > left) {
      void* q = nullptr;
      const size_t take = std::max<size_t>(bytes, piece);
      if (hipMalloc(&q, take) != hipSuccess) return false;
      p.push_back(q);
      at = static_cast<char*>(q);
      left = take;
    }
    *out = reinterpret_cast<T*>(at);
    at += bytes;
    left -= bytes;
    return true;
  }
  bool get_report() {
    void* q = nullptr;
    if (hipHostMalloc(&q, sizeof(rd::dl::Report), hipHostMallocDefault) != hipSuccess) return false;
    mapped = static_cast<rd::dl::Report*>(q);
    return true;
  }
  const volatile rd::dl::Report* report() const { return mapped ? mapped : &own; }
  // Waits for the stream and for the report.
  bool read_report(const rd::dl::Mesh& m, const rd::dl::Refine& r, hipStream_t s) {
    const hipError_t e = mapped ? rd::dl::launch_report(m, r, control, mapped, s)
                                : hipMemcpyAsync(&own.c, control, sizeof(own.c), hipMemcpyDeviceToHost, s);
    return e == hipSuccess && hipStreamSynchronize(s) == hipSuccess;
  }
};

// Corner and neighbour tables [3][nt] of nt triangles (tri: [nt][3]): the
// triangle across an edge is the other one at its first vertex that has the
// second.
rd_status dl_tables(int64_t nt, const int32_t* tri, const HostGeom& geo, rd::Workers& pool, rd::UVec<int32_t>& tsoa,
                    rd::UVec<int32_t>& nbr) {
  tsoa.resize(3 * nt);
  nbr.resize(3 * nt);
  std::atomic<bool> many{false};
  pool.each(nt, [&](int64_t t) {
    for (int i = 0; i < 3; ++i) {
      const int32_t b = tri[3 * t + (i + 1) % 3], c = tri[3 * t + (i + 2) % 3];
      int32_t u = -1;
      for (int32_t j = geo.row[b]; j < geo.row[b + 1]; ++j) {
        const int32_t w = geo.slot[j] / 3;
        if (w == t || (tri[3 * (int64_t)w] != c && tri[3 * (int64_t)w + 1] != c && tri[3 * (int64_t)w + 2] != c)) continue;
        if (u >= 0) many = true;
        u = w;
      }
      tsoa[i * nt + t] = tri[3 * t + i];
      nbr[i * nt + t] = u;
    }
  });
  return many ? fail(RD_EINVAL, "an edge belongs to more than two triangles") : RD_OK;
}

bool hip_ok(hipError_t e) { return e == hipSuccess; }

// Flip rounds until no interior edge of m is illegal. Round and test-pass
// numbers continue across calls (*round, *pass: the pass about to run, whose
// marked triangles' edges are tested). `ahead` rounds are enqueued at a time,
// then what `more` enqueues (which takes effect only if the run is done by
// then), and the host waits for the report: *ahead follows the number of
// rounds that runs take.
template <class More>
rd_status dl_flip_all(rd::dl::Mesh& m, const rd::dl::Refine& r, DlBuffers& b, hipStream_t s, int64_t* flips,
                      int32_t* round, int32_t* pass, int* ahead, const More& more) {
  constexpr int32_t kMaxRounds = 1000000;
  const int32_t round0 = *round, pass0 = *pass;
  const volatile rd::dl::Report* h = b.report();
  int start = rd::dl::kFresh;
  for (int32_t n = 0;;) {
    for (int k = 0; k < *ahead; ++k, ++n, start = rd::dl::kGoOn)
      if (!hip_ok(rd::dl::launch_round(m, b.control, start, round0 + 1 + n, pass0 + n, r.count, b.exact_blocks, s)))
        return fail(RD_EDEVICE, "flip pass failed");
    if (!more() || !b.read_report(m, r, s)) return fail(RD_EDEVICE, "flip pass failed");
    if (h->c.stuck) return fail(RD_EDEVICE, "a round flipped no edge");
    // scratch for the exact pass: 41 KB a thread, one for every edge seen up to 4096
    const int want = b.exact_spare * (int)std::min<int64_t>(64 / b.exact_spare, (h->c.need + 63) / 64);
    if (h->c.starved || want > 4 * b.exact_blocks) {
      if (want > b.exact_blocks) {
        if (!b.get(&m.work, rd::dl::exact_scratch(want))) return fail(RD_ENOMEM, "device allocation failed");
        b.exact_blocks = want;
      }
      if (h->c.starved) {
        n = h->c.rounds;
        start = rd::dl::kResume;
        continue;
      }
    }
    if (h->c.done) break;
    if (n >= kMaxRounds) return fail(RD_EDEVICE, "flipping did not finish");
    *ahead = std::min(2 * *ahead, 32);
  }
  *flips += h->c.flips;
  *round = round0 + h->c.rounds;
  *pass = pass0 + h->c.rounds + 1;  // the last pass found nothing illegal
  *ahead = std::max(2, std::min(h->c.rounds + 2, 32));
  return RD_OK;
}

// Device arrays of the flip passes for a capacity of ts triangles.
bool dl_flip_arrays(rd::dl::Mesh& m, DlBuffers& b, int64_t ts) {
  return b.get(&m.tri, 3 * ts) && b.get(&m.nbr, 3 * ts) && b.get(&m.claim, ts) && b.get(&m.cand, ts) &&
         b.get(&m.flipped, ts) && b.get(&m.partner, ts) && b.get(&m.count, 3) && b.get(&m.mark, ts) &&
         b.get(&m.undecided, 3 * ts / 2 + 1);
}

// Renumber vertices, then triangles, in Morton order (the moved arrays are
// swapped in: m's and o's pointers trade places).
rd_status dl_reorder(rd::dl::Mesh& m, rd::dl::Order& o, int64_t nv, void* tmp, size_t tmp_bytes, hipStream_t s) {
  if (!hip_ok(rd::dl::launch_vkeys(m, o, nv, s)) || !hip_ok(rd::dl::launch_sort(o, nv, tmp, tmp_bytes, s)) ||
      !hip_ok(rd::dl::launch_invert(o, nv, s)) || !hip_ok(rd::dl::launch_vapply(m, o, nv, s)) ||
      !hip_ok(rd::dl::launch_vrename(m, o, s)))
    return fail(RD_EDEVICE, "vertex reordering failed");
  std::swap(m.x, o.xt);
  std::swap(m.y, o.yt);
  if (!hip_ok(rd::dl::launch_tkeys(m, o, s)) || !hip_ok(rd::dl::launch_sort(o, m.nt, tmp, tmp_bytes, s)) ||
      !hip_ok(rd::dl::launch_invert(o, m.nt, s)) || !hip_ok(rd::dl::launch_tapply(m, o, s)))
    return fail(RD_EDEVICE, "triangle reordering failed");
  std::swap(m.tri, o.tt);
  std::swap(m.nbr, o.nb);
  return RD_OK;
}

struct StreamGuard {
  hipStream_t s = nullptr;
  ~StreamGuard() {
    if (s) {
      (void)hipStreamSynchronize(s);
      (void)hipStreamDestroy(s);
    }
  }
};

}  // namespace

static rd_status delaunay_flip(int64_t n_vertices, const double* x, const double* y, double period_x, double period_y,
                               int64_t n_triangles, int32_t* tri, int64_t* n_flips, int32_t* n_rounds) {
  rd_mesh_desc desc{};
  desc.n_vertices = n_vertices;
  desc.n_triangles = n_triangles;
  desc.x = x;
  desc.y = y;
  desc.tri = tri;
  desc.period_x = period_x;
  desc.period_y = period_y;
  desc.gamma = 1.4;  // not used; the check requires a valid value
  HostGeom geo;
  rd::Workers pool(workers_for(n_triangles));
  rd_status st = check_desc(&desc, &geo, pool);
  if (st != RD_OK) return st;
  const int64_t nt = n_triangles, nv = n_vertices;
  rd::UVec<int32_t> nbr, tsoa;
  if ((st = dl_tables(nt, tri, geo, pool, tsoa, nbr)) != RD_OK) return st;
  DlBuffers b;
  StreamGuard g;  // declared after the buffers: the stream is drained before they are freed
  rd::dl::Mesh m;
  m.nt = nt;
  m.ts = nt;
  m.px = period_x;
  m.py = period_y;
  if (nt <= kSmallDl) b.piece = size_t(1) << 20;
  if (!b.get(&m.x, nv) || !b.get(&m.y, nv) || !dl_flip_arrays(m, b, nt) || !b.get(&b.control, 1))
    return fail(RD_ENOMEM, "device allocation failed");
  if (hipStreamCreate(&g.s) != hipSuccess) return fail(RD_EDEVICE, "hipStreamCreate failed");
  const hipStream_t s = g.s;
  if (!hip_ok(hipMemcpyAsync(m.x, x, sizeof(double) * nv, hipMemcpyHostToDevice, s)) ||
      !hip_ok(hipMemcpyAsync(m.y, y, sizeof(double) * nv, hipMemcpyHostToDevice, s)) ||
      !hip_ok(hipMemcpyAsync(m.tri, tsoa.data(), sizeof(int32_t) * 3 * nt, hipMemcpyHostToDevice, s)) ||
      !hip_ok(hipMemcpyAsync(m.nbr, nbr.data(), sizeof(int32_t) * 3 * nt, hipMemcpyHostToDevice, s)) ||
      !hip_ok(hipMemsetAsync(m.flipped, 0, sizeof(int32_t) * nt, s)) ||
      !hip_ok(hipMemsetAsync(m.mark, 0, sizeof(int32_t) * nt, s)))
    return fail(RD_EDEVICE, "upload failed");
  int64_t flips = 0;
  int32_t round = 0, pass = 0;  // every mark is 0: the first pass tests every edge
  int ahead = 2;  // a jittered lattice takes one round that flips and one that finds nothing
  if ((st = dl_flip_all(m, rd::dl::Refine(), b, s, &flips, &round, &pass, &ahead, [] { return true; })) != RD_OK)
    return st;
  if (!hip_ok(hipMemcpyAsync(tsoa.data(), m.tri, sizeof(int32_t) * 3 * nt, hipMemcpyDeviceToHost, s)) ||
      !hip_ok(hipStreamSynchronize(s)))
    return fail(RD_EDEVICE, "download failed");
  for (int64_t t = 0; t < nt; ++t)
    for (int i = 0; i < 3; ++i) tri[3 * t + i] = tsoa[i * nt + t];
  if (n_flips) *n_flips = flips;
  if (n_rounds) *n_rounds = round;
  return RD_OK;
}

RD_API rd_status rd_delaunay_flip(int64_t n_vertices, const double* x, const double* y, double period_x,
                                  double period_y, int64_t n_triangles, int32_t* tri, int64_t* n_flips,
                                  int32_t* n_rounds) {
  return guarded([&] { return delaunay_flip(n_vertices, x, y, period_x, period_y, n_triangles, tri, n_flips, n_rounds); });
}

static rd_status delaunay_refine(int64_t* n_vertices, double* x, double* y, int64_t max_vertices, double period_x,
                                 double period_y, int64_t* n_triangles, int32_t* tri, int64_t max_triangles,
                                 double max_radius, double max_ratio, const double* size_grid, int32_t grid_nx,
                                 int32_t grid_ny, int32_t max_iterations, int32_t morton, int32_t* n_iterations,
                                 int64_t* n_flips) {
  if (!n_vertices || !n_triangles) return fail(RD_EINVAL, "null count pointer");
  const int64_t nv0 = *n_vertices, nt0 = *n_triangles;
  if (max_vertices < nv0 || max_triangles < nt0) return fail(RD_EINVAL, "capacity below the current size");
  if (max_vertices >= INT32_MAX || max_triangles >= INT32_MAX / 3)  // edge keys 3 t + i are int32
    return fail(RD_EINVAL, "capacity beyond the 32-bit index range");
  if (!(max_radius >= 0.0) || !std::isfinite(max_radius)) return fail(RD_EINVAL, "max_radius must be >= 0");
  if (!(max_ratio == 0.0 || max_ratio >= 1.0) || !std::isfinite(max_ratio))
    return fail(RD_EINVAL, "max_ratio must be 0 (no bound) or >= 1");
  if (max_iterations < 1) return fail(RD_EINVAL, "max_iterations must be >= 1");
  if (morton != 0 && morton != 1) return fail(RD_EINVAL, "morton must be 0 or 1");
  if (size_grid) {
    if (grid_nx < 1 || grid_ny < 1 || (int64_t)grid_nx * grid_ny > (1 << 26))
      return fail(RD_EINVAL, "size grid dimensions must be >= 1 (at most 2^26 nodes)");
    for (int64_t k = 0; k < (int64_t)grid_nx * grid_ny; ++k)
      if (!(size_grid[k] > 0.0) || !std::isfinite(size_grid[k]))
        return fail(RD_EINVAL, "size grid values must be positive and finite");
  }
  rd_mesh_desc desc{};
  desc.n_vertices = nv0;
  desc.n_triangles = nt0;
  desc.x = x;
  desc.y = y;
  desc.tri = tri;
  desc.period_x = period_x;
  desc.period_y = period_y;
  desc.gamma = 1.4;  // not used; the check requires a valid value
  HostGeom geo;
  rd::Workers pool(workers_for(nt0));
  rd_status st = check_desc(&desc, &geo, pool);
  if (st != RD_OK) return st;
  for (int64_t v = 0; v < nv0; ++v)
    if ((period_x > 0.0 && !(x[v] >= 0.0 && x[v] < period_x)) || (period_y > 0.0 && !(y[v] >= 0.0 && y[v] < period_y)))
      return fail(RD_EINVAL, "a coordinate on a periodic axis is outside [0, period)");
  rd::UVec<int32_t> nbr, tsoa;
  if ((st = dl_tables(nt0, tri, geo, pool, tsoa, nbr)) != RD_OK) return st;
  for (int64_t t = 0; t < nt0; ++t)
    for (int i = 0; i < 3; ++i) {
      if (nbr[i * nt0 + t] >= 0) continue;
      const int32_t b = tsoa[((i + 1) % 3) * nt0 + t], c = tsoa[((i + 2) % 3) * nt0 + t];
      if (x[b] != x[c] && y[b] != y[c]) return fail(RD_EINVAL, "a boundary edge is not axis-aligned");
    }
  // Arrays for `vs` vertices and `ts` triangles. The caller's limits are often
  // far beyond what the mesh comes to need (mapping arrays of that size took
  // longer than the refinement), so they grow with it: an iteration over nt
  // triangles adds at most 2 nt, and no more vertices than triangles.
  struct Arrays {
    DlBuffers b;
    rd::dl::Mesh m;
    rd::dl::Refine r;
    rd::dl::Order o;
    char *scan_tmp = nullptr, *sort_tmp = nullptr;
    size_t scan_bytes = 0, sort_bytes = 0;
  };
  DlBuffers b;
  b.piece = size_t(1) << 20;
  b.exact_spare = 4;
  std::unique_ptr<Arrays> A(new Arrays());
  StreamGuard g;  // declared after the buffers: the stream is drained before they are freed
  auto allocate = [&](Arrays& a, int64_t vs, int64_t ts) {
    a.m.ts = ts;
    rd::dl::Refine& r = a.r;
    a.scan_bytes = rd::dl::scan_tmp_bytes(ts);
    if (!a.b.get(&a.m.x, vs) || !a.b.get(&a.m.y, vs) || !dl_flip_arrays(a.m, a.b, ts) || !a.b.get(&r.prio, ts) ||
        !a.b.get(&r.px, ts) || !a.b.get(&r.py, ts) || !a.b.get(&r.loc, ts) || !a.b.get(&r.where, ts) ||
        !a.b.get(&r.lock, ts) || !a.b.get(&r.win, ts) || !a.b.get(&r.wpos, ts) || !a.b.get(&r.tnew, ts) ||
        !a.b.get(&r.tpos, ts) || !a.b.get(&r.split, ts) || !a.b.get(&r.child, 2 * ts) || !a.b.get(&r.count, 3) ||
        !a.b.get(&a.scan_tmp, a.scan_bytes))
      return false;
    if (!morton) return true;
    const int64_t n = std::max(vs, ts);
    a.sort_bytes = rd::dl::sort_tmp_bytes(n);
    return a.b.get(&a.o.key, n) && a.b.get(&a.o.skey, n) && a.b.get(&a.o.idx, n) && a.b.get(&a.o.perm, n) &&
           a.b.get(&a.o.inv, n) && a.b.get(&a.o.xt, vs) && a.b.get(&a.o.yt, vs) && a.b.get(&a.o.tt, 3 * ts) &&
           a.b.get(&a.o.nb, 3 * ts) && a.b.get(&a.sort_tmp, a.sort_bytes);
  };
  const int64_t ts0 = std::min<int64_t>(max_triangles, std::max<int64_t>(4 * nt0, 1 << 16));
  A->m.nt = nt0;
  A->m.px = period_x;
  A->m.py = period_y;
  A->r.nv = nv0;
  A->r.r2 = max_radius * max_radius;
  A->r.b2 = max_ratio * max_ratio;
  if (!allocate(*A, std::min(max_vertices, nv0 + ts0 - nt0), ts0) || !b.get(&b.control, 1) || !b.get_report())
    return fail(RD_ENOMEM, "device allocation failed");
  if (size_grid) {
    // grid frame: the period on a periodic axis (nodes wrap), else the input's extent
    auto frame = [&](const double* c, double period, int32_t n, double& g0, double& gd) {
      double lo = c[0], hi = c[0];
      for (int64_t v = 1; v < nv0; ++v) {
        lo = std::min(lo, c[v]);
        hi = std::max(hi, c[v]);
      }
      g0 = period > 0.0 ? 0.0 : lo;
      gd = period > 0.0 ? period / n : (n > 1 ? (hi - lo) / (n - 1) : 1.0);
    };
    frame(x, period_x, grid_nx, A->r.gx0, A->r.gdx);
    frame(y, period_y, grid_ny, A->r.gy0, A->r.gdy);
    double* g = nullptr;
    const int64_t ng = (int64_t)grid_nx * grid_ny;
    if (!b.get(&g, ng)) return fail(RD_ENOMEM, "device allocation failed");
    if (hipMemcpy(g, size_grid, sizeof(double) * ng, hipMemcpyHostToDevice) != hipSuccess)
      return fail(RD_EDEVICE, "upload failed");
    A->r.sgrid = g;
    A->r.gnx = grid_nx;
    A->r.gny = grid_ny;
  }
  if (morton) {
    // Morton frame: the period on a periodic axis, else the input's extent
    auto frame = [&](const double* c, double period, double& c0, double& sc) {
      double lo = c[0], hi = c[0];
      for (int64_t v = 1; v < nv0; ++v) {
        lo = std::min(lo, c[v]);
        hi = std::max(hi, c[v]);
      }
      c0 = period > 0.0 ? 0.0 : lo;
      sc = 4294967296.0 / (period > 0.0 ? period : hi - lo);
    };
    frame(x, period_x, A->o.x0, A->o.sx);
    frame(y, period_y, A->o.y0, A->o.sy);
  }
  if (hipStreamCreate(&g.s) != hipSuccess) return fail(RD_EDEVICE, "hipStreamCreate failed");
  const hipStream_t s = g.s;
  // a table of three rows of n entries, rows `to` and `from` entries apart
  auto rows = [&](int32_t* dst, int64_t to, const int32_t* src, int64_t from, int64_t n, hipMemcpyKind k) {
    return hip_ok(hipMemcpy2DAsync(dst, sizeof(int32_t) * to, src, sizeof(int32_t) * from, sizeof(int32_t) * n, 3, k, s));
  };
  auto clear = [&](Arrays& a) {
    return hip_ok(hipMemsetAsync(a.m.flipped, 0, sizeof(int32_t) * a.m.ts, s)) &&
           hip_ok(hipMemsetAsync(a.m.mark, 0, sizeof(int32_t) * a.m.ts, s)) &&
           hip_ok(hipMemsetAsync(a.r.split, 0, sizeof(int32_t) * a.m.ts, s));
  };
  if (!hip_ok(hipMemcpyAsync(A->m.x, x, sizeof(double) * nv0, hipMemcpyHostToDevice, s)) ||
      !hip_ok(hipMemcpyAsync(A->m.y, y, sizeof(double) * nv0, hipMemcpyHostToDevice, s)) ||
      !rows(A->m.tri, ts0, tsoa.data(), nt0, nt0, hipMemcpyHostToDevice) ||
      !rows(A->m.nbr, ts0, nbr.data(), nt0, nt0, hipMemcpyHostToDevice) || !clear(*A))
    return fail(RD_EDEVICE, "upload failed");
  int64_t flips = 0;
  int32_t round = 0, it = 0, pass = 0;  // every mark is 0: the first pass tests every edge
  int64_t nv = nv0, nt = nt0, nt_ordered = nt0;
  // the mesh reached so far goes back to the caller, also when a limit stops the loop
  auto download = [&](rd_status result) {
    tsoa.resize(3 * nt);
    if (!hip_ok(hipMemcpyAsync(x, A->m.x, sizeof(double) * nv, hipMemcpyDeviceToHost, s)) ||
        !hip_ok(hipMemcpyAsync(y, A->m.y, sizeof(double) * nv, hipMemcpyDeviceToHost, s)) ||
        !rows(tsoa.data(), nt, A->m.tri, A->m.ts, nt, hipMemcpyDeviceToHost) || !hip_ok(hipStreamSynchronize(s)))
      return fail(RD_EDEVICE, "download failed");
    for (int64_t t = 0; t < nt; ++t)
      for (int i = 0; i < 3; ++i) tri[3 * t + i] = tsoa[i * nt + t];
    *n_vertices = nv;
    *n_triangles = nt;
    if (n_iterations) *n_iterations = it;
    if (n_flips) *n_flips = flips;
    return result;
  };
  int ahead = 2;  // as rd_delaunay_flip
  // the same arrays with room for the next iteration
  auto grow = [&]() -> rd_status {
    const int64_t ts = std::min<int64_t>(max_triangles, std::max(4 * nt, 2 * A->m.ts));
    std::unique_ptr<Arrays> n(new Arrays());
    n->m.nt = nt;
    n->m.px = period_x;
    n->m.py = period_y;
    n->m.work = A->m.work;
    n->r = A->r;
    n->o = A->o;
    if (!allocate(*n, std::min(max_vertices, nv + ts - nt), ts)) return fail(RD_ENOMEM, "device allocation failed");
    auto move = [&](void* dst, const void* src, size_t bytes) {
      return hip_ok(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, s));
    };
    if (!clear(*n) || !move(n->m.x, A->m.x, sizeof(double) * nv) || !move(n->m.y, A->m.y, sizeof(double) * nv) ||
        !rows(n->m.tri, ts, A->m.tri, A->m.ts, nt, hipMemcpyDeviceToDevice) ||
        !rows(n->m.nbr, ts, A->m.nbr, A->m.ts, nt, hipMemcpyDeviceToDevice) ||
        !move(n->m.flipped, A->m.flipped, sizeof(int32_t) * nt) || !move(n->m.mark, A->m.mark, sizeof(int32_t) * nt) ||
        !move(n->r.split, A->r.split, sizeof(int32_t) * nt) || !hip_ok(hipStreamSynchronize(s)))
      return fail(RD_EDEVICE, "growing the mesh failed");
    A.swap(n);
    return RD_OK;
  };
  for (;;) {
    if (A->m.ts < std::min<int64_t>(max_triangles, 3 * nt) && (st = grow()) != RD_OK) return st;
    rd::dl::Mesh& m = A->m;
    rd::dl::Refine& r = A->r;
    rd::dl::Order& o = A->o;
    // the flips, then (unless a renumbering, which the host decides, comes in
    // between) the candidates and the insertion set of the next iteration
    r.seed = 0x9e3779b9u * (uint32_t)(it + 1);
    auto candidates = [&] {
      return hip_ok(rd::dl::launch_candidates(m, r, b.control, s)) &&
             hip_ok(rd::dl::launch_scan(r.win, r.wpos, nt, A->scan_tmp, A->scan_bytes, s)) &&
             hip_ok(rd::dl::launch_scan(r.tnew, r.tpos, nt, A->scan_tmp, A->scan_bytes, s));
    };
    const bool renumber = it > 0 && morton && 4 * nt >= 5 * nt_ordered;  // after every 25 % of growth, and at the end
    if ((st = dl_flip_all(m, r, b, s, &flips, &round, &pass, &ahead, [&] { return renumber || candidates(); })) != RD_OK)
      return st;
    if (renumber) {
      if ((st = dl_reorder(m, o, nv, A->sort_tmp, A->sort_bytes, s)) != RD_OK) return st;
      nt_ordered = nt;
      if (!candidates() || !b.read_report(m, r, s))
        return fail(RD_EDEVICE, "insertion-set passes failed");
    }
    const volatile rd::dl::Report* h = b.report();
    if (h->count[0] == 0) {
      if (h->count[1] > 0)
        return download(fail(RD_EUNSUPPORTED, "a circumcentre lies more than a quarter period from its triangle"));
      if (morton && nt != nt_ordered && (st = dl_reorder(m, o, nv, A->sort_tmp, A->sort_bytes, s)) != RD_OK) return st;
      return download(RD_OK);
    }
    if (it >= max_iterations) return download(fail(RD_EINVAL, "refinement needs more than max_iterations iterations"));
    ++it;
    const int64_t nwin = h->nwin, nadd = h->nadd;
    if (nwin == 0)
      return download(fail(RD_EUNSUPPORTED, "no candidate could be inserted (" + std::to_string(h->count[1]) +
                                                " not located, " + std::to_string(h->count[2]) + " cavities too large)"));
    if (nv + nwin > max_vertices || nt + nadd > max_triangles)
      return download(fail(RD_ENOMEM, "the refined mesh needs more than max_vertices or max_triangles"));
    r.nv = nv;
    if (!hip_ok(rd::dl::launch_insert(m, r, it, pass, s)) ||
        !hip_ok(rd::dl::launch_fixsplit(m, r, it, nt + nadd, s)))
      return fail(RD_EDEVICE, "insertion failed");
    nv += nwin;
    nt += nadd;
    m.nt = nt;
  }
}

RD_API rd_status rd_delaunay_refine(int64_t* n_vertices, double* x, double* y, int64_t max_vertices,
                                    double period_x, double period_y, int64_t* n_triangles, int32_t* tri,
                                    int64_t max_triangles, double max_radius, double max_ratio,
                                    const double* size_grid, int32_t grid_nx, int32_t grid_ny,
                                    int32_t max_iterations, int32_t morton, int32_t* n_iterations,
                                    int64_t* n_flips) {
  return guarded([&] {
    return delaunay_refine(n_vertices, x, y, max_vertices, period_x, period_y, n_triangles, tri, max_triangles,
                           max_radius, max_ratio, size_grid, grid_nx, grid_ny, max_iterations, morton, n_iterations,
                           n_flips);
  });
}

// --------------------------------------------------------- three dimensions --
//
// Host side of the tetrahedral path: validation and geometry (volumes, vertex
// volumes), the tiles (rd3_tiling.h), buffers and the launch order of a step
// (kernels in rd3_kernels.hip, which form the face normals themselves).

struct rd3_mesh {
  rd3::Dev3 d;
  bool renumbered = false;  // the vertices are not in the caller's order
  int* bad = nullptr;  // first vertex of a host state that is not physical
  std::vector<void*> bufs;
  hipStream_t stream = nullptr;
  ~rd3_mesh() {
    if (stream) {
      (void)hipStreamSynchronize(stream);
      (void)hipStreamDestroy(stream);
    }
    for (void* q : bufs) (void)hipFree(q);
  }
};

namespace {

double unwrap3(double d, double period) {
  if (period > 0.0) {
    if (d > 0.5 * period) d -= period;
    else if (d < -0.5 * period) d += period;
  }
  return d;
}

// The buffers of a mesh, in one allocation, tables from the host first: those
// of a small mesh go up in one copy (a copy takes 12 us, and there are ten).
class Buffers3 {
 public:
  template <class T, class A>
  Buffers3& put(T** p, const std::vector<T, A>& h) {
    return add(p, h.data(), sizeof(T) * h.size());
  }
  template <class T>
  Buffers3& get(T** p, size_t n) {
    return add(p, nullptr, sizeof(T) * n);
  }
  rd_status take(rd3_mesh* m) {
    void* q = nullptr;
    if (hipMalloc(&q, bytes_) != hipSuccess) return fail(RD_ENOMEM, "device allocation failed");
    m->bufs.push_back(q);
    char* const base = static_cast<char*>(q);
    std::vector<char> stage(tables_ <= kSlab ? tables_ : 0);
    for (const Entry& e : list_) {
      *e.p = base + e.at;
      if (!e.from || e.size == 0) continue;
      if (!stage.empty()) std::memcpy(&stage[e.at], e.from, e.size);
      else HIPCHK(hipMemcpy(base + e.at, e.from, e.size, hipMemcpyHostToDevice));
    }
    if (!stage.empty()) HIPCHK(hipMemcpy(base, stage.data(), tables_, hipMemcpyHostToDevice));
    return RD_OK;
  }

 private:
  struct Entry {
    void** p;
    const void* from;
    size_t at, size;
  };
  std::vector<Entry> list_;
  size_t bytes_ = 0, tables_ = 0;
  Buffers3& add(void* p, const void* from, size_t size) {
    list_.push_back({static_cast<void**>(p), from, bytes_, size});
    bytes_ += (std::max<size_t>(size, 1) + 255) & ~size_t(255);
    if (from) tables_ = bytes_;
    return *this;
  }
};

rd_status rd3_check_step(int scheme, int time) {
  if (scheme < RD_N || scheme > RD_BMIN) return fail(RD_EINVAL, "unknown scheme for three dimensions");
  if (time != RD_EULER1 && time != RD_RK2) return fail(RD_EINVAL, "unknown time integration");
  return RD_OK;
}

// One step with the time step from the CFL limit, or (cfl = 0) the one set on
// the stream.
rd_status rd3_stages(rd3_mesh* m, double cfl, int scheme, int time, hipEvent_t* ev) {
  const rd3::Dev3& d = m->d;
  const hipStream_t s = m->stream;
  auto mark = [&](int k) { return ev ? hipEventRecord(ev[k], s) : hipSuccess; };
  HIPCHK(rd3::launch3_tile(d, 1, scheme, cfl > 0.0, s));
  HIPCHK(mark(1));
  if (cfl > 0.0) HIPCHK(rd3::launch3_cfl(d, cfl, s));
  HIPCHK(mark(2));
  HIPCHK(rd3::launch3_gather(d, time == RD_RK2 ? 1 : 0, s));
  HIPCHK(mark(3));
  if (time == RD_RK2) {
    HIPCHK(rd3::launch3_tile(d, 2, scheme, false, s));
    HIPCHK(mark(4));
    HIPCHK(rd3::launch3_gather(d, 2, s));
    HIPCHK(mark(5));
  }
  return RD_OK;
}

}  // namespace

// Meshes of up to this many vertices keep the caller's numbering: their state
// then goes out as it stands, without a launch to reorder it first
// (rd3_get_state, us, without / with: 11 / 23 at 512 vertices, 36 / 49 at
// 13824), and it is in the caches in any order (a step with its state set: 71 /
// 71 at 2744 vertices, 80 / 78 at 8000, 88 / 87 at 13824; state in, an Euler step,
// state out 142 / 168 at 19683 and 195 / 233 at 27000; ten RK2 steps 608 / 599 and
// 745 / 732, in random order 622 / 608 and 758 / 732, 901 / 858 at 39304).
constexpr int64_t kRenumber3 = 32768;

static rd_status rd3_create(const rd3_mesh_desc* desc, rd3_mesh** out) {
  if (!desc || !out) return fail(RD_EINVAL, "null argument");
  *out = nullptr;
  const int64_t nv = desc->n_vertices, nt = desc->n_tets;
  if (nv < 4 || nt < 1) return fail(RD_EINVAL, "empty mesh");
  if (nv >= INT32_MAX || nt >= INT32_MAX / 4) return fail(RD_EINVAL, "mesh too large for 32-bit indices");
  if (!desc->x || !desc->y || !desc->z || !desc->tet) return fail(RD_EINVAL, "null array");
  if (!(desc->gamma > 1.0)) return fail(RD_EINVAL, "gamma must exceed 1");
  const double per[3] = {desc->period_x, desc->period_y, desc->period_z};
  for (double p : per)
    if (!(p >= 0.0) || !std::isfinite(p)) return fail(RD_EINVAL, "invalid period");
  const double* xyz[3] = {desc->x, desc->y, desc->z};
  std::vector<double> V(nv, 0.0);
  for (int64_t t = 0; t < nt; ++t) {
    int32_t v[4];
    for (int i = 0; i < 4; ++i) {
      v[i] = desc->tet[4 * t + i];
      if (v[i] < 0 || v[i] >= nv) return fail(RD_EINVAL, "tetrahedron " + std::to_string(t) + ": index out of range");
    }
    double p[4][3];
    for (int i = 0; i < 4; ++i)
      for (int k = 0; k < 3; ++k) p[i][k] = i == 0 ? 0.0 : unwrap3(xyz[k][v[i]] - xyz[k][v[0]], per[k]);
    auto cr = [](const double* a, const double* b, double* c) {
      c[0] = a[1] * b[2] - a[2] * b[1];
      c[1] = a[2] * b[0] - a[0] * b[2];
      c[2] = a[0] * b[1] - a[1] * b[0];
    };
    double c[3];
    cr(p[2], p[3], c);
    const double six = p[1][0] * c[0] + p[1][1] * c[1] + p[1][2] * c[2];
    if (!(six > 0.0)) return fail(RD_EINVAL, "tetrahedron " + std::to_string(t) + " is not positively oriented");
    for (int i = 0; i < 4; ++i) V[v[i]] += six / 6.0 / 4.0;
  }
  for (int64_t v = 0; v < nv; ++v)
    if (!(V[v] > 0.0)) return fail(RD_EINVAL, "vertex " + std::to_string(v) + " belongs to no tetrahedron");
  std::unique_ptr<rd3_mesh> m(new rd3_mesh());
  rd3::Dev3& d = m->d;
  int dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
    return fail(RD_EDEVICE, "no HIP device");
  // tetrahedra per tile: 256, or fewer on a mesh that would give the compute
  // units less than two such tiles each
  int target = rd3::kTileTets;
  while (target > 64 && nt < (int64_t)target * 2 * ncu) target /= 2;
  rd3::TilePlan3 P;
  m->renumbered = nv > kRenumber3;
  // 12^3 cells: 1.8 ms by one worker, 1.0 by four, 1.3 by eight; 8^3: 0.36, 0.28, 0.46
  rd::Workers pool(nt < 5000 ? 1 : nt < 30000 ? std::min(4, host_threads()) : host_threads());
  const std::string why = rd3::build_tiles3(nv, nt, desc->tet, xyz, per, target, m->renumbered, pool, P);
  if (!why.empty()) return fail(RD_EINVAL, why);
  d.nv = nv;
  d.ntiles = (int32_t)P.tile.size();
  d.threads = target;
  d.max_lv = P.max_lv;
  d.max_tet = P.max_tet;
  rd3::tile3_lds(d, P.max_jd);
  d.gamma = desc->gamma;
  d.g1 = d.gamma - 1.0;
  d.ig1 = 1.0 / d.g1;
  d.gfac = d.g1 / d.gamma;
  for (int k = 0; k < 3; ++k) {
    d.per[k] = per[k];
    d.half[k] = per[k] > 0.0 ? 0.5 * per[k] : HUGE_VAL;
  }
  std::vector<double> Vi(nv);
  rd::UVec<double2> r1(5 * nv);
  pool.each(nv, [&](int64_t v) {
    const int64_t i = P.inv[v];
    Vi[i] = V[v];
    for (int k = 0; k < 3; ++k) r1[5 * i + k] = make_double2(0.0, 0.0);
    r1[5 * i + 3] = make_double2(xyz[0][v], xyz[1][v]);
    r1[5 * i + 4] = make_double2(xyz[2][v], 0.0);
  });
  rd3::Tile3* dtile;
  uint32_t* dtet;
  int32_t *dlv, *drpos, *djb, *drbeg, *dinv;
  uint16_t* ddeg;
  double* dV;
  const int nb = rd3::cfl_blocks(nv);
  Buffers3 buffers;
  buffers.put(&dtile, P.tile).put(&dtet, P.tet).put(&dlv, P.lv).put(&drpos, P.rpos).put(&ddeg, P.deg).put(&djb, P.jb);
  buffers.put(&drbeg, P.rbeg).put(&dinv, P.inv).put(&dV, Vi).put(&d.r1, r1);
  buffers.get(&d.W, 5 * nv).get(&d.Ws, 5 * nv).get(&d.r2, 5 * nv).get(&d.rec, 6 * P.lv.size()).get(&d.dt, 1);
  buffers.get(&d.bmin, nb).get(&d.flag, 1).get(&m->bad, 1);
  rd_status st = buffers.take(m.get());
  if (st != RD_OK) return st;
  HIPCHK(hipStreamCreate(&m->stream));
  HIPCHK(hipMemsetAsync(d.W, 0, sizeof(double) * 5 * nv, m->stream));
  HIPCHK(hipMemsetAsync(d.flag, 0, sizeof(int), m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  d.tile = dtile;
  d.tet = reinterpret_cast<const uint4*>(dtet);
  d.lv = dlv;
  d.rpos = drpos;
  d.deg = ddeg;
  d.jb = djb;
  d.rbeg = drbeg;
  d.inv = dinv;
  d.V = dV;
  *out = m.release();
  return RD_OK;
}

RD_API rd_status rd3_mesh_create(const rd3_mesh_desc* desc, rd3_mesh** out) {
  return guarded([&] { return rd3_create(desc, out); });
}

RD_API rd_status rd3_mesh_destroy(rd3_mesh* mesh) {
  delete mesh;
  return RD_OK;
}

RD_API rd_status rd3_set_state(rd3_mesh* m, const double* W, int on_device) {
  if (!m || !W) return fail(RD_EINVAL, "null argument");
  const int64_t nv = m->d.nv;
  int64_t first = nv;
  if (!on_device) {  // through Ws, which holds nothing between steps
    if (nv <= kHostCheck3) first = first_unphysical(W, nv, 3, m->d.gamma);
    if (first == nv) HIPCHK(hipMemcpyAsync(m->d.Ws, W, sizeof(double) * 5 * nv, hipMemcpyHostToDevice, m->stream));
    if (nv > kHostCheck3) {
      int named = 0;
      HIPCHK(rd::launch_check_state(m->d.Ws, nv, 3, m->d.gamma, m->bad, m->stream));
      HIPCHK(hipMemcpyAsync(&named, m->bad, sizeof(int), hipMemcpyDeviceToHost, m->stream));
      HIPCHK(hipStreamSynchronize(m->stream));
      first = std::min<int64_t>(named, nv);
    }
    if (first < nv)
      return fail(RD_ENONPHYS, "vertex " + std::to_string(first) + ": rho <= 0, p <= 0 or not finite");
  }
  HIPCHK(rd::launch_fill_int(m->d.flag, 0, 1, m->stream));
  HIPCHK(rd3::launch3_set(m->d, on_device ? W : m->d.Ws, m->stream));
  if (!on_device && nv <= kHostCheck3) HIPCHK(hipStreamSynchronize(m->stream));
  return RD_OK;
}

RD_API rd_status rd3_get_state(rd3_mesh* m, double* W, int on_device) {
  if (!m || !W) return fail(RD_EINVAL, "null argument");
  const bool reorder = on_device || m->renumbered;
  if (reorder) HIPCHK(rd3::launch3_get(m->d, on_device ? W : m->d.Ws, m->stream));
  if (!on_device)
    HIPCHK(hipMemcpyAsync(W, reorder ? m->d.Ws : m->d.W, sizeof(double) * 5 * m->d.nv, hipMemcpyDeviceToHost, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  return RD_OK;
}

RD_API rd_status rd3_max_dt(rd3_mesh* m, double cfl, double* dt) {
  if (!m || !dt) return fail(RD_EINVAL, "null argument");
  if (!(cfl > 0.0)) return fail(RD_EINVAL, "cfl must be positive");
  HIPCHK(rd3::launch3_tile(m->d, 0, RD_N, true, m->stream));
  HIPCHK(rd3::launch3_cfl(m->d, cfl, m->stream));
  HIPCHK(hipMemcpyAsync(dt, m->d.dt, sizeof(double), hipMemcpyDeviceToHost, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  return RD_OK;
}

RD_API rd_status rd3_step(rd3_mesh* m, double dt, int scheme, int time) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  rd_status st = rd3_check_step(scheme, time);
  if (st != RD_OK) return st;
  if (!(dt > 0.0) || !std::isfinite(dt)) return fail(RD_EINVAL, "dt must be positive");
  HIPCHK(rd3::launch3_set_dt(m->d, dt, m->stream));
  return rd3_stages(m, 0.0, scheme, time, nullptr);
}

RD_API rd_status rd3_step_cfl(rd3_mesh* m, int n_steps, double cfl, int scheme, int time) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  rd_status st = rd3_check_step(scheme, time);
  if (st != RD_OK) return st;
  if (!(cfl > 0.0) || n_steps < 0) return fail(RD_EINVAL, "cfl must be positive and n_steps >= 0");
  for (int k = 0; k < n_steps; ++k)
    if ((st = rd3_stages(m, cfl, scheme, time, nullptr)) != RD_OK) return st;
  return RD_OK;
}

RD_API rd_status rd3_step_timed(rd3_mesh* m, int n_steps, double cfl, int scheme, int time, double* ms) {
  if (!m || !ms) return fail(RD_EINVAL, "null argument");
  rd_status st = rd3_check_step(scheme, time);
  if (st != RD_OK) return st;
  if (!(cfl > 0.0) || n_steps < 1) return fail(RD_EINVAL, "cfl must be positive and n_steps >= 1");
  hipEvent_t ev[6];
  for (auto& e : ev) HIPCHK(hipEventCreate(&e));
  struct Free {
    hipEvent_t* e;
    ~Free() {
      for (int k = 0; k < 6; ++k) (void)hipEventDestroy(e[k]);
    }
  } guard{ev};
  for (int k = 0; k < 5; ++k) ms[k] = 0.0;
  for (int n = 0; n < n_steps; ++n) {
    HIPCHK(hipEventRecord(ev[0], m->stream));
    if ((st = rd3_stages(m, cfl, scheme, time, ev)) != RD_OK) return st;
    HIPCHK(hipStreamSynchronize(m->stream));
    const int last = time == RD_RK2 ? 5 : 3;
    for (int k = 0; k < last; ++k) {
      float t = 0.0f;
      HIPCHK(hipEventElapsedTime(&t, ev[k], ev[k + 1]));
      ms[k < 2 ? 1 - k : k] += t / n_steps;  // the CFL reduction follows the first tetrahedron pass
    }
  }
  return RD_OK;
}

RD_API rd_status rd3_sync(rd3_mesh* m) {
  if (!m) return fail(RD_EINVAL, "null mesh");
  int flag = 0;
  HIPCHK(hipMemcpyAsync(&flag, m->d.flag, sizeof(int), hipMemcpyDeviceToHost, m->stream));
  HIPCHK(hipStreamSynchronize(m->stream));
  if (flag) return fail(RD_ENONPHYS, "a non-physical state was produced");
  return RD_OK;
}

