// gfx950 kernels of the patch form of the step (bodies in rd_patch.h): one
// workgroup per patch, one thread per triangle and per owned vertex.
#include "rd_kcommon.h"
#include "rd_patch.h"
#include "rd_patch_launch.h"

namespace rd {

// A double moved between the lanes of a wave (DPP control CTRL; lanes with no
// source keep their own value).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
  const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
  const uint32_t h = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)((uint64_t)h << 32 | l));
}
// Minimum over a wave, in lane 63 (row shifts by 1, 2, 4, 8, then the last
// lanes of rows broadcast to the rows after them; all in registers, where a
// butterfly through LDS would wait on each of its six steps).
__device__ __forceinline__ double wave_min(double x) {
  x = rmin(x, dpp_move<0x111>(x));
  x = rmin(x, dpp_move<0x112>(x));
  x = rmin(x, dpp_move<0x114>(x));
  x = rmin(x, dpp_move<0x118>(x));
  x = rmin(x, dpp_move<0x142>(x));
  return rmin(x, dpp_move<0x143>(x));
}

// Minimum over the workgroup (at most 16 waves), valid in every thread. One
// barrier: a kernel that calls it twice gives each call its own red.
__device__ __forceinline__ double patch_min(double x, double* red) {
  x = wave_min(x);
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if ((threadIdx.x & 63) == 63) red[w] = x;
  __syncthreads();
  double y = red[0];
  for (int i = 1; i < nw; ++i) y = rmin(y, red[i]);
  return y;
}

// Internal id of local vertex l of a patch.
__device__ __forceinline__ int32_t patch_vertex(const Patches& p, const PatchDesc& q, int32_t l) {
  return l < q.own ? q.v0 + l : p.halo[q.h0 + l - q.own];
}

// f(j, slot of the j-th part) for the n parts of owned vertex l, eight loads
// ahead of their use.
template <class Get, class F>
__device__ __forceinline__ void patch_parts(const Patches& p, const PatchDesc& q, int32_t l, int32_t n, const Get& get,
                                            const F& f) {
  using T = decltype(get(0));
  T x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j < n) x[j] = get(q.jb8[j] + l);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j < n) f(x[j]);
  for (int32_t j = 8; j < n; ++j) f(get(p.jb[q.jb + j] + l));
}

// dt of the patch's mesh: given, reduced by k_patch_dt, or (p.cfl > 0) the
// minimum of the mesh's patch bounds taken here.
__device__ __forceinline__ double patch_dt(const Patches& p, int32_t m, const double* pmin) {
  if (p.dt_val > 0.0) return p.dt_val;
  if (!(p.cfl > 0.0)) return p.dt[m];
  __shared__ double red[16];
  double x = INFINITY;
  for (int32_t b = p.mbeg[m] + threadIdx.x; b < p.mbeg[m + 1]; b += blockDim.x) x = rmin(x, pmin[b]);
  return p.cfl * patch_min(x, red);
}

// LDS: vertex records first; the parts (and CFL terms) of owned corners over
// them, or behind them when the patch has more triangles than threads.
template <bool STAGE2, bool CFL>
__host__ __device__ inline size_t patch_vert_bytes(int32_t max_lv) {
  return (size_t)max_lv * (16 + 32 + (STAGE2 ? 64 : 0) + (CFL ? 8 : 0));
}

// A patch triangle's three words (local corner ids and part slots).
struct PatchTri {
  uint32_t w[3];
  __device__ __forceinline__ int32_t lv(int c) const { return (int32_t)(w[c] & 0xffffu); }
  __device__ __forceinline__ int32_t dst(int c) const { return (int32_t)(w[c] >> 16); }
  __device__ __forceinline__ bool owned(int c) const { return w[c] < 0xffff0000u; }
};
__device__ __forceinline__ PatchTri patch_tri(const Patches& p, int64_t at) {
  PatchTri t;
  for (int c = 0; c < 3; ++c) t.w[c] = p.tri[c * p.ptn + at];
  return t;
}

// What a thread needs of its owned vertex, loaded before the barrier that
// the parts wait for.
struct PatchOwn {
  double V = 0.0;
  int32_t deg = 0, wall = -1;
};
__device__ __forceinline__ PatchOwn patch_own(const Patches& p, const PatchDesc& q, int32_t l) {
  PatchOwn o;
  if (l < q.own) {
    const int64_t v = q.v0 + l;
    o.V = p.V[v];
    o.deg = p.deg[v];
    if (p.wb) o.wall = p.wb[v];
  }
  return o;
}

// Corner differences; only patches on a seam unwrap (elsewhere unwrapping
// changes nothing).
__device__ __forceinline__ TriDiff patch_diff(const Patches& p, const PatchDesc& q, const double2& a, const double2& b,
                                              const double2& c) {
  if (q.seam) return tri_diff(p, a, b, c);
  return TriDiff{b.x - a.x, b.y - a.y, c.x - a.x, c.y - a.y};
}

// Records of a patch's local vertices: those in LDS, or the i-th in memory.
template <bool MEM>
__device__ __forceinline__ auto patch_rec(const Patches& p, const PatchDesc& q, const Lds4& lds, int i) {
  if constexpr (MEM) return Mem4{p.rec + i * p.nloc + q.xy0};
  else return lds;
}

// The two passes of a step: one workgroup per patch, four waves per SIMD. (A
// grid of the workgroups the device holds at once, each walking a run of
// patches with the next one's records loaded ahead, was measured slower:
// 0.64 and 1.01 ms against 0.37 and 0.46 at 2048^2; what is live across the
// loop does not fit beside the triangle.)
// AFTER: the state is still one Euler step back; it is brought forward as the
// vertices are loaded (by every patch that holds them, alike) and written to
// the other buffer by their owner. A run of n Euler steps is then n passes and
// one update instead of n of each: 20 steps of the N scheme take 7.0 us a step
// against 9.9 at 64^2 and 308 against 406 at 2048^2.
// RES: the residual itself (sum of parts and wall term, ghosts' sums of parts
// too) in D's place.
// MEM: the wide patches (see Patches::wide) alone.
template <int SCHEME, bool CFL, bool AFTER, bool RES = false, bool MEM = false>
__global__ __launch_bounds__(kPatchThreads, 4) void k_patch1(Patches p) {
  extern __shared__ double2 lds[];
  const int c0 = p.cur[AFTER ? p.ci : 0];
  const D4* W = p.W[c0];
  const int32_t tid = threadIdx.x, nthr = blockDim.x;
  const bool big = !MEM && p.max_tri > nthr;
  const Lds4 Zl{lds, p.max_lv};
  double2* xy = lds + 2 * p.max_lv;
  double* sl = reinterpret_cast<double*>(xy + p.max_lv);
  const Lds4 P{big ? lds + patch_vert_bytes<false, CFL>(p.max_lv + (p.max_lv & 1)) / 16 : lds, p.max_slots};
  double* lam = reinterpret_cast<double*>(P.a + 2 * p.max_slots);
  if (blockIdx.x == 0 && tid == 0) {
    if (AFTER) p.cur[p.ci ^ 1] = c0 ^ 1;
    else p.cur[1] = c0;
  }
  const int32_t k = MEM ? p.wide[blockIdx.x] : (int32_t)xcd_block();
  const PatchDesc q = (MEM ? p.all : p.desc)[k];
  const auto Z = patch_rec<MEM>(p, q, Zl, 0);
  double* sig = MEM ? p.rsig + q.xy0 : sl;
  const double2* at = MEM ? p.xy + q.xy0 : xy;
  PatchTri t;  // loaded ahead of the vertices it indexes
  if (tid < q.nt) t = patch_tri(p, q.t0 + tid);
  const double dt = AFTER ? patch_dt(p, q.mesh, p.pminp) : 0.0;
  for (int32_t l = tid; l < q.nlv; l += nthr) {
    const int32_t v = patch_vertex(p, q, l);
    if (!MEM) xy[l] = p.xy[q.xy0 + l];
    double s;
    bool ok;
    const D4 w = AFTER ? patch_star(W[v], p.Dp[v], dt) : W[v];
    Z.set(l, patch_z(p, w, &s, &ok).v);
    if (CFL) sig[l] = s;
    if (AFTER && l < q.own) {
      p.W[c0 ^ 1][v] = w;
      if (!ok && p.V[v] > 0.0) p.flag[q.mesh] = 1;
    }
  }
  __syncthreads();
  for (int32_t j0 = 0; j0 < q.nt; j0 += nthr) {
    const int32_t j = j0 + tid;
    double out[3][4], term = 0.0;
    if (j0 > 0 && j < q.nt) t = patch_tri(p, q.t0 + j);
    if (j < q.nt) {
      const D4 z[3] = {Z.get(t.lv(0)), Z.get(t.lv(1)), Z.get(t.lv(2))};
      const TriDiff g = patch_diff(p, q, at[t.lv(0)], at[t.lv(1)], at[t.lv(2)]);
      if (CFL) term = rmax(rmax(sig[t.lv(0)], sig[t.lv(1)]), sig[t.lv(2)]);
      double pN[2][4], phi[4];
      const double lmax = stage1_parts<SCHEME>(g, z, p.gas, p.vr + 3 * q.mesh, out, pN, phi);
      if (CFL) term = lmax * term;
    }
    if (!big && !MEM) __syncthreads();
    if (j < q.nt)
      for (int c = 0; c < 3; ++c)
        if (t.owned(c)) {
          P.set(t.dst(c), out[c]);
          if (CFL) lam[t.dst(c)] = term;
        }
  }
  PatchOwn own = patch_own(p, q, tid);
  __syncthreads();
  double bound = INFINITY;
  for (int32_t l = tid; l < q.own; l += nthr) {
    if (l >= nthr) own = patch_own(p, q, l);
    const int64_t v = q.v0 + l;
    const double V = own.V;
    if (CFL) {
      double y = 0.0;
      patch_parts(p, q, l, own.deg, [&](int32_t s) { return lam[s]; }, [&](double a) { y += a; });
      bound = rmin(bound, 2.0 * fabs(V) * rcp(y));
    }
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    patch_parts(p, q, l, own.deg, [&](int32_t s) { return P.get(s); },
                [&](const D4& x) { for (int c = 0; c < 4; ++c) acc[c] += x.v[c]; });
    for (int c = 0; c < 4; ++c) acc[c] *= kSymScale;
    if (own.wall >= 0) {
      double wt[4];
      wall_term(p.went, p.wptr[own.wall], p.wptr[own.wall + 1], v, p.gamma,
                [&](int64_t i) { return AFTER ? patch_star(W[i], p.Dp[i], dt) : W[i]; }, wt);
      for (int c = 0; c < 4; ++c) acc[c] = acc[c] + wt[c];
    }
    const double f = V > 0.0 ? rcp(V) : 0.0;
    D4 o;
    for (int c = 0; c < 4; ++c) o.v[c] = RES ? acc[c] : (V > 0.0 ? f * acc[c] : 0.0);
    p.D[v] = o;
  }
  if (CFL) {
    __shared__ double red[16];
    bound = wave_min(bound);
    if ((tid & 63) == 63) red[tid >> 6] = bound;
    __syncthreads();
    if (tid == 0) {
      const int nw = (nthr + 63) >> 6;
      for (int i = 0; i < nw; ++i) bound = i ? rmin(bound, red[i]) : red[0];
      p.pmin[k] = bound;
    }
  }
}

template <int SCHEME, bool LUMP, bool MEM = false>
__global__ __launch_bounds__(kPatchThreads, 4) void k_patch2(Patches p) {
  extern __shared__ double2 lds[];
  const int c0 = p.cur[1];
  const D4* W = p.W[c0];
  D4* Wn = p.W[c0 ^ 1];
  const int32_t tid = threadIdx.x, nthr = blockDim.x;
  const bool big = !MEM && p.max_tri > nthr;
  const Lds4 Znl{lds, p.max_lv}, Zsl{lds + 2 * p.max_lv, p.max_lv}, Dl{lds + 4 * p.max_lv, p.max_lv};
  double2* xy = lds + 6 * p.max_lv;
  const Lds4 P{big ? lds + patch_vert_bytes<true, false>(p.max_lv + (p.max_lv & 1)) / 16 : lds, p.max_slots};
  if (blockIdx.x == 0 && tid == 0) p.cur[0] = c0 ^ 1;
  const PatchDesc q = MEM ? p.all[p.wide[blockIdx.x]] : p.desc[xcd_block()];
  const auto Zn = patch_rec<MEM>(p, q, Znl, 0), Zs = patch_rec<MEM>(p, q, Zsl, 1), D = patch_rec<MEM>(p, q, Dl, 2);
  const double2* at = MEM ? p.xy + q.xy0 : xy;
  PatchTri t;  // loaded ahead of the vertices it indexes
  if (tid < q.nt) t = patch_tri(p, q.t0 + tid);
  const double dt = patch_dt(p, q.mesh, p.pmin), idt = rcp(dt);
  for (int32_t l = tid; l < q.nlv; l += nthr) {
    const int32_t v = patch_vertex(p, q, l);
    if (!MEM) xy[l] = p.xy[q.xy0 + l];
    const D4 w = W[v], ws = patch_star(w, p.D[v], dt);
    Zn.set(l, patch_z(p, w, nullptr, nullptr).v);
    bool ok;
    Zs.set(l, patch_z(p, ws, nullptr, &ok).v);
    D.set(l, patch_rate(w, ws, idt).v);
    if (!ok && l < q.own) p.flag[q.mesh] = 1;
  }
  __syncthreads();
  for (int32_t j0 = 0; j0 < q.nt; j0 += nthr) {
    const int32_t j = j0 + tid;
    double out[3][4];
    if (j0 > 0 && j < q.nt) t = patch_tri(p, q.t0 + j);
    if (j < q.nt) {
      const TriDiff g = patch_diff(p, q, at[t.lv(0)], at[t.lv(1)], at[t.lv(2)]);
      patch_tri2<SCHEME, LUMP>(p, g, [&](int i) { return Zn.get(t.lv(i)); }, [&](int i) { return Zs.get(t.lv(i)); },
                               [&](int i) { return D.get(t.lv(i)); }, p.vr + 3 * q.mesh, out);
    }
    if (!big && !MEM) __syncthreads();
    if (j < q.nt)
      for (int c = 0; c < 3; ++c)
        if (t.owned(c)) P.set(t.dst(c), out[c]);
  }
  PatchOwn own = patch_own(p, q, tid);
  D4 wo, so;  // W^n and the stage-1 D of the owned vertex
  if (tid < q.own) {
    wo = W[q.v0 + tid];
    so = p.D[q.v0 + tid];
  }
  __syncthreads();
  for (int32_t l = tid; l < q.own; l += nthr) {
    const int64_t v = q.v0 + l;
    if (l >= nthr) {
      own = patch_own(p, q, l);
      wo = W[v];
      so = p.D[v];
    }
    const int32_t b = own.wall;
    const double V = own.V;
    const D4 ws = patch_star(wo, so, dt);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    patch_parts(p, q, l, own.deg, [&](int32_t s) { return P.get(s); },
                [&](const D4& x) { for (int c = 0; c < 4; ++c) acc[c] += x.v[c]; });
    if (b >= 0) {
      double wn[4], wt[4];
      wall_term(p.went, p.wptr[b], p.wptr[b + 1], v, p.gamma, [&](int64_t i) { return W[i]; }, wn);
      wall_term(p.went, p.wptr[b], p.wptr[b + 1], v, p.gamma,
                [&](int64_t i) { return patch_star(W[i], p.D[i], dt); }, wt);
      for (int c = 0; c < 4; ++c) acc[c] = acc[c] + 0.5 * (wn[c] + wt[c]);
    }
    D4 o = wo;
    if (V > 0.0) {
      const double f = dt * rcp(V);
      for (int c = 0; c < 4; ++c) o.v[c] = ws.v[c] - f * acc[c];
      if (!derive(p.gamma, o.v).ok) p.flag[q.mesh] = 1;
    }
    Wn[v] = o;
  }
}

// Forward Euler: W <- W - dt D in place, and cur[0] its buffer.
__global__ __launch_bounds__(kPatchThreads) void k_patch_euler(Patches p) {
  const int32_t k = (int32_t)xcd_block();
  const PatchDesc q = p.all[k];
  const int c0 = p.cur[p.ci];
  D4* W = p.W[c0];
  if (p.ci == 1 && blockIdx.x == 0 && threadIdx.x == 0) p.cur[0] = c0;
  const double dt = patch_dt(p, q.mesh, p.pmin);
  for (int32_t l = threadIdx.x; l < q.own; l += blockDim.x) {
    const int64_t v = q.v0 + l;
    const D4 o = patch_star(W[v], p.D[v], dt);
    W[v] = o;
    if (p.V[v] > 0.0 && !derive(p.gamma, o.v).ok) p.flag[q.mesh] = 1;
  }
}

// The smallest CFL bound alone (rd_max_dt): every patch its own and, with
// `done` (a count of workgroups, 0 between launches), the workgroup that
// finishes last the mesh's, into dt and straight into the host's memory.
__global__ __launch_bounds__(kPatchThreads) void k_patch_cfl(Patches p, double cfl, unsigned* done, double* host) {
  extern __shared__ double2 lds[];
  const int32_t k = (int32_t)xcd_block();
  const PatchDesc q = p.all[k];
  const int c0 = p.cur[0];
  const D4* W = p.W[c0 == kForm32 ? 0 : c0];  // a state in the FP32 form: its copy (launch_patch_copy)
  const int32_t tid = threadIdx.x, nthr = blockDim.x;
  double2* xy = lds;
  double* sig = reinterpret_cast<double*>(xy + p.all_lv);
  double* lam = sig + p.all_lv;
  for (int32_t l = tid; l < q.nlv; l += nthr) {
    const int32_t v = patch_vertex(p, q, l);
    xy[l] = p.xy[q.xy0 + l];
    sig[l] = derive(p.gamma, W[v].v).sig;
  }
  __syncthreads();
  for (int32_t j = tid; j < q.nt; j += nthr) {
    const PatchTri t = patch_tri(p, q.t0 + j);
    const TriDiff g = patch_diff(p, q, xy[t.lv(0)], xy[t.lv(1)], xy[t.lv(2)]);
    SymEdge<double> e[3];
    const double term =
        sym_edges(g.d1x, g.d1y, g.d2x, g.d2y, e) * rmax(rmax(sig[t.lv(0)], sig[t.lv(1)]), sig[t.lv(2)]);
    for (int c = 0; c < 3; ++c)
      if (t.owned(c)) lam[t.dst(c)] = term;
  }
  __syncthreads();
  double bound = INFINITY;
  for (int32_t l = tid; l < q.own; l += nthr) {
    double x = 0.0;
    patch_parts(p, q, l, p.deg[q.v0 + l], [&](int32_t s) { return lam[s]; }, [&](double a) { x += a; });
    bound = rmin(bound, 2.0 * fabs(p.V[q.v0 + l]) * rcp(x));
  }
  __shared__ double red[16];
  bound = patch_min(bound, red);
  __shared__ unsigned last;
  if (tid == 0) {
    p.pmin[k] = bound;
    if (done) __threadfence();
    last = done && atomicAdd(done, 1u) + 1u == gridDim.x;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  double x = INFINITY;
  for (int32_t b = tid; b < p.npatch; b += nthr) x = rmin(x, __hip_atomic_load(&p.pmin[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  __syncthreads();
  x = patch_min(x, red);
  if (tid == 0) {
    p.dt[0] = cfl * x;
    *host = cfl * x;
    *done = 0;
  }
}

// Per mesh: dt = cfl * the minimum of its patches' bounds.
__global__ __launch_bounds__(1024) void k_patch_dt(Patches p, double cfl, double* host) {
  const int m = blockIdx.x;
  double x = INFINITY;
  for (int32_t b = p.mbeg[m] + threadIdx.x; b < p.mbeg[m + 1]; b += blockDim.x) x = rmin(x, p.pmin[b]);
  __shared__ double red[16];
  x = patch_min(x, red);
  if (threadIdx.x == 0) {
    p.dt[m] = cfl * x;
    if (host) host[m] = cfl * x;
  }
}

// Smallest and largest flow speed |v| over each patch's vertices (the Bx
// sensor's range) at W^n, or at W* (STAR); then per mesh.
template <bool STAR>
__global__ __launch_bounds__(kPatchThreads) void k_patch_vrange(Patches p) {
  const int32_t k = (int32_t)xcd_block();
  const PatchDesc q = p.all[k];
  const D4* W = p.W[p.cur[STAR ? 1 : 0]];
  const double dt = !STAR || p.dt_val > 0.0 ? p.dt_val : p.dt[q.mesh];
  double lo = INFINITY, hi = 0.0;
  for (int32_t l = threadIdx.x; l < q.own; l += blockDim.x) {
    const int64_t v = q.v0 + l;
    const D4 w = STAR ? patch_star(W[v], p.D[v], dt) : W[v];
    const double sp = flow_speed(w);
    lo = rmin(lo, sp);
    hi = rmax(hi, sp);
  }
  __shared__ double red[32];
  lo = patch_min(lo, red);
  hi = -patch_min(-hi, red + 16);
  if (threadIdx.x == 0) {
    p.vpart[2 * k] = lo;
    p.vpart[2 * k + 1] = hi;
  }
}

__global__ __launch_bounds__(1024) void k_patch_vrange_final(Patches p) {
  const int m = blockIdx.x;
  double lo = INFINITY, hi = 0.0;
  for (int32_t b = p.mbeg[m] + threadIdx.x; b < p.mbeg[m + 1]; b += blockDim.x) {
    lo = rmin(lo, p.vpart[2 * b]);
    hi = rmax(hi, p.vpart[2 * b + 1]);
  }
  __shared__ double red[32];
  lo = patch_min(lo, red);
  hi = -patch_min(-hi, red + 16);
  if (threadIdx.x == 0) {
    p.vr[3 * m] = lo;
    p.vr[3 * m + 1] = hi;
  }
}

// The caller's [4][nv] arrays to the first state buffer and from the state,
// one thread per caller's vertex v (inv[v] is its internal vertex): the arrays
// are read and written in whole lines, the 32-byte records scattered. With
// `bad` nothing where it names a vertex.
__global__ __launch_bounds__(kBlock) void k_patch_set(Patches p, const int32_t* inv, const double* soa, const int* bad) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (bad && *bad < p.nv) return;
  if (v == 0) p.cur[0] = 0;
  if (v >= p.nv) return;
  D4 w;
  for (int k = 0; k < 4; ++k) w.v[k] = soa[k * p.nv + v];
  p.W[0][inv[v]] = w;
  if (!derive(p.gamma, w.v).ok) p.flag[0] = 1;
}

__global__ __launch_bounds__(kBlock) void k_state_get(State st, int64_t nv, double* soa) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v >= nv) return;
  const D4 w = *st.at(v);
  for (int k = 0; k < 4; ++k) soa[k * nv + v] = w.v[k];
}

// The same with records in the caller's order.
__global__ __launch_bounds__(kBlock) void k_state_get4(State st, int64_t nv, D4* out) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v < nv) out[v] = *st.at(v);
}
__global__ __launch_bounds__(kBlock) void k_patch_set4(Patches p, const int32_t* inv, const D4* in) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v < p.nv) p.W[0][inv[v]] = in[v];
}

__global__ __launch_bounds__(kBlock) void k_patch_enter(State st, int64_t nv) {
  const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (v < nv && *st.cur == kForm32) st.W[0][st.inv[v]] = *st.at(v);
}
__global__ void k_patch_entered(int* cur) {
  if (cur[0] == kForm32) cur[0] = 0;
}

// Batch: the states of all members into (or out of) the batch. Block b covers
// kBlock vertices of member mb[b], from its vertex vb[b] on.
__global__ __launch_bounds__(kBlock) void k_patch_members(State st, int* cur, int* flags, const PatchMember* mem,
                                                          const int32_t* mb, const int32_t* vb, int out) {
  const int32_t m = mb[blockIdx.x];
  const PatchMember q = mem[m];
  const int64_t v = vb[blockIdx.x] + (int64_t)threadIdx.x;  // the caller's vertex of the member
  if (v == 0) {  // words that no thread of this launch reads
    if (!out) flags[m] = 0;
    else if (flags[m]) *q.flag = 1;
    if (out) *q.cur = 0;
    else if (m == 0) *cur = 0;
  }
  if (v >= q.nv) return;
  const int64_t u = q.v0 + v;  // the caller's vertex of the batch
  if (out) q.st.W[0][q.st.inv[v]] = *st.at(u);
  else st.W[0][st.inv[u]] = *q.st.at(v);
}

// ------------------------------------------------------------- launchers --

size_t patch_lds_bytes(const Patches& p, int stage, bool cfl, bool wide) {
  const int32_t lv = p.max_lv + (p.max_lv & 1);
  const size_t vert = stage == 2 ? patch_vert_bytes<true, false>(lv)
                                 : (cfl ? patch_vert_bytes<false, true>(lv) : patch_vert_bytes<false, false>(lv));
  const size_t parts = (size_t)p.max_slots * (stage == 1 && cfl ? 40 : 32);
  if (wide) return parts;
  return p.max_tri > p.threads ? vert + parts : (vert > parts ? vert : parts);
}

enum { kStep, kAfter, kResidual };

template <int SCHEME, bool MEM>
static hipError_t patch_go(const Patches& p, int what, int stage, bool cfl, hipStream_t s) {
  const dim3 g(MEM ? p.nwide : p.npatch), b(p.threads);
  const size_t lds = patch_lds_bytes(p, stage, cfl, MEM);
  if (what == kResidual) hipLaunchKernelGGL((k_patch1<SCHEME, false, false, true, MEM>), g, b, lds, s, p);
  else if (what == kAfter) {
    if constexpr (SCHEME == SCH_BX) return hipErrorInvalidValue;
    else hipLaunchKernelGGL((k_patch1<SCHEME, true, true, false, MEM>), g, b, lds, s, p);
  } else if (stage == 2 && p.slump) hipLaunchKernelGGL((k_patch2<SCHEME, true, MEM>), g, b, lds, s, p);
  else if (stage == 2) hipLaunchKernelGGL((k_patch2<SCHEME, false, MEM>), g, b, lds, s, p);
  else if (cfl) hipLaunchKernelGGL((k_patch1<SCHEME, true, false, false, MEM>), g, b, lds, s, p);
  else hipLaunchKernelGGL((k_patch1<SCHEME, false, false, false, MEM>), g, b, lds, s, p);
  return hipGetLastError();
}

template <int SCHEME>
static hipError_t patch_go(const Patches& p, int what, int stage, bool cfl, hipStream_t s) {
  const hipError_t e = patch_go<SCHEME, false>(p, what, stage, cfl, s);
  return e == hipSuccess && p.nwide ? patch_go<SCHEME, true>(p, what, stage, cfl, s) : e;
}

static hipError_t patch_go(const Patches& p, int scheme, int what, int stage, bool cfl, hipStream_t s) {
  switch (scheme) {
    case SCH_N: return patch_go<SCH_N>(p, what, stage, cfl, s);
    case SCH_LDA: return patch_go<SCH_LDA>(p, what, stage, cfl, s);
    case SCH_B: return patch_go<SCH_B>(p, what, stage, cfl, s);
    case SCH_BMAX: return patch_go<SCH_BMAX>(p, what, stage, cfl, s);
    case SCH_BMIN: return patch_go<SCH_BMIN>(p, what, stage, cfl, s);
    case SCH_BX: return patch_go<SCH_BX>(p, what, stage, cfl, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_patch_residual(const Patches& p, int scheme, hipStream_t s) {
  return patch_go(p, scheme, kResidual, 1, false, s);
}

hipError_t launch_patch_after(const Patches& p, int scheme, hipStream_t s) {
  return patch_go(p, scheme, kAfter, 1, true, s);
}

hipError_t launch_patch(const Patches& p, int scheme, int stage, bool cfl, hipStream_t s) {
  return patch_go(p, scheme, kStep, stage, cfl, s);
}

hipError_t launch_patch_euler(const Patches& p, hipStream_t s) {
  hipLaunchKernelGGL(k_patch_euler, dim3(p.npatch), dim3(p.threads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_patch_cfl(const Patches& p, double cfl, unsigned* done, double* host, hipStream_t s) {
  const size_t lds = (size_t)p.all_lv * 24 + (size_t)p.max_slots * 8;
  hipLaunchKernelGGL(k_patch_cfl, dim3(p.npatch), dim3(p.threads), lds, s, p, cfl, done, host);
  return hipGetLastError();
}

hipError_t launch_patch_dt(const Patches& p, double cfl, hipStream_t s, double* host) {
  hipLaunchKernelGGL(k_patch_dt, dim3(p.nmesh), dim3(1024), 0, s, p, cfl, host);
  return hipGetLastError();
}

hipError_t launch_patch_vrange(const Patches& p, bool star, hipStream_t s) {
  if (star) hipLaunchKernelGGL(k_patch_vrange<true>, dim3(p.npatch), dim3(p.threads), 0, s, p);
  else hipLaunchKernelGGL(k_patch_vrange<false>, dim3(p.npatch), dim3(p.threads), 0, s, p);
  hipLaunchKernelGGL(k_patch_vrange_final, dim3(p.nmesh), dim3(1024), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_patch_set(const Patches& p, const int32_t* inv, const double* soa, const int* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_patch_set, dim3(nblk(p.nv)), dim3(kBlock), 0, s, p, inv, soa, bad);
  return hipGetLastError();
}
hipError_t launch_state_get(const State& st, int64_t nv, double* soa, hipStream_t s) {
  hipLaunchKernelGGL(k_state_get, dim3(nblk(nv)), dim3(kBlock), 0, s, st, nv, soa);
  return hipGetLastError();
}
hipError_t launch_state_get4(const State& st, int64_t nv, D4* out, hipStream_t s) {
  hipLaunchKernelGGL(k_state_get4, dim3(nblk(nv)), dim3(kBlock), 0, s, st, nv, out);
  return hipGetLastError();
}
hipError_t launch_patch_set4(const Patches& p, const int32_t* inv, const D4* in, hipStream_t s) {
  hipLaunchKernelGGL(k_patch_set4, dim3(nblk(p.nv)), dim3(kBlock), 0, s, p, inv, in);
  return hipGetLastError();
}
hipError_t launch_patch_copy(const Patches& p, const State& st, hipStream_t s) {
  hipLaunchKernelGGL(k_patch_enter, dim3(nblk(p.nv)), dim3(kBlock), 0, s, st, p.nv);
  return hipGetLastError();
}
hipError_t launch_patch_enter(const Patches& p, const State& st, hipStream_t s) {
  hipLaunchKernelGGL(k_patch_enter, dim3(nblk(p.nv)), dim3(kBlock), 0, s, st, p.nv);
  hipLaunchKernelGGL(k_patch_entered, dim3(1), dim3(1), 0, s, p.cur);
  return hipGetLastError();
}
hipError_t launch_patch_members(const State& st, int* cur, int* flags, int64_t nv, const PatchMember* mem, const int32_t* mb, const int32_t* vb, int nblocks, bool out,
                                hipStream_t s) {
  if (nv == 0) return hipSuccess;
  hipLaunchKernelGGL(k_patch_members, dim3(nblocks), dim3(kBlock), 0, s, st, cur, flags, mem, mb, vb, out ? 1 : 0);
  return hipGetLastError();
}

}  // namespace rd
