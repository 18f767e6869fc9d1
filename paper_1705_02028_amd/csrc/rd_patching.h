// Host-side construction of the vertex patches of the step (rd_patch.h).
//
// The vertices of each mesh are split into compact groups by recursive
// coordinate bisection: a group that is to become n patches is cut across the
// longer side of its bounding box into floor(n/2) and ceil(n/2) patches' worth
// of vertices, the cut moved to the nearest gap between two distinct
// coordinates (so that a lattice is cut into whole rows and columns). A patch
// owns its vertices; its triangles are all those with an owned corner, so
// that it can finish its own vertices without any other patch, and its halo
// are the other corners of those triangles. Triangles on a border belong to
// several patches. The vertices are renumbered patch by patch, within a patch
// by descending degree, then ascending caller's id.
#pragma once

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <new>
#include <memory>
#include <new>
#include <string>
#include <thread>
#include <vector>

namespace rd {

// Vector whose new elements are left as they are: large tables that several
// threads then fill (and so map into memory) together.
template <class T>
struct NoInit : std::allocator<T> {
  template <class U>
  struct rebind {
    using other = NoInit<U>;
  };
  template <class U>
  void construct(U*) noexcept {}
  template <class U, class... A>
  void construct(U* p, A&&... a) {
    ::new (static_cast<void*>(p)) U(std::forward<A>(a)...);
  }
};
template <class T>
using UVec = std::vector<T, NoInit<T>>;

struct PatchPlan {
  int32_t npatch = 0;
  int32_t max_tri = 0;                 // triangles of the largest patch
  int32_t max_lv = 0, max_slots = 0;   // local vertices and part slots of the largest patches
  UVec<int32_t> order;                 // [nv] internal vertex -> caller's vertex
  std::vector<int32_t> vbeg;           // [npatch + 1] owned internal vertices of each patch
  std::vector<int32_t> hbeg, halo;     // halo (internal ids) of each patch, ascending
  std::vector<int32_t> tbeg;           // [npatch + 1] patch triangles
  UVec<uint32_t> tri;                  // [3][patch triangle]: per corner its local id, and its part slot << 16 (0xffff: not owned)
  UVec<int32_t> tid;                   // caller's triangle of each patch triangle, or -1 - t where another patch owns it
  // Part slots of a patch: its vertices stand in descending degree, and the
  // j-th parts (ascending triangle) of those that have one are consecutive:
  // slot = jb[jbeg[k] + j] + local vertex.
  UVec<uint16_t> deg;                  // [nv] triangles of each owned vertex
  std::vector<int32_t> jbeg, jb;
  std::vector<int32_t> pmesh;          // [npatch] mesh of each patch
  std::vector<uint8_t> seam;           // [npatch] 1: some triangle has a corner difference beyond half a period
  std::vector<int32_t> mbeg;           // [nmesh + 1] patches of each mesh
};

struct PatchInput {
  int64_t nv = 0, nt = 0;
  const int32_t* tri = nullptr;  // [nt][3]
  const double *x = nullptr, *y = nullptr;
  double hpx = INFINITY, hpy = INFINITY;          // half periods, infinite on an axis that is not periodic
  const int32_t *row = nullptr, *slot = nullptr;  // vertex -> corner CSR (corner 3 t + i), ascending t in each row
  const std::vector<int64_t>*voff = nullptr, *toff = nullptr;
  int32_t max_tri = 512;  // a patch with more triangles is cut again (one vertex at least)
  int32_t own = 0;        // wanted owned vertices per patch
  int threads = 1;
};

// f(q) for q = 0 .. w - 1, each on a thread of its own where one can be
// had; what a worker throws (memory) is thrown again here.
template <class F>
void run_workers(int w, const F& f) {
  std::atomic<bool> failed{false};
  auto safe = [&](int q) {
    try {
      f(q);
    } catch (...) {
      failed = true;
    }
  };
  std::vector<std::thread> t;
  t.reserve(w);
  for (int q = 1; q < w; ++q) {
    try {
      t.emplace_back(safe, q);
    } catch (...) {
      safe(q);
    }
  }
  safe(0);
  for (auto& x : t) x.join();
  if (failed) throw std::bad_alloc();
}

class PatchBuilder {
 public:
  PatchBuilder(const PatchInput& in, PatchPlan& P) : in_(in), P_(P) {}

  std::string build() {
    const size_t nmesh = in_.voff->size() - 1;
    P_ = PatchPlan();
    P_.order.resize(in_.nv);
    pts_.resize(in_.nv);
    parallel(in_.nv, [&](int64_t i) { pts_[i] = Point{in_.x[i], in_.y[i], (int32_t)i}; });
    // groups: per mesh a list of group bounds, found by bisection in parallel
    std::vector<int64_t> cuts;  // group starts
    std::vector<int32_t> mesh_groups(nmesh + 1, 0);
    for (size_t k = 0; k < nmesh; ++k) {
      const int64_t n = std::max<int64_t>(1, ((*in_.voff)[k + 1] - (*in_.voff)[k] + in_.own - 1) / in_.own);
      mesh_groups[k + 1] = mesh_groups[k] + (int32_t)n;
    }
    const int64_t ngroups = mesh_groups[nmesh];
    cuts.assign(ngroups + 1, in_.nv);
    if (nmesh == 1) {
      if (in_.threads > 1) swap_.resize(in_.nv);
      bisect(0, in_.nv, 0, ngroups, cuts, in_.threads);
      UVec<Point>().swap(swap_);
    } else {
      parallel((int64_t)nmesh, [&](int64_t k) {
        bisect((*in_.voff)[k], (*in_.voff)[k + 1], mesh_groups[k], mesh_groups[k + 1], cuts, 1);
      });
    }
    // groups whose triangles exceed the limit are cut again; every piece is ordered by degree and caller's id
    gof_.resize(in_.nv);
    parallel(ngroups, [&](int64_t g) {
      for (int64_t i = cuts[g]; i < cuts[g + 1]; ++i) gof_[pts_[i].id] = (int32_t)g;
    });
    std::vector<std::vector<int64_t>> pieces(ngroups);
    std::vector<std::vector<int32_t>> tris(ngroups);  // of the groups left whole
    parallel(ngroups, [&](int64_t g) {
      group_triangles((int32_t)g, cuts[g], cuts[g + 1], tris[g]);
      if ((int64_t)tris[g].size() <= in_.max_tri || cuts[g + 1] - cuts[g] == 1) {
        pieces[g] = {cuts[g]};
      } else {
        pieces[g] = split_to_fit(cuts[g], cuts[g + 1]);
        tris[g].clear();
      }
      for (int64_t i = cuts[g]; i < cuts[g + 1]; ++i) P_.order[i] = pts_[i].id;
      for (size_t q = 0; q < pieces[g].size(); ++q) {
        const int64_t b = pieces[g][q], e = q + 1 < pieces[g].size() ? pieces[g][q + 1] : cuts[g + 1];
        std::sort(P_.order.begin() + b, P_.order.begin() + e, [&](int32_t p, int32_t r) {
          const int32_t dp = in_.row[p + 1] - in_.row[p], dr = in_.row[r + 1] - in_.row[r];
          return dp > dr || (dp == dr && p < r);
        });
      }
    });
    P_.mbeg.push_back(0);
    for (size_t k = 0; k < nmesh; ++k) {
      for (int32_t g = mesh_groups[k]; g < mesh_groups[k + 1]; ++g)
        for (int64_t b : pieces[g]) {
          tris_.emplace_back();
          if (pieces[g].size() == 1) tris_.back().swap(tris[g]);
          P_.vbeg.push_back((int32_t)b);
          P_.pmesh.push_back((int32_t)k);
        }
      P_.mbeg.push_back((int32_t)P_.vbeg.size());
    }
    P_.npatch = (int32_t)P_.vbeg.size();
    P_.vbeg.push_back((int32_t)in_.nv);
    UVec<Point>().swap(pts_);
    UVec<int32_t>().swap(gof_);
    return fill();
  }

 private:
  const PatchInput& in_;
  PatchPlan& P_;
  struct Point {
    double x, y;
    int32_t id;
  };
  UVec<Point> pts_, swap_;  // vertices, partitioned as the order is found; room for parallel cuts
  std::vector<std::vector<int32_t>> tris_;  // triangles of each patch (empty: still to be found)
  UVec<int32_t> gof_;       // group of each of the caller's vertices

  template <class F>
  void parallel(int64_t n, const F& f) {
    const int w = (int)std::max<int64_t>(1, std::min<int64_t>(in_.threads, n));
    run_workers(w, [&](int q) {
      for (int64_t i = n * q / w; i < n * (q + 1) / w; ++i) f(i);
    });
  }

  // Position in [b, e) of the cut that leaves about `want` vertices before
  // it, pts[b, e) partitioned around it along the longer side; on several
  // threads by a histogram of the coordinate first.
  int64_t cut(int64_t b, int64_t e, int64_t want, int64_t lo, int64_t hi, int threads = 1) {
    struct Box {
      double x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    };
    const int w = threads > 1 && e - b > 100000 ? threads : 1;
    std::vector<Box> box(w);
    auto share = [&](int q) { return b + (e - b) * q / w; };
    run_workers(w, [&](int q) {
      Box B;
      for (int64_t i = share(q); i < share(q + 1); ++i) {
        B.x0 = std::min(B.x0, pts_[i].x);
        B.x1 = std::max(B.x1, pts_[i].x);
        B.y0 = std::min(B.y0, pts_[i].y);
        B.y1 = std::max(B.y1, pts_[i].y);
      }
      box[q] = B;
    });
    Box B;
    for (const Box& o : box) {
      B.x0 = std::min(B.x0, o.x0);
      B.x1 = std::max(B.x1, o.x1);
      B.y0 = std::min(B.y0, o.y0);
      B.y1 = std::max(B.y1, o.y1);
    }
    const bool ax = B.x1 - B.x0 >= B.y1 - B.y0;
    auto co = [ax](const Point& p) { return ax ? p.x : p.y; };
    auto less = [&](const Point& p, const Point& q) { return co(p) < co(q) || (co(p) == co(q) && p.id < q.id); };
    int64_t u = b, v = e;  // the cut lies in [u, v), in place around it
    const int64_t m = b + want;
    if (w > 1) {
      constexpr int kBins = 4096;
      const double c0 = ax ? B.x0 : B.y0, len = (ax ? B.x1 : B.y1) - c0, f = len > 0.0 ? kBins / len : 0.0;
      auto bin = [&](const Point& p) { return std::min(kBins - 1, (int)((co(p) - c0) * f)); };
      std::vector<std::vector<int64_t>> count(w);
      run_workers(w, [&](int q) {
        count[q].assign(kBins, 0);
        for (int64_t i = share(q); i < share(q + 1); ++i) ++count[q][bin(pts_[i])];
      });
      int64_t before = b;
      int at = 0;
      for (;; ++at) {
        int64_t n = 0;
        for (int q = 0; q < w; ++q) n += count[q][at];
        if (before + n > m) {
          u = before;
          v = before + n;
          break;
        }
        before += n;
      }
      // three runs: bins below, the bin of the cut, bins above
      std::vector<int64_t> p0(w), p1(w), p2(w);
      int64_t a0 = b, a1 = u, a2 = v;
      for (int q = 0; q < w; ++q) {
        int64_t below = 0;
        for (int k = 0; k < at; ++k) below += count[q][k];
        p0[q] = a0;
        p1[q] = a1;
        p2[q] = a2;
        a0 += below;
        a1 += count[q][at];
        a2 += share(q + 1) - share(q) - below - count[q][at];
      }
      run_workers(w, [&](int q) {
        int64_t x = p0[q], y = p1[q], z = p2[q];
        for (int64_t i = share(q); i < share(q + 1); ++i) {
          const int k = bin(pts_[i]);
          swap_[k < at ? x++ : (k == at ? y++ : z++)] = pts_[i];
        }
      });
      run_workers(w, [&](int q) {
        std::copy(swap_.begin() + share(q), swap_.begin() + share(q + 1), pts_.begin() + share(q));
      });
    }
    auto o = pts_.begin();
    std::nth_element(o + u, o + m, o + v, less);
    // the run of vertices with the coordinate of the cut: move the cut to its nearer end
    const double at = co(pts_[m]);
    int64_t below = u - b, same = 0;
    for (int64_t i = u; i < v; ++i) {
      below += co(pts_[i]) < at;
      same += co(pts_[i]) == at;
    }
    int64_t k = m;
    const int64_t k0 = b + below, k1 = k0 + same;
    if (m - k0 <= k1 - m && k0 >= b + lo && k0 <= b + hi) k = k0;
    else if (k1 >= b + lo && k1 <= b + hi) k = k1;
    else if (k0 >= b + lo && k0 <= b + hi) k = k0;
    if (k != m && k > u && k < v) std::nth_element(o + u, o + k, o + v, less);
    return k;
  }

  // Cuts order[b, e) into groups g0 .. g1 - 1; cuts[g] receives their starts.
  void bisect(int64_t b, int64_t e, int64_t g0, int64_t g1, std::vector<int64_t>& cuts, int threads) {
    const int64_t n = g1 - g0;
    if (n == 1) {
      cuts[g0] = b;
      return;
    }
    const int64_t na = n / 2, nb = n - na;
    // a snapped cut may move by at most an eighth of the smaller side's vertices
    const int64_t len = e - b, want = len * na / n;
    const int64_t slack = std::min(want, len - want) / 8;
    const int64_t lo = std::max(na, want - slack), hi = std::min(len - nb, want + slack);
    const int64_t k = cut(b, e, std::min(std::max(want, na), len - nb), lo, hi, threads);
    run_workers(threads > 1 ? 2 : 1, [&](int q) {
      if (threads > 1) {
        if (q == 0) bisect(b, k, g0, g0 + na, cuts, threads / 2);
        else bisect(k, e, g0 + na, g1, cuts, threads - threads / 2);
      } else {
        bisect(b, k, g0, g0 + na, cuts, 1);
        bisect(k, e, g0 + na, g1, cuts, 1);
      }
    });
  }

  // Triangles of a whole group: each taken at its corner of least id in it.
  void group_triangles(int32_t g, int64_t b, int64_t e, std::vector<int32_t>& T) const {
    T.reserve(2 * (e - b) + 2 * in_.own / 7 + 16);
    for (int64_t i = b; i < e; ++i) {
      const int32_t v = pts_[i].id;
      for (int32_t j = in_.row[v]; j < in_.row[v + 1]; ++j) {
        const int32_t t = in_.slot[j] / 3;
        const int32_t* c = in_.tri + 3 * (int64_t)t;
        bool first = true;
        for (int q = 0; q < 3; ++q) first = first && !(c[q] < v && gof_[c[q]] == g);
        if (first) T.push_back(t);
      }
    }
    std::sort(T.begin(), T.end());
  }

  std::vector<int64_t> split_to_fit(int64_t b, int64_t e) {
    if (e - b <= 1) return {b};
    std::vector<int32_t> t;
    for (int64_t i = b; i < e; ++i)
      for (int32_t j = in_.row[pts_[i].id]; j < in_.row[pts_[i].id + 1]; ++j) t.push_back(in_.slot[j] / 3);
    std::sort(t.begin(), t.end());
    if (std::unique(t.begin(), t.end()) - t.begin() <= in_.max_tri) return {b};
    const int64_t len = e - b, want = len / 2, slack = want / 8;
    const int64_t k = cut(b, e, want, std::max<int64_t>(1, want - slack), std::min(len - 1, want + slack));
    std::vector<int64_t> out = split_to_fit(b, k), more = split_to_fit(k, e);
    out.insert(out.end(), more.begin(), more.end());
    return out;
  }

  // Triangles, halo and part slots of every patch.
  std::string fill() {
    const int32_t np = P_.npatch;
    UVec<int32_t> inv(in_.nv);
    parallel(in_.threads, [&](int64_t q) {
      for (int64_t i = in_.nv * q / in_.threads; i < in_.nv * (q + 1) / in_.threads; ++i) inv[P_.order[i]] = (int32_t)i;
    });
    UVec<int32_t> pof(in_.nv);  // patch of each internal vertex
    parallel(np, [&](int64_t k) {
      for (int32_t i = P_.vbeg[k]; i < P_.vbeg[k + 1]; ++i) pof[i] = (int32_t)k;
    });
    // counts, then contents: a triangle is taken at its first owned corner
    P_.tbeg.assign(np + 1, 0);
    P_.hbeg.assign(np + 1, 0);
    P_.deg.resize(in_.nv);
    std::vector<std::vector<int32_t>>&tris = tris_, halos(np);
    std::vector<int32_t> slots(np);
    parallel(np, [&](int64_t k) {
      std::vector<int32_t>&T = tris[k], &H = halos[k];
      const int32_t v0 = P_.vbeg[k], v1 = P_.vbeg[k + 1];
      int32_t s = 0;
      const bool known = !T.empty();
      for (int32_t i = v0; i < v1; ++i) {
        const int32_t v = P_.order[i];
        P_.deg[i] = (uint16_t)(in_.row[v + 1] - in_.row[v]);
        s += in_.row[v + 1] - in_.row[v];
        if (!known)
          for (int32_t j = in_.row[v]; j < in_.row[v + 1]; ++j) T.push_back(in_.slot[j] / 3);
      }
      if (!known) {
        std::sort(T.begin(), T.end());
        T.erase(std::unique(T.begin(), T.end()), T.end());
      }
      for (int32_t t : T)
        for (int c = 0; c < 3; ++c) {
          const int32_t w = inv[in_.tri[3 * (int64_t)t + c]];
          if (w < v0 || w >= v1) H.push_back(w);
        }
      slots[k] = s;
      std::sort(H.begin(), H.end());
      H.erase(std::unique(H.begin(), H.end()), H.end());
    });
    int64_t nt = 0, nh = 0;
    for (int32_t k = 0; k < np; ++k) {
      nt += (int64_t)tris[k].size();
      nh += (int64_t)halos[k].size();
      if (nt >= (int64_t(1) << 31) || nh >= (int64_t(1) << 31)) return "too many patch triangles";
      const int32_t lv = P_.vbeg[k + 1] - P_.vbeg[k] + (int32_t)halos[k].size();
      if (lv >= 65535 || slots[k] >= 65535) return "a patch has too many vertices";
      P_.tbeg[k + 1] = (int32_t)nt;
      P_.hbeg[k + 1] = (int32_t)nh;
      P_.max_tri = std::max(P_.max_tri, (int32_t)tris[k].size());
      P_.max_lv = std::max(P_.max_lv, lv);
      P_.max_slots = std::max(P_.max_slots, slots[k]);
    }
    P_.jbeg.assign(np + 1, 0);
    for (int32_t k = 0; k < np; ++k) {  // the first owned vertex has the largest degree
      int32_t base = 0;
      int32_t n = P_.vbeg[k + 1] - P_.vbeg[k];
      for (int32_t j = 0; j < P_.deg[P_.vbeg[k]]; ++j) {
        while (n > 0 && P_.deg[P_.vbeg[k] + n - 1] <= j) --n;
        P_.jb.push_back(base);
        base += n;
      }
      P_.jbeg[k + 1] = (int32_t)P_.jb.size();
    }
    P_.tri.resize(3 * nt);
    P_.tid.resize(nt);
    P_.seam.assign(np, 0);
    P_.halo.resize(nh);
    parallel(np, [&](int64_t k) {
      const std::vector<int32_t>&T = tris[k], &H = halos[k];
      const int32_t v0 = P_.vbeg[k], v1 = P_.vbeg[k + 1], own = v1 - v0;
      std::copy(H.begin(), H.end(), P_.halo.begin() + P_.hbeg[k]);
      const int32_t* jb = P_.jb.data() + P_.jbeg[k];
      std::vector<uint16_t> next(own, 0);  // triangles are ascending: ranks in order of appearance
      for (size_t j = 0; j < T.size(); ++j) {
        const int64_t at = P_.tbeg[k] + (int64_t)j;
        int32_t owner = INT32_MAX;
        for (int c = 0; c < 3; ++c) {
          const int32_t w = inv[in_.tri[3 * (int64_t)T[j] + c]];
          owner = std::min(owner, pof[w]);
          uint16_t lv, dst;
          if (w >= v0 && w < v1) {
            lv = (uint16_t)(w - v0);
            dst = (uint16_t)(jb[next[w - v0]++] + lv);
          } else {
            lv = (uint16_t)(own + (std::lower_bound(H.begin(), H.end(), w) - H.begin()));
            dst = 0xffff;
          }
          P_.tri[c * nt + at] = lv | (uint32_t)dst << 16;
        }
        P_.tid[at] = owner == k ? T[j] : -1 - T[j];
        const int32_t* c = in_.tri + 3 * (int64_t)T[j];
        for (int i = 1; i < 3; ++i)
          if (std::fabs(in_.x[c[i]] - in_.x[c[0]]) > in_.hpx || std::fabs(in_.y[c[i]] - in_.y[c[0]]) > in_.hpy)
            P_.seam[k] = 1;
      }
      std::vector<int32_t>().swap(tris[k]);
    });
    return std::string();
  }
};

inline std::string build_patch_plan(const PatchInput& in, PatchPlan& P) { return PatchBuilder(in, P).build(); }

}  // namespace rd
