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
#include <array>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdint>
#include <memory>
#include <mutex>
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

class Workers;

struct PatchPlan {
  int32_t npatch = 0;
  int32_t max_tri = 0;                 // triangles of the largest patch
  int32_t max_lv = 0, max_slots = 0;   // local vertices and part slots of the largest patches
  UVec<int32_t> order, inv;            // [nv] internal vertex -> caller's vertex, and back
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
  Workers* workers = nullptr;  // these instead, where given
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

// A few threads that run one function after another: f(q) for q = 0 .. size() -
// 1, the caller's thread among them. They are started by the first run and
// live as long as the object (starting eight costs about as much as building
// the plan of a small mesh); between runs that follow each other at once they
// spin, then sleep. One run at a time, none from within another.
class Workers {
 public:
  explicit Workers(int n) : n_(std::max(1, n)) {}
  Workers(const Workers&) = delete;
  Workers& operator=(const Workers&) = delete;
  ~Workers() {
    if (t_.empty()) return;
    {
      std::lock_guard<std::mutex> g(m_);
      stop_ = true;
      gen_.fetch_add(1);
    }
    cv_.notify_all();
    for (auto& x : t_) x.join();
  }
  int size() const { return n_; }

  // What a worker throws (memory) is thrown again here.
  template <class F>
  void run(const F& f) {
    if (n_ == 1) {
      f(0);
      return;
    }
    start();
    failed_ = false;
    arg_ = &f;
    call_ = [](const void* p, int q) { (*static_cast<const F*>(p))(q); };
    left_.store((int)t_.size());
    {
      std::lock_guard<std::mutex> g(m_);
      gen_.fetch_add(1);
    }
    cv_.notify_all();
    one(0);
    for (int q = (int)t_.size() + 1; q < n_; ++q) one(q);  // threads that could not be had
    for (int k = 0; left_.load() > 0; ++k)
      if (k > kSpin) std::this_thread::yield();
    if (failed_) throw std::bad_alloc();
  }

  // f(i) for i = 0 .. n - 1, in equal shares
  template <class F>
  void each(int64_t n, const F& f) {
    run([&](int q) {
      for (int64_t i = n * q / n_; i < n * (q + 1) / n_; ++i) f(i);
    });
  }

 private:
  static constexpr int kSpin = 2000;
  const int n_;
  std::vector<std::thread> t_;
  std::mutex m_;
  std::condition_variable cv_;
  std::atomic<uint32_t> gen_{0};
  std::atomic<int> left_{0};
  std::atomic<bool> failed_{false};
  bool stop_ = false, started_ = false;
  const void* arg_ = nullptr;
  void (*call_)(const void*, int) = nullptr;

  void one(int q) {
    try {
      call_(arg_, q);
    } catch (...) {
      failed_ = true;
    }
  }
  void start() {
    if (started_) return;
    started_ = true;
    t_.reserve(n_ - 1);
    for (int q = 1; q < n_; ++q) {
      try {
        t_.emplace_back([this, q] { loop(q); });
      } catch (...) {
        break;
      }
    }
  }
  void loop(int q) {
    for (uint32_t seen = 0;;) {
      for (int k = 0; k < kSpin && gen_.load() == seen; ++k) std::this_thread::yield();
      if (gen_.load() == seen) {
        std::unique_lock<std::mutex> g(m_);
        cv_.wait(g, [&] { return gen_.load() != seen; });
      }
      seen = gen_.load();
      if (stop_) return;
      one(q);
      left_.fetch_sub(1);
    }
  }
};

class PatchBuilder {
 public:
  PatchBuilder(const PatchInput& in, PatchPlan& P) : in_(in), P_(P), own_(in.threads), w_(in.workers ? *in.workers : own_) {}

  std::string build() {
    const size_t nmesh = in_.voff->size() - 1;
    P_ = PatchPlan();
    P_.order.resize(in_.nv);
    pts_.resize(in_.nv);
    swap_.resize(in_.nv);
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
      points(0, in_.nv, w_.size() > 1);
      bisect_all(ngroups, cuts);
    } else {
      tasks((int64_t)nmesh, [&](int64_t k) {
        points((*in_.voff)[k], (*in_.voff)[k + 1], false);
        bisect((*in_.voff)[k], (*in_.voff)[k + 1], mesh_groups[k], mesh_groups[k + 1], cuts);
      });
    }
    // triangles of every group, counted in the order of the triangles; groups
    // with more than the limit are cut again
    where_.resize(in_.nv);
    w_.each(ngroups, [&](int64_t g) {
      for (int64_t i = cuts[g]; i < cuts[g + 1]; ++i) where_[pts_[i].id].patch = (int32_t)g;
    });
    count_triangles(ngroups);
    std::vector<std::vector<int64_t>> pieces(ngroups);
    std::atomic<bool> split{false};
    tasks(ngroups, [&](int64_t g) {
      if (total(g) <= in_.max_tri || cuts[g + 1] - cuts[g] == 1) {
        pieces[g] = {cuts[g]};
      } else {
        pieces[g] = split_to_fit(cuts[g], cuts[g + 1]);
        if (pieces[g].size() > 1) split = true;
      }
    });
    P_.mbeg.push_back(0);
    for (size_t k = 0; k < nmesh; ++k) {
      for (int32_t g = mesh_groups[k]; g < mesh_groups[k + 1]; ++g)
        for (int64_t b : pieces[g]) {
          P_.vbeg.push_back((int32_t)b);
          P_.pmesh.push_back((int32_t)k);
        }
      P_.mbeg.push_back((int32_t)P_.vbeg.size());
    }
    P_.npatch = (int32_t)P_.vbeg.size();
    P_.vbeg.push_back((int32_t)in_.nv);
    // every patch by descending degree, then the caller's id
    P_.deg.resize(in_.nv);
    w_.run([&](int q) {
      std::vector<uint64_t> key;
      for (int64_t k = share(P_.npatch, q); k < share(P_.npatch, q + 1); ++k) {
        const int32_t v0 = P_.vbeg[k], v1 = P_.vbeg[k + 1];
        key.clear();
        for (int32_t i = v0; i < v1; ++i) {
          const int32_t v = pts_[i].id;
          key.push_back((uint64_t)(uint32_t)(INT32_MAX - (in_.row[v + 1] - in_.row[v])) << 32 | (uint32_t)v);
        }
        std::sort(key.begin(), key.end());
        for (int32_t i = v0; i < v1; ++i) {
          const int32_t v = (int32_t)(uint32_t)key[i - v0];
          P_.order[i] = v;
          P_.deg[i] = (uint16_t)(INT32_MAX - (int32_t)(key[i - v0] >> 32));
          where_[v] = Where{i, (int32_t)k};
        }
      }
    });
    UVec<Point>().swap(pts_);
    UVec<Point>().swap(swap_);
    if (split) count_triangles(P_.npatch);
    return fill();
  }

 private:
  const PatchInput& in_;
  PatchPlan& P_;
  Workers own_;
  Workers& w_;
  // A vertex, its coordinates in units of the longer side of its mesh's box
  // (single precision is enough to cut by).
  struct Point {
    float x, y;
    int32_t id;
  };
  UVec<Point> pts_, swap_;  // vertices, partitioned as the order is found; room for the cuts
  struct Where {
    int32_t at, patch;  // internal id; patch (its group, before the patches are final)
  };
  UVec<Where> where_;                         // of each of the caller's vertices
  std::vector<std::vector<int32_t>> counts_;  // [worker][patch] triangles of the worker's share that belong to it

  int64_t share(int64_t n, int q) const { return n * q / w_.size(); }

  // f(i) for i = 0 .. n - 1, each by the next free worker
  template <class F>
  void tasks(int64_t n, const F& f) {
    std::atomic<int64_t> next{0};
    w_.run([&](int) {
      for (int64_t i; (i = next.fetch_add(1)) < n;) f(i);
    });
  }

  // Points of the vertices [b, e) of one mesh.
  void points(int64_t b, int64_t e, bool parallel) {
    struct Box {
      double x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    };
    const int n = parallel ? w_.size() : 1;
    std::vector<Box> box(n);
    auto part = [&](int q) { return b + (e - b) * q / n; };
    auto bounds = [&](int q) {
      Box B;
      for (int64_t i = part(q); i < part(q + 1); ++i) {
        B.x0 = std::min(B.x0, in_.x[i]);
        B.x1 = std::max(B.x1, in_.x[i]);
        B.y0 = std::min(B.y0, in_.y[i]);
        B.y1 = std::max(B.y1, in_.y[i]);
      }
      box[q] = B;
    };
    if (parallel) w_.run(bounds);
    else bounds(0);
    Box B;
    for (const Box& o : box) {
      B.x0 = std::min(B.x0, o.x0);
      B.x1 = std::max(B.x1, o.x1);
      B.y0 = std::min(B.y0, o.y0);
      B.y1 = std::max(B.y1, o.y1);
    }
    const double len = std::max(B.x1 - B.x0, B.y1 - B.y0);
    const double f = len > 1e-300 && len < INFINITY ? 1.0 / len : 0.0;
    auto put = [&](int q) {
      for (int64_t i = part(q); i < part(q + 1); ++i)
        pts_[i] = Point{(float)((in_.x[i] - B.x0) * f), (float)((in_.y[i] - B.y0) * f), (int32_t)i};
    };
    if (parallel) w_.run(put);
    else put(0);
  }

  // Position in [b, e) of the cut that leaves about `want` vertices before
  // it, pts[b, e) partitioned around it along the longer side (into the bins of
  // a histogram below, at and above the cut first); by all workers, or
  // (parallel: false) the caller.
  int64_t cut(int64_t b, int64_t e, int64_t want, int64_t lo, int64_t hi, bool parallel = false) {
    struct Box {
      float x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    };
    const int w = parallel ? w_.size() : 1;
    std::vector<Box> box(w);
    auto part = [&](int q) { return b + (e - b) * q / w; };
    auto all = [&](const auto& f) {
      if (parallel) w_.run(f);
      else f(0);
    };
    all([&](int q) {
      Box B;
      for (int64_t i = part(q); i < part(q + 1); ++i) {
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
    if (e - b > 256) {
      const int bins = (int)std::min<int64_t>(4096, (e - b) / 16);
      const float c0 = ax ? B.x0 : B.y0, len = (ax ? B.x1 : B.y1) - c0;
      const float f = len > 0.0f ? bins / len : 0.0f;
      auto bin = [&](const Point& p) { return std::min(bins - 1, (int)((co(p) - c0) * f)); };
      std::vector<int32_t> count((size_t)w * bins, 0);
      all([&](int q) {
        int32_t* c = &count[(size_t)q * bins];
        for (int64_t i = part(q); i < part(q + 1); ++i) ++c[bin(pts_[i])];
      });
      int64_t before = b;
      int at = 0;
      for (;; ++at) {
        int64_t n = 0;
        for (int q = 0; q < w; ++q) n += count[(size_t)q * bins + at];
        if (before + n > m) {
          u = before;
          v = before + n;
          break;
        }
        before += n;
      }
      // three runs: bins below, the bin of the cut, bins above
      std::vector<std::array<int64_t, 3>> to(w);
      int64_t next[3] = {b, u, v};
      for (int q = 0; q < w; ++q) {
        const int32_t* c = &count[(size_t)q * bins];
        int64_t n[3] = {0, c[at], part(q + 1) - part(q) - c[at]};
        for (int k = 0; k < at; ++k) n[0] += c[k];
        n[2] -= n[0];
        for (int k = 0; k < 3; ++k) {
          to[q][k] = next[k];
          next[k] += n[k];
        }
      }
      all([&](int q) {
        std::array<int64_t, 3> x = to[q];
        for (int64_t i = part(q); i < part(q + 1); ++i) {
          const int k = bin(pts_[i]);
          swap_[x[(k >= at) + (k > at)]++] = pts_[i];
        }
      });
      all([&](int q) { std::copy(swap_.begin() + part(q), swap_.begin() + part(q + 1), pts_.begin() + part(q)); });
    }
    auto o = pts_.begin();
    std::nth_element(o + u, o + m, o + v, less);
    // the run of vertices with the coordinate of the cut: move the cut to its nearer end
    const float at = co(pts_[m]);
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

  struct Range {
    int64_t b, e, g0, g1;  // vertices, groups they are to become
  };
  // The cut of a range in two, returned as the first vertex and group of its second part.
  Range halves(const Range& r, bool parallel) {
    const int64_t n = r.g1 - r.g0, na = n / 2, nb = n - na;
    // a snapped cut may move by at most an eighth of the smaller side's vertices
    const int64_t len = r.e - r.b, want = len * na / n;
    const int64_t slack = std::min(want, len - want) / 8;
    const int64_t lo = std::max(na, want - slack), hi = std::min(len - nb, want + slack);
    const int64_t k = cut(r.b, r.e, std::min(std::max(want, na), len - nb), lo, hi, parallel);
    return Range{k, r.e, r.g0 + na, r.g1};
  }

  // Cuts pts[b, e) into groups g0 .. g1 - 1; cuts[g] receives their starts.
  void bisect(int64_t b, int64_t e, int64_t g0, int64_t g1, std::vector<int64_t>& cuts) {
    if (g1 - g0 == 1) {
      cuts[g0] = b;
      return;
    }
    const Range s = halves(Range{b, e, g0, g1}, false);
    bisect(b, s.b, g0, s.g0, cuts);
    bisect(s.b, e, s.g0, g1, cuts);
  }

  // The same for one mesh: the largest ranges cut by all workers together, then
  // each range by whichever worker is free.
  void bisect_all(int64_t ngroups, std::vector<int64_t>& cuts) {
    std::vector<Range> todo{{0, in_.nv, 0, ngroups}};
    auto take = [&](Range& r, bool parallel) {  // r keeps its first part
      const Range s = halves(r, parallel);
      r.e = s.b;
      r.g1 = s.g0;
      return s;
    };
    for (size_t k = 0; w_.size() > 1 && k < todo.size();) {
      if (todo[k].e - todo[k].b < 50000 || todo[k].g1 - todo[k].g0 == 1) ++k;
      else todo.push_back(take(todo[k], true));
    }
    std::mutex m;
    int busy = 0;  // workers that may still add ranges
    bool failed = false;
    auto work = [&] {
      for (bool mine = false;;) {
        Range r{0, 0, 0, 0};
        {
          std::lock_guard<std::mutex> g(m);
          busy -= mine;
          mine = !todo.empty();
          if (mine) {
            r = todo.back();
            todo.pop_back();
            ++busy;
          }
          if (failed || (!mine && busy == 0)) return;
        }
        if (!mine) {
          std::this_thread::yield();
          continue;
        }
        while (w_.size() > 1 && r.e - r.b > 4000 && r.g1 - r.g0 > 1) {
          const Range s = take(r, false);
          std::lock_guard<std::mutex> g(m);
          todo.push_back(s);
        }
        bisect(r.b, r.e, r.g0, r.g1, cuts);
      }
    };
    w_.run([&](int) {
      try {
        work();
      } catch (...) {  // out of memory: nobody waits for this worker's ranges
        std::lock_guard<std::mutex> g(m);
        failed = true;
        throw;
      }
    });
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

  // Calls f(k) for every patch k that triangle t belongs to.
  template <class F>
  void patches_of(const Where a[3], const F& f) const {
    f(a[0].patch);
    if (a[1].patch != a[0].patch) f(a[1].patch);
    if (a[2].patch != a[0].patch && a[2].patch != a[1].patch) f(a[2].patch);
  }
  void corners_of(int64_t t, Where a[3]) const {
    for (int c = 0; c < 3; ++c) a[c] = where_[in_.tri[3 * t + c]];
  }

  void count_triangles(int64_t n) {
    counts_.resize(w_.size());
    w_.run([&](int q) {
      std::vector<int32_t>& c = counts_[q];
      c.assign(n, 0);
      Where a[3];
      for (int64_t t = share(in_.nt, q); t < share(in_.nt, q + 1); ++t) {
        corners_of(t, a);
        patches_of(a, [&](int32_t k) { ++c[k]; });
      }
    });
  }
  int64_t total(int64_t k) const {
    int64_t n = 0;
    for (const auto& c : counts_) n += c[k];
    return n;
  }

  // Triangles, halo and part slots of every patch.
  std::string fill() {
    const int32_t np = P_.npatch;
    P_.inv.resize(in_.nv);
    w_.each(in_.nv, [&](int64_t v) { P_.inv[v] = where_[v].at; });
    // each worker's triangles go to every patch behind those of the workers
    // before it, so a patch's are ascending
    P_.tbeg.assign(np + 1, 0);
    int64_t nt = 0;
    for (int32_t k = 0; k < np; ++k) {
      P_.tbeg[k] = (int32_t)nt;
      for (auto& c : counts_) {
        const int32_t n = c[k];
        c[k] = (int32_t)nt;  // now where its first one goes
        nt += n;
      }
      if (nt >= (int64_t(1) << 31)) return "too many patch triangles";
      P_.max_tri = std::max(P_.max_tri, (int32_t)(nt - P_.tbeg[k]));
    }
    P_.tbeg[np] = (int32_t)nt;
    P_.tri.resize(3 * nt);
    P_.tid.resize(nt);
    w_.run([&](int q) {
      std::vector<int32_t>& next = counts_[q];
      Where a[3];
      for (int64_t t = share(in_.nt, q); t < share(in_.nt, q + 1); ++t) {
        corners_of(t, a);
        const int32_t owner = std::min(a[0].patch, std::min(a[1].patch, a[2].patch));
        patches_of(a, [&](int32_t k) {
          const int64_t at = next[k]++;
          P_.tid[at] = (int32_t)(owner == k ? t : -1 - t);
          for (int c = 0; c < 3; ++c) P_.tri[c * nt + at] = (uint32_t)a[c].at;  // internal id for now
        });
      }
    });
    UVec<Where>().swap(where_);
    counts_.clear();
    // patch by patch: halo, part slots, local ids
    P_.hbeg.assign(np + 1, 0);
    P_.jbeg.assign(np + 1, 0);
    P_.seam.assign(np, 0);
    struct Part {
      std::vector<int32_t> halo, jb;
      int32_t max_lv = 0, max_slots = 0;
      bool large = false;
    };
    std::vector<Part> part(w_.size());
    const bool periodic = in_.hpx < INFINITY || in_.hpy < INFINITY;
    w_.run([&](int q) {
      Part& o = part[q];
      UVec<int32_t> loc(in_.nv);  // of a vertex met in this patch its place in H; checked there, so never cleared
      std::vector<int32_t> H;
      std::vector<uint16_t> next;
      std::vector<double> x, y;
      for (int64_t k = share(np, q); k < share(np, q + 1); ++k) {
        const int32_t v0 = P_.vbeg[k], v1 = P_.vbeg[k + 1], own = v1 - v0;
        const int64_t t0 = P_.tbeg[k], t1 = P_.tbeg[k + 1];
        H.clear();
        for (int c = 0; c < 3; ++c)
          for (int64_t at = t0; at < t1; ++at) {
            const int32_t w = (int32_t)P_.tri[c * nt + at];
            if (w >= v0 && w < v1) continue;
            const uint32_t l = (uint32_t)loc[w];
            if (l < H.size() && H[l] == w) continue;
            loc[w] = (int32_t)H.size();
            H.push_back(w);
          }
        std::sort(H.begin(), H.end());
        for (size_t i = 0; i < H.size(); ++i) loc[H[i]] = (int32_t)i;
        // part slots: the first owned vertex has the largest degree
        const size_t j0 = o.jb.size();
        int32_t slots = 0;
        for (int32_t j = 0, n = own; j < P_.deg[v0]; ++j) {
          while (n > 0 && P_.deg[v0 + n - 1] <= j) --n;
          o.jb.push_back(slots);
          slots += n;
        }
        P_.jbeg[k + 1] = (int32_t)(o.jb.size() - j0);
        P_.hbeg[k + 1] = (int32_t)H.size();
        o.halo.insert(o.halo.end(), H.begin(), H.end());
        const int64_t lv = own + (int64_t)H.size();
        if (lv >= 65535 || slots >= 65535) {
          o.large = true;
          return;
        }
        o.max_lv = std::max(o.max_lv, (int32_t)lv);
        o.max_slots = std::max(o.max_slots, slots);
        if (periodic) {
          x.resize(lv);
          y.resize(lv);
          for (int64_t l = 0; l < lv; ++l) {
            const int32_t v = P_.order[l < own ? v0 + l : H[l - own]];
            x[l] = in_.x[v];
            y[l] = in_.y[v];
          }
        }
        next.assign(own, 0);  // triangles are ascending: ranks in order of appearance
        for (int64_t at = t0; at < t1; ++at) {
          int32_t l[3];
          for (int c = 0; c < 3; ++c) {
            uint32_t& p = P_.tri[c * nt + at];
            const int32_t w = (int32_t)p;
            uint32_t dst = 0xffff;
            if (w >= v0 && w < v1) {
              l[c] = w - v0;
              dst = (uint32_t)(o.jb[j0 + next[l[c]]++] + l[c]);
            } else {
              l[c] = own + loc[w];
            }
            p = (uint32_t)l[c] | dst << 16;
          }
          if (periodic)
            for (int i = 1; i < 3; ++i)
              if (std::fabs(x[l[i]] - x[l[0]]) > in_.hpx || std::fabs(y[l[i]] - y[l[0]]) > in_.hpy) P_.seam[k] = 1;
        }
      }
    });
    int64_t nh = 0, nj = 0;
    for (const Part& o : part) {
      if (o.large) return "a patch has too many vertices";
      nh += (int64_t)o.halo.size();
      nj += (int64_t)o.jb.size();
      P_.max_lv = std::max(P_.max_lv, o.max_lv);
      P_.max_slots = std::max(P_.max_slots, o.max_slots);
    }
    if (nh >= (int64_t(1) << 31) || nj >= (int64_t(1) << 31)) return "too many patch triangles";
    P_.halo.reserve(nh);
    P_.jb.reserve(nj);
    for (const Part& o : part) {
      P_.halo.insert(P_.halo.end(), o.halo.begin(), o.halo.end());
      P_.jb.insert(P_.jb.end(), o.jb.begin(), o.jb.end());
    }
    for (int32_t k = 0; k < np; ++k) {
      P_.hbeg[k + 1] += P_.hbeg[k];
      P_.jbeg[k + 1] += P_.jbeg[k];
    }
    return std::string();
  }
};

inline std::string build_patch_plan(const PatchInput& in, PatchPlan& P) { return PatchBuilder(in, P).build(); }

}  // namespace rd
