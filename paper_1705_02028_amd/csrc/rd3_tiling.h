// Tiles of a tetrahedral mesh (host): tetrahedra cut by recursive coordinate
// bisection into compact tiles of equal size, vertices renumbered tile by tile
// as first met, and for every tile the tables of its workgroup (rd3_device.h).
// Whatever the caller's numbering, a tile's vertices are then few and mostly
// neighbours in memory.
#pragma once

#include <algorithm>
#include <array>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <string>
#include <utility>
#include <vector>

#include "rd3_device.h"
#include "rd_patching.h"

namespace rd3 {

struct TilePlan3 {
  std::vector<Tile3> tile;
  rd::UVec<uint32_t> tet;        // [nt][4] local vertex | slot << 16
  std::vector<int32_t> lv, rpos; // of each local vertex: vertex, record
  std::vector<uint16_t> deg;
  std::vector<int32_t> jb, rbeg, inv;  // inv: vertex of each of the caller's
  int32_t max_lv = 0, max_tet = 0, max_jd = 0;
};

// All tiles of 12^3, 24^3 and 64^3 cells: 1.1, 5.5 and 70 ms (four workers, then
// eight) against 3.0, 9.5 and 153 with nth_element of whole ranges and a sort of
// every tile's corners by vertex.
class TileBuilder3 {
 public:
  TileBuilder3(int64_t nv, int64_t nt, const int32_t* tet, const double* const xyz[3], const double per[3], int target,
               rd::Workers& pool, TilePlan3& P)
      : nv_(nv), nt_(nt), tet_(tet), target_(target), w_(pool), P_(P), it_(nt), swap_(nt) {
    for (int k = 0; k < 3; ++k) {
      xyz_[k] = xyz[k];
      per_[k] = per[k];
    }
  }

  std::string build(bool renumber) {
    w_.each(nt_, [&](int64_t t) { it_[t] = item(t); });
    // halved until there are ranges for every worker, in order: the largest by
    // all workers together, the others each by one
    std::vector<Range> top{{0, nt_}};
    while (w_.size() > 1 && (int)top.size() < 4 * w_.size()) {
      std::vector<Range> next(2 * top.size());
      bool any = false;
      auto halve = [&](size_t i, bool parallel) {
        const Range r = top[i];
        const int64_t m = r.second - r.first <= target_ ? r.second : cut(r.first, r.second, parallel);
        next[2 * i] = {r.first, m};
        next[2 * i + 1] = {m, r.second};
      };
      auto large = [&](size_t i) { return top[i].second - top[i].first > 50000; };
      for (size_t i = 0; i < top.size(); ++i) {
        any = any || top[i].second - top[i].first > target_;
        if (large(i)) halve(i, true);
      }
      if (!any) break;
      w_.each((int64_t)top.size(), [&](int64_t i) {
        if (!large(i)) halve(i, false);
      });
      top.swap(next);
    }
    std::vector<Part> part(top.size());
    P_.tet.resize(4 * nt_);
    std::atomic<size_t> next{0};
    w_.run([&](int) {
      Scratch s;
      for (size_t i; (i = next.fetch_add(1)) < top.size();) tiles(top[i], part[i], s);
    });
    for (const Part& p : part) {
      for (Tile3 t : p.tile) {
        t.l0 += (int32_t)P_.lv.size();
        t.j0 += (int32_t)P_.jb.size();
        P_.max_lv = std::max(P_.max_lv, t.nlv);
        P_.max_tet = std::max(P_.max_tet, t.nt);
        P_.max_jd = std::max(P_.max_jd, t.nj);
        P_.tile.push_back(t);
      }
      P_.lv.insert(P_.lv.end(), p.lv.begin(), p.lv.end());
      P_.jb.insert(P_.jb.end(), p.jb.begin(), p.jb.end());
      P_.deg.insert(P_.deg.end(), p.deg.begin(), p.deg.end());
      if (6 * (int64_t)P_.lv.size() >= INT32_MAX || (int64_t)P_.jb.size() >= INT32_MAX)
        return "mesh too large for 32-bit record indices";
    }
    // vertex numbers, records of a vertex by ascending tile
    P_.inv.assign(nv_, -1);
    P_.rbeg.assign(nv_ + 1, 0);
    int32_t n = 0;
    for (int32_t& v : P_.lv) {
      if (P_.inv[v] < 0) P_.inv[v] = renumber ? n++ : v;
      v = P_.inv[v];
      ++P_.rbeg[v + 1];
    }
    for (int64_t v = 0; v < nv_; ++v) P_.rbeg[v + 1] += P_.rbeg[v];
    std::vector<int32_t> fill(P_.rbeg.begin(), P_.rbeg.end() - 1);
    P_.rpos.resize(P_.lv.size());
    for (size_t l = 0; l < P_.lv.size(); ++l) P_.rpos[l] = fill[P_.lv[l]]++;
    return {};
  }

 private:
  struct Item {
    float c[3];  // centroid
    int32_t id;
  };
  using Range = std::pair<int64_t, int64_t>;
  // Tiles of one range and their tables, with the caller's vertices.
  struct Part {
    std::vector<Tile3> tile;
    std::vector<int32_t> lv, jb;
    std::vector<uint16_t> deg;
  };
  // The vertices of the tile in hand: a hash table from vertex to local vertex
  // (as first met), each one's tetrahedra, and of every corner its local vertex
  // and its rank among that vertex's corners.
  struct Scratch {
    int32_t slot[16 * kTileTets];
    int32_t vert[4 * kTileTets], deg[4 * kTileTets], pos[4 * kTileTets];
    uint16_t loc[4 * kTileTets], rank[4 * kTileTets];
    int32_t id[kTileTets];
    uint64_t key[4 * kTileTets];
  };

  const int64_t nv_, nt_;
  const int32_t* tet_;
  const double* xyz_[3];
  double per_[3];
  const int target_;
  rd::Workers& w_;
  TilePlan3& P_;
  rd::UVec<Item> it_, swap_;  // tetrahedra, partitioned as the tiles are found; room for the cuts

  Item item(int64_t t) const {
    Item r;
    for (int k = 0; k < 3; ++k) {
      const double x0 = xyz_[k][tet_[4 * t]];
      double s = 0.0;
      for (int i = 1; i < 4; ++i) {
        double dx = xyz_[k][tet_[4 * t + i]] - x0;
        if (per_[k] > 0.0) dx = dx > 0.5 * per_[k] ? dx - per_[k] : (dx < -0.5 * per_[k] ? dx + per_[k] : dx);
        s += dx;
      }
      r.c[k] = (float)(x0 + 0.25 * s);
      if (r.c[k] != r.c[k]) r.c[k] = 0.0f;
    }
    r.id = (int32_t)t;
    return r;
  }

  // Halves a range of tetrahedra across its longest side, at a multiple of the
  // tile size: by (centroid, id), so that the halves are the same however it is
  // done. A histogram finds the run of centroids with the cut in it; three runs
  // are then laid out by one pass without a branch on the data, and only the
  // middle one is sorted out item by item.
  int64_t cut(int64_t b, int64_t e, bool parallel) {
    const int w = parallel ? w_.size() : 1;
    auto all = [&](auto&& f) {
      if (parallel) w_.run(f);
      else f(0);
    };
    auto part = [&](int q) { return b + (e - b) * q / w; };
    struct Box {
      float lo[3], hi[3];
    };
    std::vector<Box> box(w);
    all([&](int q) {
      Box B;
      for (int k = 0; k < 3; ++k) B.lo[k] = B.hi[k] = it_[b].c[k];
      for (int64_t i = part(q); i < part(q + 1); ++i)
        for (int k = 0; k < 3; ++k) {
          B.lo[k] = std::min(B.lo[k], it_[i].c[k]);
          B.hi[k] = std::max(B.hi[k], it_[i].c[k]);
        }
      box[q] = B;
    });
    Box B = box[0];
    for (const Box& o : box)
      for (int k = 0; k < 3; ++k) {
        B.lo[k] = std::min(B.lo[k], o.lo[k]);
        B.hi[k] = std::max(B.hi[k], o.hi[k]);
      }
    int a = 0;
    for (int k = 1; k < 3; ++k)
      if (B.hi[k] - B.lo[k] > B.hi[a] - B.lo[a]) a = k;
    const int64_t n = (e - b + target_ - 1) / target_;
    const int64_t m = n > 1 ? b + (e - b) * (n / 2) / n : b + (e - b) / 2;
    auto less = [a](const Item& p, const Item& q) { return p.c[a] != q.c[a] ? p.c[a] < q.c[a] : p.id < q.id; };
    constexpr int bins = 64;
    const float lo = B.lo[a], scale = bins / (B.hi[a] - lo);
    int64_t u = b, v = e;
    if (e - b > 4 * bins && scale > 0.0f && std::isfinite(scale)) {
      auto bin = [&](const Item& p) { return std::min(bins - 1, (int)((p.c[a] - lo) * scale)); };
      std::vector<std::array<int32_t, bins>> count(w);
      all([&](int q) {
        std::array<int32_t, bins>& c = count[q];
        c.fill(0);
        for (int64_t i = part(q); i < part(q + 1); ++i) ++c[bin(it_[i])];
      });
      int at = 0;
      for (int64_t before = b;; ++at) {
        int64_t k = 0;
        for (int q = 0; q < w; ++q) k += count[q][at];
        if (before + k > m) {
          u = before;
          v = before + k;
          break;
        }
        before += k;
      }
      std::vector<std::array<int64_t, 3>> to(w);
      int64_t next[3] = {b, u, v};
      for (int q = 0; q < w; ++q) {
        int64_t k[3] = {0, count[q][at], part(q + 1) - part(q) - count[q][at]};
        for (int i = 0; i < at; ++i) k[0] += count[q][i];
        k[2] -= k[0];
        for (int i = 0; i < 3; ++i) {
          to[q][i] = next[i];
          next[i] += k[i];
        }
      }
      all([&](int q) {
        std::array<int64_t, 3> x = to[q];
        for (int64_t i = part(q); i < part(q + 1); ++i) {
          const int k = bin(it_[i]);
          swap_[x[(k >= at) + (k > at)]++] = it_[i];
        }
      });
      all([&](int q) { std::copy(swap_.begin() + part(q), swap_.begin() + part(q + 1), it_.begin() + part(q)); });
    }
    std::nth_element(it_.begin() + u, it_.begin() + m, it_.begin() + v, less);
    return m;
  }

  void tiles(const Range& range, Part& p, Scratch& s) {
    std::vector<Range> todo{range};
    while (!todo.empty()) {
      const Range r = todo.back();
      todo.pop_back();
      if (r.second == r.first || (r.second - r.first <= target_ && tile(r, p, s))) continue;
      const int64_t m = cut(r.first, r.second, false);
      todo.push_back({m, r.second});
      todo.push_back({r.first, m});
    }
  }

  // The range as one tile; false if it has too many vertices.
  bool tile(const Range& r, Part& p, Scratch& s) {
    const int n = (int)(r.second - r.first);
    for (int q = 0; q < n; ++q) s.id[q] = it_[r.first + q].id;
    std::sort(s.id, s.id + n);
    int bits = 4;
    while ((1 << bits) < 8 * n) ++bits;  // a table at most half full
    std::fill(s.slot, s.slot + (1 << bits), -1);
    int nlv = 0;
    for (int q = 0; q < n; ++q)
      for (int c = 0; c < 4; ++c) {
        const int32_t v = tet_[4 * (int64_t)s.id[q] + c];
        uint32_t h = ((uint32_t)v * 2654435769u) >> (32 - bits);
        while (s.slot[h] >= 0 && s.vert[s.slot[h]] != v) h = (h + 1) & ((1u << bits) - 1);
        int32_t& l = s.slot[h];
        if (l < 0) {
          l = nlv++;
          s.vert[l] = v;
          s.deg[l] = 0;
        }
        s.loc[4 * q + c] = (uint16_t)l;
        s.rank[4 * q + c] = (uint16_t)s.deg[l]++;
      }
    if (nlv > kTileVerts) return false;
    // local vertices by falling degree, then the caller's id; diagonal j holds
    // the j-th part of each that has one
    for (int l = 0; l < nlv; ++l)
      s.key[l] = (uint64_t)(4 * kTileTets - s.deg[l]) << 40 | (uint64_t)(uint32_t)s.vert[l] << 8 | (uint64_t)l;
    std::sort(s.key, s.key + nlv);
    Tile3 t;
    t.t0 = (int32_t)r.first;
    t.nt = n;
    t.l0 = (int32_t)p.lv.size();
    t.nlv = nlv;
    t.j0 = (int32_t)p.jb.size();
    t.nj = s.deg[s.key[0] & 255];
    for (int o = 0; o < nlv; ++o) {
      const int l = (int)(s.key[o] & 255);
      s.pos[l] = o;
      p.lv.push_back(s.vert[l]);
      p.deg.push_back((uint16_t)s.deg[l]);
    }
    int at = 0, have = nlv;
    for (int j = 0; j < t.nj; ++j) {
      while (p.deg[t.l0 + have - 1] <= j) --have;
      p.jb.push_back(at);
      at += have;
    }
    for (int i = 0; i < 4 * n; ++i) {
      const int l = s.pos[s.loc[i]];
      P_.tet[4 * r.first + i] = (uint32_t)l | (uint32_t)(p.jb[t.j0 + s.rank[i]] + l) << 16;
    }
    p.tile.push_back(t);
    return true;
  }
};

// tet: [4 nt] corners; xyz: coordinates; target: tetrahedra per tile, at most
// kTileTets; renumber: vertices as first met, else the caller's. Returns an
// error message, empty when built.
inline std::string build_tiles3(int64_t nv, int64_t nt, const int32_t* tet, const double* const xyz[3],
                                const double per[3], int target, bool renumber, rd::Workers& pool, TilePlan3& P) {
  return TileBuilder3(nv, nt, tet, xyz, per, target, pool, P).build(renumber);
}

}  // namespace rd3
