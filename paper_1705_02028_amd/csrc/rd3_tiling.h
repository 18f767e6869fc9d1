// Tiles of a tetrahedral mesh (host): tetrahedra cut by recursive coordinate
// bisection into compact tiles of equal size, vertices renumbered tile by tile
// as first met, and for every tile the tables of its workgroup (rd3_device.h).
// Whatever the caller's numbering, a tile's vertices are then few and mostly
// neighbours in memory.
#pragma once

#include <algorithm>
#include <cstdint>
#include <string>
#include <utility>
#include <vector>

#include "rd3_device.h"
#include "rd_patching.h"

namespace rd3 {

struct TilePlan3 {
  std::vector<Tile3> tile;
  std::vector<uint32_t> tet;     // [nt][4] local vertex | slot << 16
  std::vector<int32_t> torder;   // [nt] the caller's tetrahedron of each
  std::vector<int32_t> lv, rpos; // of each local vertex: vertex, record
  std::vector<uint16_t> deg;
  std::vector<int32_t> jb, rbeg, inv;  // inv: vertex of each of the caller's
  int32_t max_lv = 0, max_tet = 0, max_jd = 0;
};

// tet: [4 nt] corners; xyz: coordinates; target: tetrahedra per tile, at most
// kTileTets; renumber: vertices as first met, else the caller's. Returns an
// error message, empty when built.
inline std::string build_tiles3(int64_t nv, int64_t nt, const int32_t* tet, const double* const xyz[3],
                                const double per[3], int target, bool renumber, int threads, TilePlan3& P) {
  struct Item {
    float c[3];
    int32_t id;
  };
  std::vector<Item> it(nt);
  rd::run_workers(threads, [&](int w) {
    for (int64_t t = nt * w / threads; t < nt * (w + 1) / threads; ++t) {
      for (int k = 0; k < 3; ++k) {
        const double x0 = xyz[k][tet[4 * t]];
        double s = 0.0;
        for (int i = 1; i < 4; ++i) {
          double dx = xyz[k][tet[4 * t + i]] - x0;
          if (per[k] > 0.0) dx = dx > 0.5 * per[k] ? dx - per[k] : (dx < -0.5 * per[k] ? dx + per[k] : dx);
          s += dx;
        }
        it[t].c[k] = (float)(x0 + 0.25 * s);
      }
      it[t].id = (int32_t)t;
    }
  });
  // halves a range of tetrahedra across its longest side, at a multiple of the tile size
  auto cut = [&](int64_t b, int64_t e) -> int64_t {
    float lo[3], hi[3];
    for (int k = 0; k < 3; ++k) lo[k] = hi[k] = it[b].c[k];
    for (int64_t i = b; i < e; ++i)
      for (int k = 0; k < 3; ++k) {
        lo[k] = std::min(lo[k], it[i].c[k]);
        hi[k] = std::max(hi[k], it[i].c[k]);
      }
    int a = 0;
    for (int k = 1; k < 3; ++k)
      if (hi[k] - lo[k] > hi[a] - lo[a]) a = k;
    const int64_t n = (e - b + target - 1) / target;
    const int64_t m = n > 1 ? b + (e - b) * (n / 2) / n : b + (e - b) / 2;
    std::nth_element(it.begin() + b, it.begin() + m, it.begin() + e, [a](const Item& p, const Item& q) {
      return p.c[a] != q.c[a] ? p.c[a] < q.c[a] : p.id < q.id;
    });
    return m;
  };
  using Range = std::pair<int64_t, int64_t>;
  std::vector<Range> top{{0, nt}};
  while ((int)top.size() < 8 * threads) {
    std::vector<Range> next(2 * top.size());
    bool any = false;
    rd::run_workers(threads, [&](int w) {
      for (size_t i = w; i < top.size(); i += threads) {
        const Range r = top[i];
        if (r.second - r.first <= target) {
          next[2 * i] = r;
          next[2 * i + 1] = {r.second, r.second};
        } else {
          const int64_t m = cut(r.first, r.second);
          next[2 * i] = {r.first, m};
          next[2 * i + 1] = {m, r.second};
        }
      }
    });
    for (const Range& r : next) any = any || r.second - r.first > target;
    top.swap(next);
    if (!any) break;
  }
  // each range to its tiles, and the tiles' tables, with the caller's vertices
  struct Part {
    std::vector<Tile3> tile;
    std::vector<int32_t> lv, jb;
    std::vector<uint16_t> deg;
  };
  std::vector<Part> part(top.size());
  P.tet.resize(4 * nt);
  rd::run_workers(threads, [&](int w) {
    std::vector<std::pair<int32_t, int32_t>> use;  // (vertex, 4 tet + corner)
    std::vector<int32_t> first, order;
    for (size_t i = w; i < top.size(); i += threads) {
      Part& p = part[i];
      std::vector<Range> todo{top[i]};
      while (!todo.empty()) {
        const Range r = todo.back();
        todo.pop_back();
        const int64_t n = r.second - r.first;
        if (n == 0) continue;
        if (n <= target) {
          std::sort(it.begin() + r.first, it.begin() + r.second, [](const Item& a, const Item& b) { return a.id < b.id; });
          use.clear();
          for (int64_t q = r.first; q < r.second; ++q)
            for (int c = 0; c < 4; ++c)
              use.push_back({tet[4 * (int64_t)it[q].id + c], (int32_t)(4 * (q - r.first) + c)});
          std::sort(use.begin(), use.end());
          first.clear();
          for (size_t u = 0; u < use.size(); ++u)
            if (u == 0 || use[u].first != use[u - 1].first) first.push_back((int32_t)u);
          const int nlv = (int)first.size();
          first.push_back((int32_t)use.size());
          if (nlv <= kTileVerts) {
            // local vertices by falling degree; diagonal j holds the j-th part of each that has one
            order.resize(nlv);
            for (int l = 0; l < nlv; ++l) order[l] = l;
            std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
              return first[a + 1] - first[a] > first[b + 1] - first[b];
            });
            Tile3 t;
            t.t0 = (int32_t)r.first;
            t.nt = (int32_t)n;
            t.l0 = (int32_t)p.lv.size();
            t.nlv = nlv;
            t.j0 = (int32_t)p.jb.size();
            const int dmax = first[order[0] + 1] - first[order[0]];
            int at = 0, have = nlv;
            for (int j = 0; j < dmax; ++j) {
              while (first[order[have - 1] + 1] - first[order[have - 1]] <= j) --have;
              p.jb.push_back(at);
              at += have;
            }
            t.nj = dmax;
            for (int l = 0; l < nlv; ++l) {
              const int o = order[l];
              p.lv.push_back(use[first[o]].first);
              p.deg.push_back((uint16_t)(first[o + 1] - first[o]));
              for (int u = first[o]; u < first[o + 1]; ++u)
                P.tet[4 * r.first + use[u].second] = (uint32_t)l | (uint32_t)(p.jb[t.j0 + u - first[o]] + l) << 16;
            }
            p.tile.push_back(t);
            continue;
          }
        }
        const int64_t m = cut(r.first, r.second);
        todo.push_back({m, r.second});
        todo.push_back({r.first, m});
      }
    }
  });
  for (const Part& p : part) {
    for (Tile3 t : p.tile) {
      t.l0 += (int32_t)P.lv.size();
      t.j0 += (int32_t)P.jb.size();
      P.max_lv = std::max(P.max_lv, t.nlv);
      P.max_tet = std::max(P.max_tet, t.nt);
      P.max_jd = std::max(P.max_jd, t.nj);
      P.tile.push_back(t);
    }
    P.lv.insert(P.lv.end(), p.lv.begin(), p.lv.end());
    P.jb.insert(P.jb.end(), p.jb.begin(), p.jb.end());
    P.deg.insert(P.deg.end(), p.deg.begin(), p.deg.end());
    if (6 * (int64_t)P.lv.size() >= INT32_MAX || (int64_t)P.jb.size() >= INT32_MAX)
      return "mesh too large for 32-bit record indices";
  }
  P.torder.resize(nt);
  for (int64_t t = 0; t < nt; ++t) P.torder[t] = it[t].id;
  // vertex numbers, records of a vertex by ascending tile
  P.inv.assign(nv, -1);
  P.rbeg.assign(nv + 1, 0);
  int32_t next = 0;
  for (int32_t& v : P.lv) {
    if (P.inv[v] < 0) P.inv[v] = renumber ? next++ : v;
    v = P.inv[v];
    ++P.rbeg[v + 1];
  }
  for (int64_t v = 0; v < nv; ++v) P.rbeg[v + 1] += P.rbeg[v];
  std::vector<int32_t> fill(P.rbeg.begin(), P.rbeg.end() - 1);
  P.rpos.resize(P.lv.size());
  for (size_t l = 0; l < P.lv.size(); ++l) P.rpos[l] = fill[P.lv[l]]++;
  return {};
}

}  // namespace rd3
