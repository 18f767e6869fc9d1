// Host run of the patch form: builds the patches of a mesh (rd_patching.h) and
// runs the passes of rd_patch.hip patch by patch with the same bodies, every
// index checked against its range. Exposed to the CPU tests as a C interface.
#include <cmath>
#include <stdexcept>
#include <vector>

#include "rd_patch.h"
#include "rd_patching.h"

using rd::D4;

namespace {

struct Host {
  int64_t nv, nt;
  std::vector<double> x, y, V;
  std::vector<int32_t> tri, row, slot, inv, wb, wptr;
  std::vector<rd::WallEnt> went;
  std::vector<int64_t> voff, toff;
  rd::PatchPlan P;
  rd::Patches p;
};
Host h;

void require(bool ok, const char* what) {
  if (!ok) throw std::runtime_error(what);
}

// The passes over one patch as its workgroup runs them.
template <int SCHEME>
void stage(int st, bool lump, const std::vector<D4>& W, std::vector<D4>& D, std::vector<D4>& out, double dt,
           double& bound) {
  const rd::PatchPlan& P = h.P;
  const int64_t ptn = (int64_t)P.tid.size();
  for (int32_t k = 0; k < P.npatch; ++k) {
    const int32_t v0 = P.vbeg.at(k), own = P.vbeg.at(k + 1) - v0, h0 = P.hbeg.at(k);
    const int32_t nlv = own + P.hbeg.at(k + 1) - h0, t0 = P.tbeg.at(k), nt = P.tbeg.at(k + 1) - t0;
    require(own > 0 && nlv <= P.max_lv && nt <= P.max_tri, "patch sizes");
    std::vector<D4> Zn(nlv), Zs(nlv), Dl(nlv), part(P.max_slots);
    std::vector<double2> xy(nlv);
    std::vector<double> sig(nlv), lam(P.max_slots);
    std::vector<int> seen(P.max_slots, 0);
    for (int32_t l = 0; l < nlv; ++l) {
      const int32_t v = l < own ? v0 + l : P.halo.at(h0 + l - own);
      const int32_t c = P.order.at(v);
      xy[l] = make_double2(h.x.at(c), h.y.at(c));
      Zn[l] = rd::patch_z(h.p, W.at(v), &sig[l], nullptr);
      Dl[l] = D.at(v);
      Zs[l] = rd::patch_z(h.p, rd::patch_star(W.at(v), D.at(v), dt), nullptr, nullptr);
    }
    for (int32_t j = 0; j < nt; ++j) {
      uint16_t lv[3], dst[3];
      for (int c = 0; c < 3; ++c) {
        lv[c] = P.tri.at(c * ptn + t0 + j) & 0xffff;
        dst[c] = P.tri.at(c * ptn + t0 + j) >> 16;
        require(lv[c] < nlv, "local vertex");
        require((dst[c] == 0xffff) == (lv[c] >= own), "owned corners have a slot");
      }
      const rd::TriDiff g = rd::tri_diff(h.p, xy[lv[0]], xy[lv[1]], xy[lv[2]]);
      require(P.seam.at(k) || (g.d1x == xy[lv[1]].x - xy[lv[0]].x && g.d1y == xy[lv[1]].y - xy[lv[0]].y &&
                               g.d2x == xy[lv[2]].x - xy[lv[0]].x && g.d2y == xy[lv[2]].y - xy[lv[0]].y),
              "only patches on a seam unwrap");
      double o[3][4], pN[2][4], phi[4], lmax = 0.0;
      if (st == 1) {
        const D4 z[3] = {Zn[lv[0]], Zn[lv[1]], Zn[lv[2]]};
        lmax = rd::stage1_parts<SCHEME>(g, z, h.p.gas, nullptr, o, pN, phi);
      } else {
        auto zn = [&](int i) { return Zn[lv[i]]; };
        auto zs = [&](int i) { return Zs[lv[i]]; };
        auto dd = [&](int i) { return Dl[lv[i]]; };
        if (lump) rd::patch_tri2<SCHEME, true>(h.p, g, zn, zs, dd, nullptr, o);
        else rd::patch_tri2<SCHEME, false>(h.p, g, zn, zs, dd, nullptr, o);
      }
      const double term = lmax * std::fmax(std::fmax(sig[lv[0]], sig[lv[1]]), sig[lv[2]]);
      for (int c = 0; c < 3; ++c)
        if (dst[c] != 0xffff) {
          require(!seen.at(dst[c])++, "one part per slot");
          for (int q = 0; q < 4; ++q) part[dst[c]].v[q] = o[c][q];
          lam[dst[c]] = term;
        }
    }
    for (int32_t l = 0; l < own; ++l) {
      const int32_t v = v0 + l, c = P.order[v], n = P.deg.at(v);
      require(n == h.row[c + 1] - h.row[c] && n <= P.jbeg.at(k + 1) - P.jbeg[k], "every part of an owned vertex");
      const int32_t* jb = &P.jb.at(P.jbeg[k]);
      for (int32_t j = 0; j < n; ++j) require(seen.at(jb[j] + l) == 1, "slot filled");
      double acc[4], x = 0.0;
      rd::sum_parts(n, [&](int32_t j) { return part[jb[j] + l]; }, acc);
      for (int32_t j = 0; j < n; ++j) x += lam[jb[j] + l];
      const double V = h.V[c];
      const int32_t b = h.wb.empty() ? -1 : h.wb[v];
      double wn[4] = {0, 0, 0, 0}, ws[4] = {0, 0, 0, 0};
      if (b >= 0) {
        rd::wall_term(h.went.data(), h.wptr.at(b), h.wptr.at(b + 1), v, h.p.gamma, [&](int64_t i) { return W.at(i); },
                      wn);
        rd::wall_term(h.went.data(), h.wptr.at(b), h.wptr.at(b + 1), v, h.p.gamma,
                      [&](int64_t i) { return rd::patch_star(W.at(i), D.at(i), dt); }, ws);
      }
      if (st == 1) {
        bound = std::fmin(bound, 2.0 * std::fabs(V) / x);
        for (int q = 0; q < 4; ++q) out[v].v[q] = V > 0.0 ? (rd::kSymScale * acc[q] + wn[q]) / V : 0.0;
      } else {
        const D4 s = rd::patch_star(W[v], D[v], dt);
        for (int q = 0; q < 4; ++q)
          out[v].v[q] = V > 0.0 ? s.v[q] - dt / V * (acc[q] + 0.5 * (wn[q] + ws[q])) : W[v].v[q];
      }
    }
  }
}

void run(int scheme, int st, bool lump, const std::vector<D4>& W, std::vector<D4>& D, std::vector<D4>& out, double dt,
         double& bound) {
  switch (scheme) {
    case 0: stage<0>(st, lump, W, D, out, dt, bound); break;
    case 1: stage<1>(st, lump, W, D, out, dt, bound); break;
    case 2: stage<2>(st, lump, W, D, out, dt, bound); break;
    case 3: stage<3>(st, lump, W, D, out, dt, bound); break;
    default: stage<4>(st, lump, W, D, out, dt, bound); break;
  }
}

}  // namespace

extern "C" {

// Builds the patches; info: patches, largest triangle count, halo records,
// patch triangles, triangles listed as owned. Returns 0, or 1 when the builder
// refuses or a triangle is not owned exactly once.
int patch_build(int64_t nv, int64_t nt, const int32_t* tri, const double* x, const double* y, double px, double py,
                const uint8_t* ghost, int64_t nw, const int32_t* wall, int nmesh, const int64_t* voff,
                const int64_t* toff, int own, int max_tri, int threads, int64_t* info) try {
  h = Host();
  h.nv = nv;
  h.nt = nt;
  h.x.assign(x, x + nv);
  h.y.assign(y, y + nv);
  h.tri.assign(tri, tri + 3 * nt);
  h.row.assign(nv + 1, 0);
  h.slot.resize(3 * nt);
  for (int32_t v : h.tri) h.row[v + 1]++;
  for (int64_t i = 0; i < nv; ++i) h.row[i + 1] += h.row[i];
  std::vector<int32_t> fill(h.row.begin(), h.row.end() - 1);
  for (int64_t s = 0; s < 3 * nt; ++s) h.slot[fill[h.tri[s]]++] = (int32_t)s;
  h.voff.assign(voff, voff + nmesh + 1);
  h.toff.assign(toff, toff + nmesh + 1);
  rd::PatchInput in;
  in.nv = nv;
  in.nt = nt;
  in.tri = h.tri.data();
  in.x = h.x.data();
  in.y = h.y.data();
  if (px > 0.0) in.hpx = 0.5 * px;
  if (py > 0.0) in.hpy = 0.5 * py;
  in.row = h.row.data();
  in.slot = h.slot.data();
  in.voff = &h.voff;
  in.toff = &h.toff;
  in.max_tri = max_tri;
  in.own = own;
  in.threads = threads;
  if (!rd::build_patch_plan(in, h.P).empty()) return 1;
  const rd::PatchPlan& P = h.P;
  h.inv.assign(nv, -1);
  for (int64_t i = 0; i < nv; ++i) h.inv.at(P.order[i]) = (int32_t)i;
  for (int32_t v : h.inv) require(v >= 0, "order is a permutation");
  std::vector<int> owned(nt, 0);
  int64_t n = 0;
  for (int32_t t : P.tid)
    if (t >= 0) ++owned.at(t), ++n;
  for (int q : owned) require(q == 1, "every triangle owned once");
  for (int k = 0; k < nmesh; ++k)
    for (int32_t q = P.mbeg[k]; q < P.mbeg[k + 1]; ++q)
      require(P.pmesh[q] == k && P.vbeg[q] >= voff[k] && P.vbeg[q + 1] <= voff[k + 1], "patches within their mesh");
  rd::Patches& p = h.p;
  p.nv = nv;
  p.px = px;
  p.py = py;
  p.hpx = px > 0.0 ? 0.5 * px : HUGE_VAL;
  p.hpy = py > 0.0 ? 0.5 * py : HUGE_VAL;
  h.V.assign(nv, 0.0);
  for (int64_t t = 0; t < nt; ++t) {
    const int32_t* c = tri + 3 * t;
    const rd::TriDiff g = rd::tri_diff(p, make_double2(x[c[0]], y[c[0]]), make_double2(x[c[1]], y[c[1]]),
                                       make_double2(x[c[2]], y[c[2]]));
    for (int i = 0; i < 3; ++i) h.V[c[i]] += 0.5 * (g.d1x * g.d2y - g.d1y * g.d2x) / 3.0;
  }
  for (int64_t i = 0; i < nv; ++i)
    if (ghost && ghost[i]) h.V[i] = -h.V[i];
  if (nw > 0) {
    std::vector<std::vector<rd::WallEnt>> per(nv);
    for (int64_t e = 0; e < nw; ++e) {
      const int32_t a = wall[2 * e], b = wall[2 * e + 1];
      const double dx = rd::unwrap(x[b] - x[a], px, p.hpx), dy = rd::unwrap(y[b] - y[a], py, p.hpy);
      const double len = std::sqrt(dx * dx + dy * dy);
      per[a].push_back(rd::WallEnt{h.inv[b], 0, len / 2.0, dy / len, -dx / len});
      per[b].push_back(rd::WallEnt{h.inv[a], 1, len / 2.0, dy / len, -dx / len});
    }
    h.wb.assign(nv, -1);
    h.wptr.push_back(0);
    for (int64_t i = 0; i < nv; ++i)
      if (!per[i].empty()) {
        if (h.V[i] > 0.0) h.wb[h.inv[i]] = (int32_t)h.wptr.size() - 1;
        h.went.insert(h.went.end(), per[i].begin(), per[i].end());
        h.wptr.push_back((int32_t)h.went.size());
      }
  }
  const int64_t a[5] = {P.npatch, P.max_tri, (int64_t)P.halo.size(), (int64_t)P.tid.size(), n};
  for (int k = 0; k < 5; ++k) info[k] = a[k];
  return 0;
} catch (const std::exception&) {
  return 1;
}

// One step of W [4][nv] (caller's order) in place with dt = cfl * limit;
// returns dt, or NaN when an index check fails.
double patch_step(double* W, double cfl, int scheme, int time, int lump) try {
  std::vector<D4> w(h.nv), D(h.nv, D4{{0, 0, 0, 0}}), o(h.nv);
  for (int64_t i = 0; i < h.nv; ++i)
    for (int k = 0; k < 4; ++k) w[i].v[k] = W[k * h.nv + h.P.order[i]];
  double bound = INFINITY, none = 0.0;
  run(scheme, 1, false, w, D, o, 0.0, bound);
  const double dt = cfl * bound;
  D = o;
  if (time == 2) run(scheme, 2, lump != 0, w, D, o, dt, none);
  else
    for (int64_t i = 0; i < h.nv; ++i) o[i] = rd::patch_star(w[i], D[i], dt);
  for (int64_t i = 0; i < h.nv; ++i)
    for (int k = 0; k < 4; ++k) W[k * h.nv + h.P.order[i]] = o[i].v[k];
  return dt;
} catch (const std::exception&) {
  return NAN;
}
}
