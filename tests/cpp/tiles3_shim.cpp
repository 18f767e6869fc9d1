// The tiles of a tetrahedral mesh (rd3_tiling.h) for the CPU tests.
#include "rd3_tiling.h"

namespace {
rd3::TilePlan3 P;

template <class V, class T>
void copy(const V& v, T* out) {
  std::copy(v.begin(), v.end(), out);
}
}  // namespace

extern "C" int tiles3_build(int64_t nv, int64_t nt, const int32_t* tet, const double* x, const double* y,
                            const double* z, const double* per, int target, int renumber, int threads, int64_t* sizes) {
  const double* xyz[3] = {x, y, z};
  rd::Workers pool(threads);
  P = rd3::TilePlan3();
  if (!rd3::build_tiles3(nv, nt, tet, xyz, per, target, renumber != 0, pool, P).empty()) return 1;
  const int64_t n[7] = {(int64_t)P.tile.size(), (int64_t)P.lv.size(), (int64_t)P.jb.size(), (int64_t)P.deg.size(),
                        P.max_lv, P.max_tet, P.max_jd};
  std::copy(n, n + 7, sizes);
  return 0;
}

extern "C" void tiles3_get(int32_t* tile, uint32_t* tet, int32_t* lv, int32_t* rpos, uint16_t* deg, int32_t* jb,
                           int32_t* rbeg, int32_t* inv) {
  for (const rd3::Tile3& t : P.tile)
    for (int32_t v : {t.t0, t.nt, t.l0, t.nlv, t.j0, t.nj}) *tile++ = v;
  copy(P.tet, tet);
  copy(P.lv, lv);
  copy(P.rpos, rpos);
  copy(P.deg, deg);
  copy(P.jb, jb);
  copy(P.rbeg, rbeg);
  copy(P.inv, inv);
}
