"""Tiles of a tetrahedral mesh (rd3_tiling.h) against a restatement with whole
ranges sorted: the same tiles in the same order whatever the number of workers
and however a range is cut, on lattices (whole planes of equal centroids), with
jitter, in scrambled order, on flat and on overflowing coordinates; and the
tables of each tile against its tetrahedra."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1705_02028_amd import inputs as I

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
TILE_VERTS = 256

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("tiles3") / "tiles3_shim.so")
    cmd = ["hipcc", "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-fPIC", "-shared", "-Xclang",
           "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(ROOT, "paper_1705_02028_amd", "csrc"), os.path.join(HERE, "cpp", "tiles3_shim.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    return C.CDLL(out)


def plan(shim, m, target, renumber, threads):
    nv, nt = m["nv"], m["nt"]
    tet = np.ascontiguousarray(m["tet"], np.int32).reshape(-1, 4)
    xyz = [np.ascontiguousarray(m[k], np.float64) for k in "xyz"]
    per = np.array([m["px"], m["py"], m["pz"]], np.float64)
    p = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    n = np.zeros(7, np.int64)
    assert shim.tiles3_build(C.c_int64(nv), C.c_int64(nt), p(tet), *map(p, xyz), p(per), target, int(renumber),
                             threads, p(n)) == 0
    o = dict(tile=np.zeros((n[0], 6), np.int32), tet=np.zeros((nt, 4), np.uint32), lv=np.zeros(n[1], np.int32),
             rpos=np.zeros(n[1], np.int32), deg=np.zeros(n[3], np.uint16), jb=np.zeros(n[2], np.int32),
             rbeg=np.zeros(nv + 1, np.int32), inv=np.zeros(nv, np.int32))
    shim.tiles3_get(*[p(o[k]) for k in ("tile", "tet", "lv", "rpos", "deg", "jb", "rbeg", "inv")])
    o["max"] = n[4:].tolist()
    return o


def tiles_by_sorting(m, target):
    """Lists of tetrahedra, ascending in each tile."""
    tet = np.asarray(m["tet"], np.int64).reshape(-1, 4)
    c = np.zeros((len(tet), 3), np.float32)
    with np.errstate(over="ignore"):
        for k, (a, per) in enumerate(zip("xyz", (m["px"], m["py"], m["pz"]))):
            x = np.asarray(m[a])[tet]
            s = np.zeros(len(tet))
            for i in (1, 2, 3):
                d = x[:, i] - x[:, 0]
                if per > 0:
                    d = np.where(d > 0.5 * per, d - per, np.where(d < -0.5 * per, d + per, d))
                s = s + d
            c[:, k] = (x[:, 0] + 0.25 * s).astype(np.float32)
    out = []

    def go(ids):
        if len(ids) == 0:
            return
        if len(ids) <= target and len(np.unique(tet[ids])) <= TILE_VERTS:
            out.append(np.sort(ids))
            return
        with np.errstate(invalid="ignore"):
            span = c[ids].max(0) - c[ids].min(0)
        a = 0
        for k in (1, 2):
            if span[k] > span[a]:
                a = k
        n = -(-len(ids) // target)
        at = len(ids) * (n // 2) // n if n > 1 else len(ids) // 2
        o = ids[np.lexsort((ids, c[ids, a]))]
        go(o[:at])
        go(o[at:])

    go(np.arange(len(tet)))
    return out


def box(n, jitter, scramble=False):
    m = dict(I.cube_tets(n, jitter=jitter, seed=3))
    if scramble:
        rng = np.random.default_rng(4)
        p = rng.permutation(m["nv"])
        for k in "xyz":
            m[k] = np.ascontiguousarray(m[k][p])
        tet = np.asarray(m["tet"]).reshape(-1, 4)
        m["tet"] = np.argsort(p)[tet][rng.permutation(len(tet))].astype(np.int32)
    return m


def soup(n, scale):
    """n tetrahedra that share no vertex, in a box without periods."""
    rng = np.random.default_rng(n)
    o = rng.uniform(0.0, 10.0, (n, 1, 3))
    p = o + np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]]) + rng.uniform(-0.1, 0.1, (n, 4, 3))
    p = (p * np.asarray(scale)).reshape(-1, 3)
    m = dict(I.cube_tets(3))
    m.update(zip("xyz", np.ascontiguousarray(p.T)))
    m.update(tet=np.arange(4 * n, dtype=np.int32).reshape(-1, 4), nv=4 * n, nt=n, px=0.0, py=0.0, pz=0.0)
    return m


MESHES = {"lattice": lambda: box(9, 0.0), "jitter": lambda: box(10, 0.15), "scrambled": lambda: box(9, 0.1, True),
          "large": lambda: box(21, 0.15), "large_lattice": lambda: box(21, 0.0), "one": lambda: soup(1, 1.0),
          "soup": lambda: soup(700, 1.0), "flat": lambda: soup(700, [1e-45, 1e-45, 1e-45]),
          "tiny": lambda: soup(700, 1e-36), "overflow": lambda: soup(700, 1e38)}


@pytest.mark.parametrize("name", list(MESHES))
@pytest.mark.parametrize("target", [64, 256])
def test_tiles(shim, name, target):
    m = MESHES[name]()
    tet = np.asarray(m["tet"], np.int64).reshape(-1, 4)
    want = tiles_by_sorting(m, target)
    for threads, renumber in ((1, True), (4, True), (8, False)):
        P = plan(shim, m, target, renumber, threads)
        assert len(P["tile"]) == len(want)
        back = np.full(m["nv"], -1)
        back[P["inv"]] = np.arange(m["nv"])
        assert (back >= 0).all()
        if not renumber:
            assert np.array_equal(P["inv"], np.arange(m["nv"]))
        t0 = l0 = j0 = 0
        first = []
        for (a, n, l, nlv, j, nj), ids in zip(P["tile"], want):
            assert (a, n, l, j) == (t0, len(ids), l0, j0)
            lv, deg = P["lv"][l:l + nlv], P["deg"][l:l + nlv]
            word = P["tet"][a:a + n]
            loc, slot = word & 0xffff, word >> 16
            assert np.array_equal(back[lv[loc]], tet[ids])
            assert np.array_equal(np.bincount(loc.ravel(), minlength=nlv), deg)
            # by falling degree, then the caller's id
            assert np.array_equal(np.lexsort((back[lv], -deg.astype(int))), np.arange(nlv))
            # slot of the k-th part of a vertex: diagonal k, in the order of the tetrahedra
            o = np.argsort(loc.ravel(), kind="stable")
            rank = np.empty(4 * n, int)
            rank[o] = np.concatenate([np.arange(d) for d in deg])
            jb = P["jb"][j:j + nj]
            assert nj == deg[0] and np.array_equal(jb, np.concatenate([[0], np.cumsum([(deg > k).sum() for k in range(nj)])])[:-1])
            assert np.array_equal(slot.ravel(), jb[rank] + loc.ravel())
            assert np.array_equal(np.sort(slot.ravel()), np.arange(4 * n))
            first.extend(lv)
            t0, l0, j0 = t0 + n, l0 + nlv, j0 + nj
        assert t0 == m["nt"]
        if renumber:  # numbered as first met
            u, i = np.unique(first, return_index=True)
            assert np.array_equal(u, np.arange(m["nv"])) and (np.diff(i) > 0).all()
        o = np.argsort(P["lv"], kind="stable")
        assert np.array_equal(P["rpos"][o], np.arange(l0))
        assert np.array_equal(P["rbeg"], np.concatenate([[0], np.cumsum(np.bincount(P["lv"], minlength=m["nv"]))]))
        assert P["max"] == [P["tile"][:, 3].max(), P["tile"][:, 1].max(), P["tile"][:, 5].max()]
