"""The patch form on the host: the patches of a mesh (rd_patching.h) and the
passes of one step over them with the GPU kernels' bodies, every index
checked, against the CPU oracle. The sizes sit where the cutting can go wrong:
meshes smaller than a patch, groups cut again to fit a workgroup, a vertex in
more triangles than a patch may have, two meshes end to end, any numbering."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1705_02028_amd import inputs as I

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("patch") / "patch_shim.so")
    cmd = ["hipcc", "--offload-arch=gfx950", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_1705_02028_amd", "csrc"), os.path.join(HERE, "cpp", "patch_shim.cpp"),
           "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    lib = C.CDLL(out)
    lib.patch_step.restype = C.c_double
    lib.patch_step.argtypes = [C.c_void_p, C.c_double, C.c_int, C.c_int, C.c_int]
    return lib


def build(shim, m, own=210, max_tri=512, voff=None, toff=None, threads=3):
    tri = np.ascontiguousarray(m["tri"], np.int32)
    wall = np.ascontiguousarray(m["wall"], np.int32).reshape(-1, 2)
    ghost = np.ascontiguousarray(m["ghost"], np.uint8)
    vo = np.array([0, m["nv"]] if voff is None else voff, np.int64)
    to = np.array([0, m["nt"]] if toff is None else toff, np.int64)
    info = np.zeros(5, np.int64)
    p = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    x, y = np.ascontiguousarray(m["x"]), np.ascontiguousarray(m["y"])
    st = shim.patch_build(C.c_int64(m["nv"]), C.c_int64(m["nt"]), p(tri), p(x), p(y), C.c_double(m["px"]),
                          C.c_double(m["py"]), p(ghost), C.c_int64(len(wall)), p(wall), C.c_int(len(vo) - 1), p(vo),
                          p(to), C.c_int(own), C.c_int(max_tri), C.c_int(threads), p(info))
    assert st == 0
    return dict(zip(("patches", "max_tri", "halo", "listed", "owned"), info.tolist()))


def err(a, b):
    return max(np.abs(a[k] - b[k]).max() / np.abs(b[k]).max() for k in range(4))


MESHES = {
    "periodic": lambda: I.split_square(24, diagonal="random", seed=1, jitter=0.2),
    "channel": lambda: I.split_square(21, periodic=(False, False), bc=("ghost", "wall"), renumber="random", seed=2),
    "box": lambda: I.split_square(17, periodic=(False, True), bc=("wall", "ghost"), diagonal="random", seed=3),
    "two": lambda: I.split_square(2, periodic=(False, False), bc=("wall", "wall")),
}


@pytest.mark.parametrize("case", sorted(MESHES))
def test_patch_steps_match_the_oracle(orc, shim, case):
    m = MESHES[case]()
    W = I.random_smooth_state(m, seed=4, amp=0.2)
    om = orc.OracleMesh(m)
    dt = om.max_dt(W, 0.4)
    for scheme in range(5):
        for time in (1, 2):
            ref = om.step(W, dt, scheme, time)
            for kw in (dict(), dict(own=20), dict(own=40, max_tri=20)):
                info = build(shim, m, **kw)
                assert info["owned"] == m["nt"]
                got = W.copy()
                # the FP64 bar of one step: 1e-12 of each field's largest value
                assert abs(shim.patch_step(got.ctypes.data, 0.4, scheme, time, 0) - dt) <= 1e-14 * dt
                assert err(got, ref) <= 1e-12, (scheme, time, kw)


def test_results_do_not_depend_on_the_patches(shim):
    m = I.split_square(40, periodic=(True, False), bc=("ghost", "wall"), diagonal="random", seed=5, jitter=0.2,
                       renumber="random")
    W = I.random_smooth_state(m, seed=6, amp=0.2)
    outs = []
    for kw in (dict(), dict(own=30), dict(own=5000, max_tri=100000), dict(own=1)):
        build(shim, m, threads=1 + len(outs), **kw)
        for lump in (0, 1):
            got = W.copy()
            assert shim.patch_step(got.ctypes.data, 0.4, 2, 2, lump) > 0.0
            outs.append((lump, got))
    for lump, got in outs[2:]:
        assert np.array_equal(got, outs[lump][1])


def fan(n):
    """n triangles around one vertex."""
    a = 2 * np.pi * np.arange(n) / n
    x, y = np.r_[0.0, np.cos(a)], np.r_[0.0, np.sin(a)]
    k = np.arange(n)
    tri = np.stack([np.zeros(n, int), 1 + k, 1 + (k + 1) % n], 1)
    return dict(x=x, y=y, tri=tri.astype(np.int32), px=0.0, py=0.0, ghost=np.r_[0, np.ones(n)].astype(np.uint8),
                wall=np.zeros((0, 2), np.int32), nv=n + 1, nt=n, gamma=1.4)


@pytest.mark.parametrize("n", [3, 511, 512, 513, 1023])
def test_a_vertex_of_high_degree(orc, shim, n):
    m = fan(n)
    W = I.random_smooth_state(m, seed=7)
    info = build(shim, m, max_tri=512 if n <= 512 else 256)
    assert info["max_tri"] == n
    om = orc.OracleMesh(m)
    got = W.copy()
    dt = shim.patch_step(got.ctypes.data, 0.4, 2, 2, 0)
    assert err(got, om.step(W, dt, orc.B, orc.RK2)) <= 1e-12


def test_meshes_end_to_end(shim):
    a = I.split_square(12, periodic=(False, False), bc=("ghost", "ghost"), diagonal="random", seed=8)
    b = I.split_square(5, periodic=(False, False), bc=("ghost", "ghost"))
    m = I.concat_meshes([a, b, a])
    m["ghost"] = m["ghost"].astype(np.uint8)
    info = build(shim, m, own=20, voff=m["voff"], toff=m["toff"])
    assert info["owned"] == m["nt"] and info["patches"] >= 2 * 8 + 2
