"""A vertex in more triangles than a workgroup has threads, on the GPU against
the oracle: a closed fan (one other vertex per triangle; the parts then stand
behind the vertex records in LDS) and a pinwheel of triangles that share only
that vertex (two others per triangle: from 583 triangles on the vertex records
do not fit LDS and stand in memory)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1705_02028_amd import inputs as I
from test_gpu_parity import say


@pytest.fixture(scope="module")
def rd():
    from paper_1705_02028_amd import rd
    return rd


def around(n, closed):
    """n triangles around vertex 0, and a small mesh apart from them."""
    k = np.arange(n)
    a = 2 * np.pi * k / n
    if closed:
        x, y = np.r_[0.0, np.cos(a)], np.r_[0.0, np.sin(a)]
        tri = np.stack([0 * k, 1 + k, 1 + (k + 1) % n], 1)
    else:
        b = a + np.pi / n
        x, y = np.r_[0.0, np.cos(a), np.cos(b)], np.r_[0.0, np.sin(a), np.sin(b)]
        tri = np.stack([0 * k, 1 + k, 1 + n + k], 1)
    s = I.split_square(9, periodic=(False, False), bc=("ghost", "ghost"), diagonal="random", seed=8)
    nv = x.size
    ghost = np.r_[0, np.ones(nv - 1), np.asarray(s["ghost"])].astype(np.uint8)
    tri = np.concatenate([tri, np.asarray(s["tri"]).reshape(-1, 3) + nv]).astype(np.int32)
    return dict(x=np.r_[x, s["x"] + 3.0], y=np.r_[y, s["y"]], tri=tri, px=0.0, py=0.0, ghost=ghost,
                wall=np.zeros((0, 2), np.int32), nv=ghost.size, nt=len(tri), gamma=1.4)


def err(a, b):
    return max(np.abs(a[k] - b[k]).max() / np.abs(b[k]).max() for k in range(4))


@pytest.mark.parametrize("closed,n", [(True, 513), (True, 1023), (False, 513), (False, 582), (False, 583), (False, 1023)])
def test_every_call_matches_the_oracle(orc, rd, closed, n):
    m = around(n, closed)
    W = I.random_smooth_state(m, seed=7)
    om = orc.OracleMesh(m)
    dt = om.max_dt(W, 0.4)
    g = rd.Mesh(m)
    # the FP64 bar of one step: 1e-12 of each field's largest value
    for scheme in range(6):
        for time in (rd.EULER1, rd.RK2):
            for lump in ((0, 1) if time == rd.RK2 else (0,)):
                say(f"{'fan' if closed else 'pinwheel'} {n} scheme {scheme} time {time} lumping {lump}")
                g.lumping = lump
                om.set_lumping(bool(lump))
                ref = om.step(W, dt, scheme, time)
                for steps in (1, 2):
                    if steps == 2:
                        ref = om.step(ref, om.max_dt(ref, 0.4), scheme, time)
                    g.set_state(W)
                    g.step_cfl(steps, 0.4, scheme, time, rd.FP64)
                    assert err(g.get_state(), ref) <= steps * 1e-12
                g.set_state(W)
                g.step(dt, scheme, time, rd.FP64)
                assert err(g.get_state(), om.step(W, dt, scheme, time)) <= 1e-12
        g.set_state(W)
        assert g.max_dt(0.4) == pytest.approx(dt, rel=1e-13, abs=0.0)
        assert err(g.residual(scheme), om.residual(W, scheme)) <= 1e-12
    g.close()


@pytest.mark.parametrize("scheme", range(6))
def test_a_batch_with_such_a_member(rd, scheme):
    """Each member's bits are those it has alone, in whichever form."""
    ms = [around(900, False), I.split_square(12, periodic=(False, False), bc=("ghost", "ghost"), seed=8)]
    Ws = [I.random_smooth_state(m, seed=7) for m in ms]
    gs = [rd.Mesh(m) for m in ms]
    for g, W in zip(gs, Ws):
        g.set_state(W)
    b = rd.Batch(gs)
    b.run(3, 0.4, scheme, rd.RK2, rd.FP64)
    for m, g, W in zip(ms, gs, Ws):
        h = rd.Mesh(m)
        h.set_state(W)
        h.step_cfl(3, 0.4, scheme, rd.RK2, rd.FP64)
        assert np.array_equal(g.get_state(), h.get_state())
        h.close()
    b.close()
    for g in gs:
        g.close()
