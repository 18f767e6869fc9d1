"""Three-dimensional steps at the sizes where the tiles of a mesh can go wrong
(one tetrahedron, one tile, a tile and a remainder, each tile size, vertices in
scrambled order, tetrahedra that share no vertex) against the
three-dimensional oracle. Tolerance: the sums of a step are of at most a few
hundred terms each within a few ulp, so 1e-12 of each component's scale."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1705_02028_amd import inputs as I


@pytest.fixture(scope="module")
def rd():
    import torch
    assert torch.cuda.is_available()
    from paper_1705_02028_amd import rd
    return rd


@pytest.fixture(scope="module")
def O():
    import oracle3
    oracle3.build(force=False)
    return oracle3


def rel_err(a, b):
    return float((np.abs(a - b) / np.abs(b).max(axis=1, keepdims=True)).max())


def box(n, scramble):
    m = dict(I.cube_tets(n, jitter=0.1, seed=3))
    if scramble:
        rng = np.random.default_rng(4)
        p = rng.permutation(m["nv"])
        inv = np.argsort(p)
        for k in ("x", "y", "z"):
            m[k] = np.ascontiguousarray(m[k][p])
        tet = np.asarray(m["tet"]).reshape(-1, 4)
        m["tet"] = np.ascontiguousarray(inv[tet][rng.permutation(len(tet))].astype(np.int32))
    return m


def soup(n):
    """n tetrahedra that share no vertex, in a box without periods."""
    rng = np.random.default_rng(n)
    o = rng.uniform(0.0, 10.0, (n, 1, 3))
    p = o + np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]]) + rng.uniform(-0.1, 0.1, (n, 4, 3))
    p = p.reshape(-1, 3)
    m = dict(I.cube_tets(3))
    m.update(x=np.ascontiguousarray(p[:, 0]), y=np.ascontiguousarray(p[:, 1]), z=np.ascontiguousarray(p[:, 2]),
             tet=np.arange(4 * n, dtype=np.int32).reshape(-1, 4), nv=4 * n, nt=n)
    m.update(px=0.0, py=0.0, pz=0.0)
    return m


MESHES = {"box3": lambda: box(3, False), "box8": lambda: box(8, True), "box24": lambda: box(24, True),
          "one": lambda: soup(1), "soup63": lambda: soup(63), "soup300": lambda: soup(300)}


@pytest.mark.parametrize("name", list(MESHES))
@pytest.mark.parametrize("scheme", [0, 1, 2, 3, 4])
def test_tiles_match_the_oracle(rd, O, name, scheme):
    m = MESHES[name]()
    rng = np.random.default_rng(7)
    rho = rng.uniform(0.7, 1.4, m["nv"])
    u = rng.uniform(-0.6, 0.6, (3, m["nv"]))
    p = rng.uniform(0.7, 1.4, m["nv"])
    W = np.vstack([rho, rho * u, p / 0.4 + 0.5 * rho * (u * u).sum(0)])
    g, o = rd.Mesh3(m), O.OracleMesh3(m)
    g.set_state(W)
    dt = o.max_dt(W, 0.2)
    assert g.max_dt(0.2) == pytest.approx(dt, rel=1e-12)
    for time in (1, 2):
        g.set_state(W)
        g.step(dt, scheme, time)
        ref = o.step(W, dt, scheme, time)
        got = g.get_state()
        assert rel_err(got, ref) <= 1e-12, time
        g.set_state(W)
        g.step_cfl(1, 0.2, scheme, time)
        assert rel_err(g.get_state(), ref) <= 1e-12, time
    g.close()


@pytest.mark.parametrize("N", [25, 32, 33])
@pytest.mark.parametrize("scramble", [False, True])
def test_numbering_kept_or_not(rd, O, N, scramble):
    """Meshes of up to 32768 vertices keep the caller's numbering on the device,
    larger ones do not: a state comes back as it was set, and steps match the
    oracle, in either."""
    import torch
    m = box(N, scramble)
    W = I.ic3_kelvin_helmholtz(m, seed=5)
    om = O.OracleMesh3(m)
    g = rd.Mesh3(m)
    g.set_state(W)
    assert np.array_equal(g.get_state(), W)
    ref = W
    for _ in range(2):
        dt = om.max_dt(ref, 0.4)
        assert abs(g.max_dt(0.4) - dt) <= 1e-12 * dt
        g.step_cfl(1, 0.4, rd.B, rd.RK2)
        ref = om.step(ref, dt, rd.B, rd.RK2)
        assert rel_err(g.get_state(), ref) <= 2e-12
    out = torch.empty((5, m["nv"]), dtype=torch.float64, device="cuda")
    rd._check(rd.lib().rd3_get_state(g.h, out.data_ptr(), 1))
    assert np.array_equal(out.cpu().numpy(), g.get_state())
    g.close()
