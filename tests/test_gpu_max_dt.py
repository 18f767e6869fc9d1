"""rd_max_dt is the limit of the current state after steps of either precision
and form, steps of a given dt included, against the oracle at that state."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1705_02028_amd import inputs as I


@pytest.fixture(scope="module")
def rd():
    from paper_1705_02028_amd import rd
    return rd


MESHES = {
    "periodic": lambda: I.split_square(24, seed=2, diagonal="random", renumber="random"),
    "box": lambda: I.split_square(37, periodic=(False, False), bc=("ghost", "wall"), seed=2, jitter=0.1),
    "large": lambda: I.split_square(400, seed=1),  # more patches than a workgroup reduces by itself
}


@pytest.mark.parametrize("kind", sorted(MESHES))
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("tile", [0, 64])
@pytest.mark.parametrize("time", [1, 2])
def test_max_dt_is_that_of_the_current_state(orc, rd, kind, prec, tile, time):
    m = MESHES[kind]()
    om = orc.OracleMesh(m)
    states = [I.ic_kelvin_helmholtz(m, seed=k) * (1.0 + k) for k in range(2)]
    g = rd.Mesh(m)
    g.tile = tile

    def check(what):
        # a quotient of FP64 sums: fewer than fifteen roundings of 2.2e-16
        W = g.get_state()
        assert g.max_dt(0.3) == pytest.approx(om.max_dt(W, 0.3), rel=1e-14, abs=0.0), what
        assert np.array_equal(g.get_state(), W), what

    g.set_state(states[0])
    dt = om.max_dt(states[0], 0.3)
    for k in range(2):
        g.step(dt, rd.B, time, prec)
        check(f"given dt, step {k}")
    for k in range(2):
        g.step_cfl(1, 0.3, rd.B, time, prec)
        check(f"CFL step {k}")
    W = states[1].copy()
    W[3] *= 2.0  # faster sound
    g.set_state(W)
    check("a new state")
    g.step(0.1 * dt, rd.B, time, prec)
    check("given dt at the new state")
    g.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_max_dt_after_replays(orc, rd, prec):
    """The state moved by a captured step, which the host does not see."""
    m = MESHES["box"]()
    om = orc.OracleMesh(m)
    W = I.ic_kelvin_helmholtz(m, seed=1)
    s = torch.cuda.Stream()
    g = rd.Mesh(m)
    for p in (1 - prec, prec):
        g.set_state(W)
        g.step_cfl(1, 0.3, rd.B, rd.RK2, p)
    torch.cuda.synchronize()
    rd.rd_set_stream(g.h, s.cuda_stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s, capture_error_mode="thread_local"):
        g.step_cfl(1, 0.3, rd.B, rd.RK2, prec)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert g.max_dt(0.3) == pytest.approx(om.max_dt(g.get_state(), 0.3), rel=1e-14, abs=0.0), k
        g.step_cfl(1, 0.3, rd.B, rd.RK2, 1 - prec)
        assert g.max_dt(0.3) == pytest.approx(om.max_dt(g.get_state(), 0.3), rel=1e-14, abs=0.0), k
    g.close()


@pytest.mark.parametrize("N", [9, 350])  # the last workgroup's minimum; a kernel of its own above 512 patches
def test_every_call_the_same(rd, N):
    """The first call of a mesh brings the result back by a copy, later ones
    read what the device wrote to host memory."""
    m = I.split_square(N, jitter=0.2, seed=7)
    W = I.random_smooth_state(m, seed=8)
    g = rd.Mesh(m)
    g.set_state(W)
    dt = [g.max_dt(0.4) for _ in range(4)]
    g.step_cfl(1, 0.4, rd.B, rd.RK2)
    after = [g.max_dt(0.4) for _ in range(2)]
    g.set_state(g.get_state())
    h = rd.Mesh(m)
    h.set_state(g.get_state())
    assert dt == dt[:1] * 4 and after == [h.max_dt(0.4)] * 2 and after[0] != dt[0]
    g.close()
    h.close()
