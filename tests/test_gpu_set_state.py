"""A state from host memory is in place when rd_set_state returns: nothing of it
is pending on the stream, so the mesh may go on on another stream."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1705_02028_amd import inputs as I


@pytest.mark.parametrize("N", [24, 700])
@pytest.mark.parametrize("prec", [0, 1])
def test_host_state_then_another_stream(N, prec):
    from paper_1705_02028_amd import rd
    m = I.split_square(N, seed=1)
    W = [I.ic_kelvin_helmholtz(m, seed=k) * (1.0 + k) for k in range(2)]
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    g = rd.Mesh(m)
    rd.rd_set_stream(g.h, a.cuda_stream)
    g.set_state(W[0])
    g.step_cfl(1, 0.3, rd.B, rd.RK2, prec)  # the form the state is set in
    g.sync()
    for k in range(4):
        rd.rd_set_stream(g.h, (a, b)[k % 2].cuda_stream)
        g.set_state(W[k % 2])
        assert (a, b)[k % 2].query(), "work is pending on the stream"
        rd.rd_set_stream(g.h, (b, a)[k % 2].cuda_stream)
        assert np.array_equal(g.get_state(), W[k % 2])
    bad = W[0].copy()
    bad[0, 5] = 0.0
    with pytest.raises(rd.RDError, match="vertex 5 "):
        g.set_state(bad)
    assert np.array_equal(g.get_state(), W[1])
    g.step_cfl(1, 0.3, rd.B, rd.RK2, prec)
    g.sync()
    g.close()


@pytest.mark.parametrize("dim,N", [(2, 89), (2, 90), (3, 25), (3, 32), (3, 33)])
@pytest.mark.parametrize("prec", [0, 1])
def test_either_check_names_the_first_vertex(dim, N, prec):
    """Small host states are checked on the host, those of more than 8192
    vertices (32768 in three dimensions) on the device: the same vertex, and
    the state that was there stays."""
    from paper_1705_02028_amd import rd
    if dim == 2:
        m = I.split_square(N + 1, seed=1, periodic=(False, False), bc=("ghost", "ghost"))
        W, g = I.ic_kelvin_helmholtz(m, seed=1), rd.Mesh(m)
        g.set_state(W)
        g.step_cfl(1, 0.3, rd.B, rd.RK2, prec)
    else:
        m = I.cube_tets(N, seed=1)
        W, g = I.ic3_kelvin_helmholtz(m, seed=1), rd.Mesh3(m)
        g.set_state(W)
        g.step_cfl(1, 0.3, rd.B, rd.RK2)
    W = g.get_state()
    nv = m["nv"]
    for first, k, x in ((nv - 1, 0, 0.0), (nv // 2, 0, -1.0), (77, -1, np.nan), (3, -1, np.inf), (1, 1, 1e6)):
        bad = W.copy()
        bad[k, [first, nv - 1]] = x
        with pytest.raises(rd.RDError, match=f"vertex {first}\\b") as e:
            g.set_state(bad)
        assert e.value.status == rd.RD_ENONPHYS
        assert np.array_equal(g.get_state(), W)
    g.set_state(W)
    assert np.array_equal(g.get_state(), W)
    g.close()
