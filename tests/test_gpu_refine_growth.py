"""The device arrays of mesh refinement grow with the mesh when the caller's
capacities allow: a mesh that outgrows the first allocation (65536 triangles'
room for an iteration that may triple them) is equal, entry by entry, to the
same refinement in arrays of a capacity that is allocated whole; and the
in-circle tests that only exact arithmetic decides (a lattice's co-circular
corners) give the same flips whether few or all edges need them."""
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


def points(n, jitter, seed):
    m = I.split_square(n, jitter=jitter, seed=seed)
    return dict(m, x=np.mod(m["x"], 1.0), y=np.mod(m["y"], 1.0))


@pytest.mark.parametrize("morton", [False, True])
def test_grown_arrays_give_the_same_mesh(rd, morton):
    m = points(20, 0.2, 1)
    kw = dict(max_radius=7.5e-3, max_ratio=2 ** 0.5, morton=morton)
    whole = rd.rd_delaunay_refine(m, max_vertices=60000, max_triangles=60000, **kw)
    assert 65536 // 3 < whole["nt"] <= 60000
    grown = rd.rd_delaunay_refine(m, max_vertices=400000, max_triangles=800000, **kw)
    for k in ("x", "y", "tri"):
        assert np.array_equal(whole[k], grown[k]), k
    assert (whole["n_iterations"], whole["n_flips"]) == (grown["n_iterations"], grown["n_flips"])


@pytest.mark.parametrize("n", [4, 40, 120])
def test_exact_tests_alone_flip_nothing(rd, n):
    m = points(n, 0.0, 1)
    tri, flips, rounds = rd.rd_delaunay_flip(m)
    assert flips == 0 and rounds == 0
    assert np.array_equal(tri, np.asarray(m["tri"]).reshape(tri.shape))
