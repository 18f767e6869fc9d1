"""The exact in-circle pass at the edges of its launches (64 edges a workgroup,
4096 a sweep): on a regular lattice the diagonal of every cell is undecided in
FP64 and legal, so nothing may flip; with a vertex moved by an ulp the result
is Delaunay by the exact reference and the cells away from it stay."""
import numpy as np
import pytest

from paper_1705_02028_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [5, 8, 9, 64, 65])
def test_regular_lattices(N):
    from paper_1705_02028_amd import rd
    m = I.split_square(N)
    tri, flips, rounds = rd.rd_delaunay_flip(m)
    assert flips == 0 and rounds == 0
    assert np.array_equal(tri, np.asarray(m["tri"]).reshape(-1, 3))


@pytest.mark.parametrize("N", [8, 17])
def test_a_vertex_off_by_an_ulp(N):
    import delaunay as D
    from paper_1705_02028_amd import rd
    m = I.split_square(N, periodic=(False, False), bc=("ghost", "ghost"))
    v = int(np.argmin(np.hypot(m["x"] - 0.5, m["y"] - 0.5)))
    for to in (0.0, 1.0):
        q = dict(m, x=m["x"].copy())
        q["x"][v] = np.nextafter(q["x"][v], to)
        tri, flips, _ = rd.rd_delaunay_flip(q)
        assert D.violations(q, tri) == []
        assert (tri != np.asarray(m["tri"]).reshape(-1, 3)).any(axis=1).sum() <= 12
