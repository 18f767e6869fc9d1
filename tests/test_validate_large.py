"""The checks of a mesh description on meshes large enough for several workers:
the first bad triangle or vertex is named wherever it is, whatever the
numbering, and a good mesh passes."""
import numpy as np
import pytest

from paper_1705_02028_amd import inputs as I


@pytest.fixture(scope="module", params=[None, "random"])
def mesh(request):
    m = I.split_square(160, periodic=(False, False), bc=("ghost", "wall"), diagonal="random", renumber=request.param)
    return {k: (np.ascontiguousarray(v) if isinstance(v, np.ndarray) else v) for k, v in m.items()}


def refused(m, text):
    from paper_1705_02028_amd import rd
    with pytest.raises(rd.RDError, match=text) as e:
        rd.rd_mesh_validate(m)
    assert e.value.status == rd.RD_EINVAL


def test_a_good_mesh_passes(mesh):
    from paper_1705_02028_amd import rd
    assert mesh["nt"] > 30000
    rd.rd_mesh_validate(mesh)


@pytest.mark.parametrize("where", [0, 1023, 1024, 20000, -1])
def test_the_first_bad_triangle_is_named(mesh, where):
    nt, tri = mesh["nt"], np.asarray(mesh["tri"]).reshape(-1, 3)
    t = where % nt
    for later in {t, nt - 1}:
        bad = tri.copy()
        bad[[t, later]] = bad[[t, later]][:, [0, 2, 1]]
        refused(dict(mesh, tri=bad), f"triangle {t} is not counter-clockwise")
        for index in (-1, mesh["nv"], 2**31 - 1, -2**31):
            bad = tri.copy()
            bad[[t, later], 1] = index
            refused(dict(mesh, tri=bad), f"triangle {t} has a vertex index out of range")


@pytest.mark.parametrize("extra", [1, 3])
def test_the_first_unused_vertex_is_named(mesh, extra):
    """A vertex no triangle has, in the middle of the numbering and at its end."""
    nv, tri = mesh["nv"], np.asarray(mesh["tri"]).reshape(-1, 3)
    for at in (0, nv // 2, nv):
        m = dict(mesh, nv=nv + extra, tri=(tri + extra * (tri >= at)).astype(np.int32),
                 wall=(np.asarray(mesh["wall"]) + extra * (np.asarray(mesh["wall"]) >= at)).astype(np.int32))
        for k in ("x", "y", "ghost"):
            m[k] = np.insert(mesh[k], [at] * extra, 0)
        refused(m, f"vertex {at} belongs to no triangle")


@pytest.mark.parametrize("n", [1023, 1024])
def test_the_largest_degree(mesh, n):
    from paper_1705_02028_amd import rd
    a = 2 * np.pi * np.arange(n) / n
    k = np.arange(n)
    nv, tri = mesh["nv"], np.asarray(mesh["tri"]).reshape(-1, 3)
    fan = np.stack([0 * k, 1 + k, 1 + (k + 1) % n], 1) + nv
    m = dict(mesh, nv=nv + n + 1, nt=mesh["nt"] + n, tri=np.concatenate([tri, fan]).astype(np.int32),
             x=np.r_[mesh["x"], 5.0, 5.0 + np.cos(a)], y=np.r_[mesh["y"], 5.0, 5.0 + np.sin(a)],
             ghost=np.r_[mesh["ghost"], np.zeros(n + 1, mesh["ghost"].dtype)])
    if n <= 1023:
        rd.rd_mesh_validate(m)
    else:
        refused(m, f"vertex {nv} belongs to {n} triangles; at most 1023")
