"""Triangle residuals of rd_residual: exactly 0 on every triangle whose three
corners hold the same state (each corner's parameter vector is the same
arithmetic on the same numbers), and elsewhere near the differential of the
fluxes in extended precision. Tolerance there: with z the largest entry of the
corners' Z and d the largest coordinate difference, the terms add up to at most
8 z^2 d; each factor Z is within 4 roundings of its value, and 8 more follow, so
8 (4 + 4 + 8) = 128 roundings of z^2 d."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1705_02028_amd import inputs as I

MESHES = {
    "ghost": lambda: I.split_square(60, periodic=(False, False), bc=("ghost", "ghost"), diagonal="random", jitter=0.2,
                                    seed=3),
    "periodic": lambda: I.split_square(33, jitter=0.2, renumber="random", seed=4),
    "small": lambda: I.split_square(3, periodic=(False, False), bc=("wall", "wall")),
}


def z_of(W, gamma=1.4):
    rho, m, n, e = W
    p = (gamma - 1.0) * (e - 0.5 * (m * m + n * n) / rho)
    s = np.sqrt(rho)
    return np.array([s, m / s, n / s, (e + p) / s])


@pytest.mark.parametrize("name", list(MESHES))
def test_uniform_triangles(name):
    import torch
    assert torch.cuda.is_available()
    from paper_1705_02028_amd import rd
    m = MESHES[name]()
    tri = np.asarray(m["tri"]).reshape(-1, 3)
    x, y = np.asarray(m["x"]), np.asarray(m["y"])
    g = rd.Mesh(m)
    for seed in range(4):
        r = np.random.default_rng(seed)
        # a few states, each on a patch of the plane
        k = (2 * ((x > 0.5) & (seed > 0)) + ((y > 0.4) & (seed > 1))).astype(int)
        rho, u, v, p = r.uniform(0.5, 2, 4), r.uniform(-1, 1, 4), r.uniform(-1, 1, 4), r.uniform(0.5, 2, 4)
        W = np.ascontiguousarray(np.array([rho, rho * u, rho * v, p / 0.4 + 0.5 * rho * (u * u + v * v)])[:, k])
        g.set_state(W)
        _, phi = g.residual(rd.B, with_phiT=True)
        same = (W[:, tri[:, 1:]] == W[:, tri[:, :1]]).all((0, 2))
        assert same.any()
        assert (phi[:, same] == 0.0).all()
        # the others against the flux differential in extended precision
        Z = z_of(W.astype(np.longdouble))[:, tri]
        d = []
        for c, per in ((x, m["px"]), (y, m["py"])):
            q = c[tri[:, 1:]] - c[tri[:, :1]]
            d.append(np.where(q > 0.5 * per, q - per, np.where(q < -0.5 * per, q + per, q)) if per > 0 else q)
        d1x, d2x, d1y, d2y = d[0][:, 0], d[0][:, 1], d[1][:, 0], d[1][:, 1]
        dz1, dz2, s = Z[:, :, 1] - Z[:, :, 0], Z[:, :, 2] - Z[:, :, 0], Z.sum(2)
        X, Y = d2y * dz1 - d1y * dz2, d1x * dz2 - d2x * dz1
        f = np.longdouble(0.4) / np.longdouble(1.4)
        pr = [f * (s[0] * D[3] + s[3] * D[0] - s[1] * D[1] - s[2] * D[2]) for D in (X, Y)]
        want = np.array([s[0] * (X[1] + Y[2]) + s[1] * X[0] + s[2] * Y[0],
                         2 * s[1] * X[1] + pr[0] + s[1] * Y[2] + s[2] * Y[1],
                         s[1] * X[2] + s[2] * X[1] + 2 * s[2] * Y[2] + pr[1],
                         s[3] * (X[1] + Y[2]) + s[1] * X[3] + s[2] * Y[3]]) / 6
        scale = (np.abs(Z).max((0, 2)) ** 2 * np.abs(d).max((0, 2))).astype(float)
        assert (np.abs(phi - want)[:, ~same] <= 128 * 2.0**-53 * scale[~same]).all()
    g.close()
