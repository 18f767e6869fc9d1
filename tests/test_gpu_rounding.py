"""The rounding of one step. In the N scheme with global lumping the mass term
of the second stage is, per vertex, V (W* - W^n) / dt: the new state is W^n
minus dt / V times the mean of the two stages' residuals, rounded once,
whatever the rounding of W*. At a time step so short that this change is some
1e9 units in the last place, and its second order some units, FP64 residuals
give the change to a small part of a unit, and the rounding can be seen."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1705_02028_amd import inputs as I


@pytest.mark.parametrize("kw", [dict(N=24, diagonal="random", jitter=0.2), dict(N=160), dict(N=301, renumber="random")])
def test_the_new_state_is_rounded_once(orc, kw):
    from paper_1705_02028_amd import rd
    m = I.split_square(seed=3, **kw)
    W = I.random_smooth_state(m, seed=4, amp=0.2)
    om = orc.OracleMesh(m)
    dt, V = 3e-6 * om.max_dt(W, 0.4), om.geometry()["V"]
    R = om.residual(W, orc.N)
    Rs = om.residual(W - dt / V * R, orc.N)
    change = np.longdouble(dt) * (np.longdouble(0.5) * R + np.longdouble(0.5) * Rs) / V
    g = rd.Mesh(m)
    g.set_state(W)
    g.step(dt, rd.N, rd.RK2, rd.FP64)
    got = g.get_state()
    g.close()
    # components of ordinary size, whose change (good to 1e-12 of itself) is at
    # most 1e10 units: half a unit is the rounding's own
    unit = np.spacing(np.maximum(np.abs(W), np.abs(got)))
    seen = (np.abs(W) > 0.1) & (np.abs(change) < 1e10 * unit)
    assert seen.mean() > 0.4
    off = np.abs(got - (W - change)) / unit
    assert off[seen].max() <= 0.5 + 0.02
