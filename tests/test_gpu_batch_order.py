"""rd_batch_run only enqueues, its first run and one after a member's state has
moved to new buffers included: the work before it on the caller's stream is
still pending when it returns, and the results are those of steps in order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1705_02028_amd import inputs as I


@pytest.mark.parametrize("n", [2, 40])
def test_run_waits_for_nothing(n):
    from paper_1705_02028_amd import rd
    big = rd.Mesh(I.split_square(1024))
    s = torch.cuda.Stream()
    rd.rd_set_stream(big.h, s.cuda_stream)
    W0 = I.ic_kelvin_helmholtz(I.split_square(1024), seed=1)
    big.set_state(W0)
    big.step_cfl(1, 0.3, rd.B, rd.RK2, rd.FP64)
    big.sync()
    ms = [I.split_square(10 + k % 5, seed=k) for k in range(n)]
    Ws = [I.ic_kelvin_helmholtz(m, seed=k) for k, m in enumerate(ms)]
    gs = [rd.Mesh(m) for m in ms]
    for g, W in zip(gs, Ws):
        rd.rd_set_stream(g.h, s.cuda_stream)
        g.set_state(W)
    b = rd.Batch(gs, s.cuda_stream)
    ref = [rd.Mesh(m) for m in ms]
    for r, W in zip(ref, Ws):
        r.set_state(W)
    for k in range(3):
        if k == 2:
            for h in (gs[0], ref[0]):  # its state moves to buffers of its own
                h.step_cfl(1, 0.3, rd.B, rd.RK2, rd.FP32_ACC64)
                h.sync()
        big.step_cfl(500, 0.3, rd.B, rd.RK2, rd.FP64)  # about 0.09 s of work
        before = torch.cuda.Event()
        before.record(s)
        b.run(2, 0.3, rd.B, rd.RK2, rd.FP64)
        assert not before.query(), f"run {k} waited"
        for g, r in zip(gs, ref):
            r.step_cfl(2, 0.3, rd.B, rd.RK2, rd.FP64)
            assert np.array_equal(g.get_state(), r.get_state()), k
    for x in [b, big] + gs + ref:
        x.close()
