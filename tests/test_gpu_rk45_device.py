"""The RK45 controller on the device: one call, split calls (on both sides of the
64 attempts enqueued between two looks) and plain launches give the same
bits, time, step and rejections, for one instance and for a batch, with
rejections inside the run."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from tests.gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [0, 2])
@pytest.mark.parametrize("chunk,parts", [(0, (70,)), (64, (1, 1, 5, 63)), (64, (64, 6))])
def test_rk45_split_and_plain(nb, chunk, parts):
    cfg = I.config("c1")
    cfg.update(n=(9, 7, 5), layers=[0] * 5, scheme="rk45")
    if nb:
        cfg["T"] = [280.0, 340.0]
    P = [I.initial_P(cfg, s) for s in range(max(nb, 1))]
    announce("RK45 on the device, batch %d, graphs %d, calls %s" % (nb, chunk, parts))

    def run(chunk, parts):
        ctx = T.Context(cfg, T.TDGL_FP64, batch=nb)
        try:
            T.tdgl_set_graph_chunk(ctx.ctx, chunk)
            T.tdgl_set_rk_tolerances(ctx.ctx, 1e-9, 1e-7)
            ctx.set_P(np.stack(P) if nb else P[0])
            for n in parts:
                ctx.step(n)
            return ctx.get_P(), T.tdgl_get_rk_state(ctx.ctx)
        finally:
            ctx.close()

    got, (tau, h, rej) = run(chunk, parts)
    want, (tau1, h1, rej1) = run(64, (70,))
    assert rej1 > 0 and rej == rej1 and h == h1
    assert abs(tau - tau1) <= 70 * 2.0 ** -53 * tau1      # summed per call
    assert np.array_equal(got, want)
