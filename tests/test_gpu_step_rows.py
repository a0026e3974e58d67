"""The rows per group of the time steps follow the number of groups over all
instances; states and energies must not: a batch, single contexts and
two-row groups give the same bits.  Grids on both sides of the group limits
and of the row lengths where they change, with a ragged last group."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from tests.gpu_helpers import announce, gpu_context
from tests.test_gpu_batch import _batch_context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb,scheme", [((12, 21, 5), 24, "heun"), ((16, 19, 9), 24, "ab3m2"),
                                         ((30, 37, 7), 16, "heun"), ((60, 17, 9), 24, "euler"),
                                         ((40, 23, 11), 12, "heun"), ((90, 13, 5), 30, "heun"),
                                         ((130, 11, 3), 20, "heun"), ((140, 13, 3), 40, "heun")])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_rows_leave_results_alone(n, nb, scheme, prec):
    cfg = I.config("c1")
    cfg.update(n=n, layers=[0] * n[2], scheme=scheme, T=300.0)
    announce("rows of %s, %d instances, %s %s" % (n, nb, scheme, prec))
    dt = np.float32 if prec == "f32" else np.float64
    P = np.stack([I.initial_P(cfg, s, dt) for s in range(nb)])
    out = []
    for rows in (0, 2):
        ctx = _batch_context(cfg, prec, nb, [300.0] * nb, 1)
        try:
            T.tdgl_set_update_rows(ctx.ctx, rows)
            ctx.set_P(P)
            ctx.step(4)
            out.append((ctx.get_P(), ctx.energies_batch()[0]))
        finally:
            ctx.close()
    assert np.array_equal(out[0][0], out[1][0])
    for b in (0, nb - 1):
        one = gpu_context(cfg, prec, path=1)
        try:
            one.set_P(P[b])
            one.step(4)
            assert np.array_equal(one.get_P(), out[0][0][b])
            assert np.array_equal(np.array(one.energies()[0]), out[0][1][b])
        finally:
            one.close()
