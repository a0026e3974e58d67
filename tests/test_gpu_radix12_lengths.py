"""Every transform length 3 * 2^a from 24 to 768, in x and in y (one has a single
stage before the last one of radix 12, others a radix 2 between): the field
against the oracle, tolerances as for the other lengths (1e-13 of the
field's norm in FP64, 2e-6 in FP32)."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from oracle import tdgl_oracle as O
from tests.gpu_helpers import announce, gpu_context, oracle_field, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,length", [(11, 24), (22, 48), (41, 96), (95, 192), (130, 384),
                                          (300, 768)])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_field_at_lengths_of_three_powers_of_two(cells, length, axis, prec):
    n = [9, 9, 2]
    n[axis] = cells
    cfg = I.config("c1")
    cfg.update(n=tuple(n), layers=[0] * 2, eext=(2e6, -1e6, 3e6))
    announce("radix 12, length %d, axis %d, %s" % (length, axis, prec))
    P = I.initial_P(cfg, 3, np.float32 if prec == "f32" else np.float64)
    want = oracle_field(P.astype(np.float64), O.Problem(cfg), T.TDGL_ALL)
    for path in (0, 1):
        ctx = gpu_context(cfg, prec, path=path)
        try:
            assert T.tdgl_get_dims(ctx.ctx)[3 + axis] == length
            ctx.set_P(P)
            got = ctx.eval_field(T.TDGL_ALL).cpu().numpy()
        finally:
            ctx.close()
        assert rel_inf(got, want) <= (1e-13 if prec == "f64" else 2e-6), path
