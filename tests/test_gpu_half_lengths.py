"""y transforms of 3 * 2^a points whose lines are half filled (the pruned form of
the y pass), and of 24 points, whose FP64 lines take other radices: field
against the oracle, 1e-13 of its norm in FP64, 2e-6 in FP32."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from oracle import tdgl_oracle as O
from tests.gpu_helpers import announce, gpu_context, oracle_field, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,length", [(9, 24), (12, 24), (24, 48), (48, 96), (96, 192), (192, 384)])
@pytest.mark.parametrize("nb", [0, 3])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_field_of_half_filled_lines(ny, length, nb, prec):
    n = (10, ny, 3)
    cfg = I.config("c1")
    cfg.update(n=n, layers=[0] * 3)
    announce("half-filled y of %d points, batch %d, %s" % (length, nb, prec))
    P = np.stack([I.initial_P(cfg, s, np.float32 if prec == "f32" else np.float64)
                  for s in range(max(nb, 1))])
    if nb:
        ctx = T.Context(dict(cfg, T=[300.0] * nb), T.TDGL_FP64 if prec == "f64" else T.TDGL_FP32,
                        batch=nb)
    else:
        ctx = gpu_context(cfg, prec)
    try:
        assert ctx.dims[4] == length
        ctx.set_P(P if nb else P[0])
        got = ctx.eval_field(T.TDGL_ALL).cpu().numpy().reshape(P.shape)
    finally:
        ctx.close()
    prob = O.Problem(cfg)
    for b in range(len(P)):
        want = oracle_field(P[b].astype(np.float64), prob, T.TDGL_ALL)
        assert rel_inf(got[b], want) <= (1e-13 if prec == "f64" else 2e-6), b
