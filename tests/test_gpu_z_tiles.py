"""The z pass with one wave per tile against the tiles of 128 bytes, on both sides
of its limits: the same bits for every length, half-filled and ragged z
lines, periodic z, vacuum, tiles that end beyond the plane, and an instance
of a batch has those of a single context; the field against the oracle."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from oracle import tdgl_oracle as O
from tests.gpu_helpers import announce, gpu_context, oracle_field, rel_inf
from tests.test_gpu_batch import _batch_context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb,periodic", [
    ((40, 25, 4), 60, (0, 0, 0)), ((33, 4, 3), 70, (0, 0, 0)),           # mz 8
    ((20, 33, 8), 64, (0, 0, 0)), ((48, 21, 7), 64, (0, 0, 0)),          # 16
    ((24, 32, 16), 40, (0, 0, 0)), ((24, 30, 11), 40, (0, 0, 0)),        # 32
    ((17, 32, 32), 24, (0, 0, 0)), ((32, 20, 21), 24, (0, 0, 0)),        # 64
    ((16, 16, 64), 4, (1, 1, 1)), ((64, 32, 32), 6, (1, 1, 0)),
    ((7, 9, 64), 1, (0, 0, 0)), ((9, 8, 41), 30, (0, 0, 0)),             # 128
    ((16, 16, 64), 7, (0, 0, 0)), ((16, 16, 64), 6, (0, 0, 0))])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_wave_tiles_give_the_bits_of_row_tiles(n, nb, periodic, prec):
    cfg = I.config("c1")
    cfg.update(n=n, periodic=periodic, mimg=1, scheme="heun", T=300.0,
               layers=[0] * (n[2] - 1) + [0 if periodic[2] else -1])
    announce("z tiles %s x %d %s %s" % (n, nb, periodic, prec))
    dt = np.float32 if prec == "f32" else np.float64
    P = np.stack([I.initial_P(cfg, s, dt) for s in range(nb)])
    out = []
    for tile in (0, 128):
        ctx = _batch_context(cfg, prec, nb, [300.0] * nb, 1)
        try:
            T.tdgl_set_z_tile(ctx.ctx, tile)
            ctx.set_P(P)
            E = ctx.eval_field(T.TDGL_ELEC).cpu().numpy()
            ctx.step(3)
            out.append((E.reshape(P.shape), ctx.get_P().reshape(P.shape)))
        finally:
            ctx.close()
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
    want = oracle_field(P[-1].astype(np.float64), O.Problem(cfg), T.TDGL_ELEC)
    assert rel_inf(out[0][0][-1], want) <= (1e-13 if prec == "f64" else 2e-6)
    one = gpu_context(cfg, prec, path=1)
    try:
        one.set_P(P[0])
        one.step(3)
        assert np.array_equal(one.get_P(), out[0][1][0])
    finally:
        one.close()
