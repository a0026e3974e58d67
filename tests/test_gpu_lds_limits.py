"""Contexts of one plan and different heights share their kernels, and with them
the kernels' limit of dynamic LDS: after a flatter box was made, the taller one
still steps, and gives the bits of a run of its own."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from tests.gpu_helpers import announce, gpu_context

pytestmark = pytest.mark.gpu

# taller, flatter, path: the two-kernel evaluation (99 and 93 KB), the fused plane
# pass (FP64 planes of 512 and 384 points of one z length)
PAIRS = [((32, 32, 16), (32, 32, 12), (0, 0, 0)), ((32, 32, 8), (32, 32, 6), (0, 0, 0)),
         ((32, 32, 16), (32, 32, 12), (1, 1, 0)), ((8, 8, 32), (8, 8, 20), (1, 1, 0))]


def _cfg(n, periodic):
    cfg = I.config("c1")
    cfg.update(n=n, layers=[0] * n[2], periodic=periodic, scheme="heun", mimg=1)
    return cfg


@pytest.mark.parametrize("tall,flat,periodic", PAIRS)
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_a_flatter_context_leaves_the_limit(tall, flat, periodic, prec):
    announce("LDS limit %s after %s periodic %s %s" % (tall, flat, periodic, prec))
    dt = np.float32 if prec == "f32" else np.float64
    a_cfg, b_cfg = _cfg(tall, periodic), _cfg(flat, periodic)
    P = I.initial_P(a_cfg, 2, dt)
    got = []
    for other in (True, False):
        a = gpu_context(a_cfg, prec)
        b = gpu_context(b_cfg, prec) if other else None
        try:
            a.set_P(P)
            if b:
                b.set_P(I.initial_P(b_cfg, 3, dt))
                b.step(2)
            a.step(5)
            got.append((a.get_P(), np.array(a.energies()[0])))
            assert T.tdgl_get_fft_path(a.ctx) == 1
        finally:
            a.close()
            if b:
                b.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
