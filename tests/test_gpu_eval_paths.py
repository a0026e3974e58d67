"""Which evaluation a context takes (0 three passes, 1 fused plane pass, 2 two
kernels) on both sides of every line of the rule, and that an instance of a
batch on one path has the bits of a single context on another.  tdgl_autotune
also times the plane pass where the rule does not take it."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from tests.gpu_helpers import PREC, announce, gpu_context
from tests.test_gpu_batch import _batch_context
from tests.test_gpu_slab import BOXES

pytestmark = pytest.mark.gpu


def eval_path(ctx):
    return T.lib().tdgl_internal_eval_path(ctx.ctx)


def _cfg(n, periodic=0, scheme="heun"):
    cfg = I.config("c1")
    cfg.update(n=n, layers=[0] * n[2], scheme=scheme, mimg=1,
               periodic=(int(periodic > 0), int(periodic > 0), int(periodic > 1)))
    return cfg


def _context(cfg, prec, nb):
    return _batch_context(cfg, prec, nb, [250.0 + 100.0 * i / nb for i in range(nb)]) if nb else \
        gpu_context(cfg, prec)


# grid, periodic in plane, instances (0: a single context), path in FP32, in FP64
RULE = [
    ((8, 8, 32), 0, 0, 1, 1), ((8, 8, 33), 0, 0, 0, 0),      # 512 and 528 points, 9 groups
    ((8, 8, 33), 0, 11, 0, 0), ((8, 8, 33), 0, 12, 1, 1),    # mz = 128: 99 and 108 groups
    ((8, 8, 60), 0, 8, 1, 1), ((8, 8, 60), 0, 7, 0, 0),      # multiples of 8: from 64 on
    ((16, 16, 20), 0, 9, 0, 1), ((16, 16, 20), 0, 11, 1, 1),  # 153, 187
    ((16, 16, 20), 0, 8, 1, 1),
    ((20, 30, 11), 0, 8, 1, 1), ((20, 30, 11), 0, 4, 0, 0),  # 200, 100 groups
    ((30, 30, 10), 0, 5, 0, 1), ((30, 30, 10), 0, 6, 1, 1),  # 165, 198
    ((30, 30, 10), 0, 7, 1, 1), ((30, 30, 10), 0, 8, 0, 1),  # 231, 264: more than the CUs
    ((60, 60, 5), 0, 4, 0, 0), ((30, 16, 17), 0, 8, 0, 0),   # 260, 264
    ((30, 30, 17), 0, 6, 0, 0),                              # 1088 points
    ((120, 120, 3), 0, 0, 1, 1), ((60, 128, 3), 0, 0, 0, 0),  # mz = 8: 129 and 65 groups
    ((64, 64, 10), 1, 6, 1, 1), ((64, 64, 10), 1, 0, 0, 0),  # periodic film: 198 and 33
]


@pytest.mark.parametrize("n,periodic,nb,p32,p64", RULE)
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_rule(n, periodic, nb, p32, p64, prec):
    announce("evaluation of %s periodic %d batch %d %s" % (n, periodic, nb, prec))
    ctx = _context(_cfg(n, periodic), prec, nb)
    try:
        path = p32 if prec == "f32" else p64
        assert eval_path(ctx) == path
        assert T.tdgl_get_fft_path(ctx.ctx) == (1 if path else 0)
    finally:
        ctx.close()


@pytest.mark.parametrize("n,used", BOXES + [((32, 8, 3), 0), ((32, 8, 4), 1), ((32, 4, 3), 1),
                                           ((16, 8, 3), 1)])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_rule_of_the_two_kernels(n, used, prec):
    announce("two kernels of %s %s" % (n, prec))
    ctx = gpu_context(_cfg(n), prec)
    try:
        assert (eval_path(ctx) == 2) == bool(used)
    finally:
        ctx.close()
    ctx = gpu_context(_cfg(n), prec, path=1)
    try:
        assert eval_path(ctx) == 0
    finally:
        ctx.close()


# every (my, mz) of planes of 513 to 1024 points: half-filled, ragged and
# periodic y, z half-filled and not; open x of 24 points, which no two kernels take
FULL = [(16, 64), (32, 32), (64, 16), (128, 8)]              # periodic in z as well
PLANES = [(ny, nz, per) for nys, nzs in (((8, 7), (33, 64)), ((16, 13), (17, 32)),
                                        ((32, 31), (9, 16)), ((64, 50), (5, 8)),
                                        ((128, 101), (3, 4)))
          for ny, nz, per in [(nys[0], nzs[0], 0), (nys[1], nzs[1], 0), (2 * nys[0], nzs[0], 1),
                              (2 * nys[0], nzs[1], 1)]] + [(ny, nz, 2) for ny, nz in FULL]


@pytest.mark.parametrize("ny,nz,periodic", PLANES)
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_planes_of_a_batch_have_the_bits_of_three_passes(ny, nz, periodic, prec):
    n, nb = (8 if periodic else 11, ny, nz), 32 if periodic else 16    # 160, 208 groups
    announce("plane bits %s periodic %d %s" % (n, periodic, prec))
    dt = np.float32 if prec == "f32" else np.float64
    cfg = _cfg(n, periodic)
    P = np.stack([I.initial_P(cfg, s, dt) for s in range(nb)])
    ctx = _context(cfg, prec, nb)
    try:
        assert eval_path(ctx) == 1
        ctx.set_P(P)
        field = ctx.eval_field().cpu().numpy()
        ctx.step(5)
        got, F = ctx.get_P(PREC[prec]), ctx.energies_batch()[0]
    finally:
        ctx.close()
    for b in (0, nb - 1):
        one = dict(cfg, T=250.0 + 100.0 * b / nb)
        ctx = gpu_context(one, prec)
        try:
            assert eval_path(ctx) == 0
            ctx.set_P(P[b])
            assert np.array_equal(ctx.eval_field().cpu().numpy(), field[b])
            ctx.step(5)
            assert np.array_equal(ctx.get_P(PREC[prec]), got[b])
            assert np.array_equal(ctx.energies()[0], F[b])
        finally:
            ctx.close()


@pytest.mark.parametrize("n,periodic", [((64, 64, 16), 1), ((32, 32, 8), 0), ((8, 8, 8), 1)])
def test_autotune_keeps_state_and_path_setting(n, periodic):
    announce("autotune of %s" % (n,))
    cfg = _cfg(n, periodic)
    P = I.initial_P(cfg, 1)
    res = []
    for tune in (True, False):
        ctx = gpu_context(cfg, "f64")
        try:
            ctx.set_P(P)
            if tune:
                fused, rows, ms = T.tdgl_autotune(ctx.ctx, 8)
                assert fused == (1 if eval_path(ctx) else 0) and rows >= 2 and ms > 0
                T.tdgl_set_fft_path(ctx.ctx, 0)              # back to the rule
            res.append(eval_path(ctx))
            ctx.step(10)
            res.append(ctx.get_P())
        finally:
            ctx.close()
    assert res[0] == res[2]
    assert np.abs(res[1] - res[3]).max() <= 1e-12 * np.abs(res[3]).max()
