"""The two-kernel evaluation of small open boxes against the oracle, at the edges
of its rule: the smallest and the largest box of each transform length, odd
sizes, z lines that nearly or just fill a third of their length, vacuum and
a second material.  Field 1e-13 / 2e-6 of its norm, energies 1e-12 / 2e-6
of their scale, 20 steps |dP| 1e-12 / 1e-5 of the state's norm (the bounds of
the other paths); instances of a batch have the bits of single contexts."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from oracle import tdgl_oracle as O
from tests.gpu_helpers import announce, gpu_context, oracle_field, rel_inf
from tests.test_gpu_batch import _batch_context
from tests.test_gpu_parity import MASKS, _cfg

pytestmark = pytest.mark.gpu

#        n, in use
BOXES = [((8, 4, 3), 1), ((7, 8, 14), 1), ((32, 7, 4), 1), ((5, 13, 7), 1), ((8, 16, 16), 1),
         ((16, 15, 8), 1), ((13, 31, 22), 1), ((15, 32, 32), 1), ((31, 29, 11), 1),
         ((62, 32, 8), 1), ((32, 16, 8), 0), ((16, 30, 6), 0), ((33, 31, 8), 0), ((8, 8, 33), 0)]


def _make(n, layers):
    if layers == "one":
        return _cfg(n, (0, 0, 0))
    lay = [0] * n[2]
    lay[-1], lay[n[2] // 2] = -1, 1
    return _cfg(n, (0, 0, 0), layers=lay, two_materials=True)


@pytest.mark.parametrize("n,used", BOXES)
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("layers", ["one", "vacuum"])
def test_slab_field_and_energies(n, used, prec, layers):
    cfg = _make(n, layers)
    announce("slab field %s %s %s" % (n, prec, layers))
    P = I.initial_P(cfg, 3, np.float32 if prec == "f32" else np.float64)
    P64 = P.astype(np.float64)
    prob = O.Problem(cfg)
    ctx = gpu_context(cfg, prec)
    try:
        ctx.set_P(P)
        assert T.tdgl_get_fft_path(ctx.ctx) == 1 or not used
        tol = 1e-13 if prec == "f64" else 2e-6
        for mask in MASKS:
            err = rel_inf(ctx.eval_field(mask).cpu().numpy(), oracle_field(P64, prob, mask))
            assert err <= tol, (mask, err)
        F, m = ctx.energies()
    finally:
        ctx.close()
    ref = gpu_context(cfg, prec, path=1)
    try:
        ref.set_P(P)
        F1, m1 = ref.energies()
    finally:
        ref.close()
    tol = 1e-12 if prec == "f64" else 2e-6
    assert rel_inf(F, F1) <= tol and rel_inf(m, m1) <= 1e-12


@pytest.mark.parametrize("n", [b[0] for b in BOXES if b[1]])
@pytest.mark.parametrize("scheme", ["euler", "heun", "ab3m2", "rk45"])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_slab_steps(n, scheme, prec):
    cfg = _make(n, "vacuum")
    cfg.update(scheme=scheme, T=300.0)
    announce("slab steps %s %s %s" % (n, scheme, prec))
    dt = np.float32 if prec == "f32" else np.float64
    P = np.stack([I.initial_P(cfg, s, dt) for s in range(3)])
    res, rk = [], []
    for path in (0, 1):
        ctx = gpu_context(cfg, prec, path=path)
        try:
            if scheme == "rk45":
                T.tdgl_set_rk_tolerances(ctx.ctx, 1e-7, 1e-5)
            ctx.set_P(P[1])
            ctx.step(13)
            ctx.step(7)
            res.append((ctx.get_P(), np.array(ctx.energies()[0])))
            if scheme == "rk45":
                rk.append(T.tdgl_get_rk_state(ctx.ctx)[0])
                rate = np.abs(ctx.eval_field().cpu().numpy()).max() / cfg["scales"]["alpha_ref"]
        finally:
            ctx.close()
    tol = 1e-12 if prec == "f64" else 1e-5
    if scheme == "rk45":                  # its steps follow the rounding: other end times
        tol += abs(rk[0] - rk[1]) * rate / np.abs(res[1][0]).max()
        assert abs(rk[0] - rk[1]) <= (1e-9 if prec == "f64" else 1e-2) * rk[1]
    assert rel_inf(res[0][0], res[1][0]) <= tol
    if scheme == "rk45":                  # one step size for the whole batch
        return
    ctx = _batch_context(cfg, prec, 3, [300.0] * 3)
    try:
        ctx.set_P(P)
        ctx.step(20)
        assert np.array_equal(ctx.get_P()[1], res[0][0])
        assert np.array_equal(ctx.energies_batch()[0][1], res[0][1])
    finally:
        ctx.close()


def test_slab_path_switch_keeps_state():
    """A switch of the path between steps remakes the spectra."""
    cfg = _make((12, 14, 8), "one")
    cfg.update(scheme="heun")
    announce("slab path switch")
    P = I.initial_P(cfg, 5)
    ctx = gpu_context(cfg, "f64")
    try:
        ctx.set_P(P)
        for path in (0, 1, 0, 1):
            T.tdgl_set_fft_path(ctx.ctx, path)
            ctx.step(5)
        got = ctx.get_P()
    finally:
        ctx.close()
    ref = gpu_context(cfg, "f64", path=1)
    try:
        ref.set_P(P)
        ref.step(20)
        assert rel_inf(got, ref.get_P()) <= 1e-12
    finally:
        ref.close()
