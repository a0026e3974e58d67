"""RK45 attempts that must not be accepted: an overflowing trial step, whose
error estimate is NaN in every cell, ends the call with TDGL_E_NONFINITE, and so
do 64 rejections in a row; P, the time and the step stay those of the last accepted
step.  A vanishing error over a vanishing tolerance (vacuum cells, absolute
tolerance 0) is no failure."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from tests.gpu_helpers import PREC, announce, gpu_context
from tests.test_gpu_batch import _batch_context

pytestmark = pytest.mark.gpu

# the two-kernel evaluation, the fused plane pass and the three passes
GRIDS = [((16, 16, 8), 0), ((8, 8, 2), 0), ((16, 16, 8), 1), ((20, 20, 8), 0)]


def _cfg(n, dtau):
    cfg = I.config("c1")
    cfg.update(n=n, layers=[0] * n[2], scheme="rk45", dtau=dtau)
    return cfg


@pytest.mark.parametrize("n,path", GRIDS)
@pytest.mark.parametrize("prec,dtau", [("f32", 1e3), ("f32", 1e20), ("f64", 1e3), ("f64", 1e150)])
@pytest.mark.parametrize("nb", [0, 2])
def test_overflowing_trial_step_fails_and_keeps_the_state(n, path, prec, dtau, nb):
    announce("RK45 overflow %s path %d %s dtau %g batch %d" % (n, path, prec, dtau, nb))
    cfg = _cfg(n, dtau)
    dt = np.float32 if prec == "f32" else np.float64
    P = np.stack([I.initial_P(cfg, s, dt) for s in range(max(nb, 1))])
    ctx = _batch_context(cfg, prec, nb, [300.0] * nb, path) if nb else gpu_context(cfg, prec, path=path)
    try:
        ctx.set_P(P if nb else P[0])
        before = ctx.get_P_device().cpu().numpy()
        with pytest.raises(T.TdglError) as e:
            ctx.step(3)
        assert e.value.status == T.TDGL_E_NONFINITE
        assert np.array_equal(ctx.get_P_device().cpu().numpy(), before)
        assert T.tdgl_get_rk_state(ctx.ctx) == (0.0, dtau, 0)
        # the context goes on from there with a step that fits
        T.tdgl_set_integrator(ctx.ctx, T.TDGL_RK45, 1e-3)
        ctx.step(2)
        got = ctx.get_P_device().cpu().numpy()
        ctx.set_P(P if nb else P[0])
        T.tdgl_set_integrator(ctx.ctx, T.TDGL_RK45, 1e-3)
        ctx.step(2)
        assert np.array_equal(ctx.get_P(PREC[prec]), got) and np.isfinite(got).all()
    finally:
        ctx.close()


@pytest.mark.parametrize("n,path", GRIDS)
def test_64_rejections_in_a_row_fail_and_keep_the_state(n, path):
    """Relative tolerance 1e-300: the estimate (about 1e-13 at first, at least
    rounding times h later) stays above it while h shrinks by 0.2 each time."""
    announce("RK45 64 rejections %s path %d" % (n, path))
    cfg = _cfg(n, 1e-3)
    ctx = gpu_context(cfg, "f64", path=path)
    try:
        T.tdgl_set_rk_tolerances(ctx.ctx, 0.0, 1e-300)
        ctx.set_P(I.initial_P(cfg, 0))
        before = ctx.get_P()
        with pytest.raises(T.TdglError) as e:
            ctx.step(1)
        assert e.value.status == T.TDGL_E_NONFINITE
        assert np.array_equal(ctx.get_P(), before)
        tau, h, rejected = T.tdgl_get_rk_state(ctx.ctx)
        assert tau == 0.0 and rejected == 64
        assert h == pytest.approx(1e-3 * 0.2 ** 64, rel=1e-12)
    finally:
        ctx.close()


@pytest.mark.parametrize("n,path", GRIDS)
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_no_error_over_no_tolerance_is_accepted(n, path, prec):
    announce("RK45 vacuum, absolute tolerance 0, %s path %d %s" % (n, path, prec))
    cfg = _cfg(n, 1e-3)
    cfg["layers"][-1] = -1
    ctx = gpu_context(cfg, prec, path=path)
    try:
        T.tdgl_set_rk_tolerances(ctx.ctx, 0.0, 1e-3)
        ctx.set_P(I.initial_P(cfg, 0, np.float32 if prec == "f32" else np.float64))
        ctx.step(3)
        got = ctx.get_P()
        assert np.isfinite(got).all() and (got[:, -1] == 0).all()
        assert T.tdgl_get_rk_state(ctx.ctx)[0] > 0.0
    finally:
        ctx.close()
