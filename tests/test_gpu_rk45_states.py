"""RK45 attempts launched plainly and as graphs (the first eight of a context are
plain): a batch of equal instances takes the attempts of a single context (one
error, one step size) and gives its bits, with rejections inside the run,
split calls and a graph cache that is dropped between them.  And one decision
of the controller, in both precisions and evaluations, to what their rounding
allows."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from tests.gpu_helpers import PREC, announce, gpu_context
from tests.test_gpu_batch import _batch_context

pytestmark = pytest.mark.gpu


def _cfg(n, terms=15, dtau=5e-3):
    cfg = I.config("c1")
    cfg.update(n=n, layers=[0] * n[2], scheme="rk45", dtau=dtau, terms=terms)
    return cfg


def _run(ctx, P, parts, chunk):
    T.tdgl_set_graph_chunk(ctx.ctx, chunk)
    T.tdgl_set_rk_tolerances(ctx.ctx, 1e-9, 1e-7)
    ctx.set_P(P)
    for i, k in enumerate(parts):
        if i == 1:
            T.tdgl_set_update_rows(ctx.ctx, 0)       # drops the captured graphs
        ctx.step(k)
    F = ctx.energies_batch()[0]
    ctx.step(2)
    return ctx.get_P(), F, T.tdgl_get_rk_state(ctx.ctx)


@pytest.mark.parametrize("n,nb,terms", [((32, 32, 16), 20, 15), ((30, 30, 20), 9, 15),
                                        ((32, 32, 16), 9, 11)])
@pytest.mark.parametrize("parts,chunk", [((12,), 64), ((5, 1, 6), 64), ((10, 2), 64), ((12,), 0)])
def test_equal_instances_take_the_attempts_of_one(n, nb, terms, parts, chunk):
    announce("RK45 of %d x %s, terms %d, calls %s, graphs %d" % (nb, n, terms, parts, chunk))
    cfg = _cfg(n, terms)
    P = I.initial_P(cfg, 4)
    one = gpu_context(cfg, "f64")
    try:
        want, F1, rk1 = _run(one, P, (12,), 0)
    finally:
        one.close()
    many = _batch_context(cfg, "f64", nb, [300.0] * nb)
    try:
        got, F, rk = _run(many, np.stack([P] * nb), parts, chunk)
    finally:
        many.close()
    assert rk1[2] > 0 and rk[1:] == rk1[1:]
    assert abs(rk[0] - rk1[0]) <= 14 * 2.0 ** -53 * rk1[0]           # summed per call
    for b in (0, nb // 2, nb - 1):
        assert np.array_equal(got[b], want) and np.array_equal(F[b], F1[0])


@pytest.mark.parametrize("n", [(16, 16, 8), (8, 16, 16), (31, 29, 11)])
@pytest.mark.parametrize("prec,path", [("f32", 0), ("f32", 1), ("f64", 0), ("f64", 1)])
def test_first_decision_follows_the_error(n, prec, path):
    """One step from one state: the next step size is h times 0.9 err^-1/5.  The
    estimate h sum e_j k_j is a sum of seven products of at most max |k|, so it is
    off by at most 8 roundings of h max |k| sum |e_j| (0.18) and by what the field's
    own error (2e-6 / 1e-13 of its largest value) puts into the k_j, 0.18 h max |k|
    times that; over the tolerance, relative to err, and a fifth of it in h."""
    announce("RK45 first decision %s %s path %d" % (n, prec, path))
    cfg = _cfg(n)
    P = I.initial_P(cfg, 6).astype(np.float32).astype(np.float64)
    res = []
    for pr, pa in ((prec, path), ("f64", 1)):
        ctx = gpu_context(cfg, pr, path=pa)
        try:
            T.tdgl_set_rk_tolerances(ctx.ctx, 1e-3, 0.0)
            ctx.set_P(P.astype(np.float32) if pr == "f32" else P)
            rate = np.abs(ctx.eval_field().cpu().numpy()).max() / cfg["scales"]["alpha_ref"]
            ctx.step(1)
            res.append((T.tdgl_get_rk_state(ctx.ctx), ctx.get_P(PREC[pr]).astype(np.float64), rate))
        finally:
            ctx.close()
    (tau, h, rej), got, _ = res[0]
    (tau1, h1, rej1), want, rate = res[1]
    assert (tau, rej) == (tau1, rej1) == (5e-3, 0)
    err = (0.9 * 5e-3 / h1) ** 5                              # of the reference, over 1e-3
    assert 1e-3 < err <= 1.0 and 0.2 < h1 / 5e-3 < 5.0        # no clamp in the way
    eps, field = (2.0 ** -24, 2e-6) if prec == "f32" else (2.0 ** -53, 1e-13)
    off = 5e-3 * 2 * rate * 0.18 * (8 * eps + field) / (1e-3 * err)
    assert abs(h / h1 - 1) <= off / 5 + 1e-12
    assert np.abs(got - want).max() <= (1e-5 if prec == "f32" else 1e-12) * np.abs(want).max()


@pytest.mark.parametrize("n", [(9, 7, 5), (8, 7, 5), (1, 1, 1)])
@pytest.mark.parametrize("nb", [0, 3])
def test_odd_numbers_of_floats(n, nb):
    """The second state buffer starts behind 3 * cells floats: on a single word
    where that is odd.  Accepted states are copied whole: calls of one step (a
    fresh look at P each) and one call of all give the same bits."""
    announce("RK45 FP32 of %s, batch %d" % (n, nb))
    cfg = _cfg(n)
    P = np.stack([I.initial_P(cfg, s, np.float32) for s in range(max(nb, 1))])
    got = []
    for parts in ((9,), (1,) * 9):
        ctx = _batch_context(cfg, "f32", nb, [300.0] * nb) if nb else gpu_context(cfg, "f32")
        try:
            ctx.set_P(P if nb else P[0])
            for k in parts:
                ctx.step(k)
            got.append(ctx.get_P(PREC["f32"]))
        finally:
            ctx.close()
    assert np.array_equal(got[0], got[1]) and np.isfinite(got[0]).all()
    assert (got[0].reshape(P.shape) != P).any(axis=(1, 2, 3, 4)).all()
