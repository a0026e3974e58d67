"""Device workspace a context asks for: no larger than what callers that kept the
number once got, per scheme, so that a buffer of that size is still accepted."""
import pytest

import paper_2605_28800_amd as T

# grid, periodic mask, precision, instances: bytes for Heun, AB3M2, RK45
SIZES = [
    ((16, 16, 8), 0, T.TDGL_FP64, 1, (776448, 923904, 1169664)),
    ((16, 16, 8), 0, T.TDGL_FP32, 1, (444672, 518400, 641280)),
    ((128, 128, 32), 3, T.TDGL_FP32, 1, (35985664, 54860032, 86317312)),
    ((128, 128, 32), 3, T.TDGL_FP64, 1, (71731456, 109480192, 172394752)),
    ((32, 32, 32), 0, T.TDGL_FP32, 24, (93887232, 122198784, 169384704)),
    ((5, 4, 3), 0, T.TDGL_FP64, 300, (7867904, 9164032, 11323904)),
    ((16, 16, 8), 0, T.TDGL_FP32, 4096, (1075856896, 1377846784, 1881163264)),
]


@pytest.mark.parametrize("n,pm,prec,nb,sizes", SIZES)
def test_workspace_is_no_larger(n, pm, prec, nb, sizes):
    ctx = T.tdgl_create_batch(T.tdgl_grid(*n, 1e-9, 1e-9, 1e-9, pm), nb, prec)
    try:
        for scheme, most in zip((T.TDGL_HEUN, T.TDGL_AB3M2, T.TDGL_RK45), sizes):
            T.tdgl_set_integrator(ctx, scheme, 1e-3)
            assert T.tdgl_workspace_size(ctx) <= most
            T.tdgl_bind_workspace(ctx, 1 << 20, most)      # an address, never read here
    finally:
        T.tdgl_destroy(ctx)
