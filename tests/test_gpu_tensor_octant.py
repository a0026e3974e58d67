"""The device-built tensor spectrum where its octant evaluation can go wrong:
cells that are not cubes (the rule's order follows the longest edge), offsets
on both sides of the entries that a whole wave shares, mirror images of odd
and even sizes, and lattice images on the window's edge (periodic dimensions,
several image counts).  Reference: the oracle's table by its own quadrature
(two half-interval Gauss-Legendre rules), transformed with numpy; tolerance
1e-13 of the largest entry, FP64 on both sides, as for the 40-digit tables."""
import numpy as np
import pytest

import paper_2605_28800_amd as T
import tdgl_inputs as I
from oracle import tdgl_oracle as O
from tests.gpu_helpers import announce, gpu_context, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,periodic,mimg", [
    ((20, 5, 3), (1.0, 1.5, 0.7), (0, 0, 0), 0),      # flat cells, one image per offset
    ((3, 17, 9), (2.0, 0.5, 1.0), (0, 0, 0), 0),
    ((1, 1, 1), (1.0, 1.0, 1.0), (0, 0, 0), 0),       # the origin alone
    ((8, 16, 3), (1.0, 0.8, 1.3), (1, 1, 0), 0),      # half windows around each cell
    ((16, 8, 5), (1.0, 1.0, 1.0), (1, 1, 0), 5),      # 144 images: more than one per lane
    ((8, 8, 8), (1.0, 1.2, 0.9), (1, 1, 1), 1),
])
def test_octant_spectrum(n, d, periodic, mimg):
    cfg = I.config("c1")
    cfg.update(n=n, d=tuple(v * 1e-9 for v in d), periodic=periodic, mimg=mimg,
               layers=[0] * n[2], tensor_source="quadrature")
    announce("tensor octant %s cells %s periodic %s mimg %d" % (n, d, periodic, mimg))
    prob = O.Problem(cfg)
    ctx = gpu_context(cfg, "f64")
    try:
        got = T.tdgl_get_tensor_spectrum(ctx.ctx)
        nx, ny, nz, mx, my, mz, hx = ctx.dims
    finally:
        ctx.close()
    kern = np.zeros((6, mz, my, mx))
    at = []
    for size, M, p in ((nz, mz, periodic[2]), (ny, my, periodic[1]), (nx, mx, periodic[0])):
        i = np.arange(size if p else 2 * size - 1)
        at.append(i if p else (i - (size - 1)) % M)
    kern[:, at[0][:, None, None], at[1][None, :, None], at[2][None, None, :]] = prob.tab
    spec = np.fft.rfftn(kern, axes=(1, 2, 3)).real
    ref = -prob.kappa / (mx * my * mz) * spec[:, :mz // 2 + 1, :my // 2 + 1, :]
    assert rel_inf(got, ref) <= 1e-13
