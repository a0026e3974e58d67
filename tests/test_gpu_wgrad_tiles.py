"""The tiled weight gradient at each of its channel blocks and tile heights, bit
for bit against the oracle on inputs whose products and sums are exact in
FP32: grids of one tile, halos at every face, the 2x repeated input, one to
many tiles per split, channels beyond one block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import nn_oracle as N  # noqa: E402
from tests.gpu_helpers import announce  # noqa: E402
from tests.test_gpu_net import _rng, channels_last, dev_bf16  # noqa: E402

# cin_p, cout_p, nb, (lz, ly, lx), up2
CASES = [
    (16, 16, 1, (0, 3, 3), 0),       # one 1 x 8 x 8 tile
    (32, 16, 3, (1, 3, 4), 0),       # two-plane tiles, blocks (1, 2)
    (16, 32, 2, (2, 4, 3), 1),       # blocks (2, 1), repeated input
    (64, 32, 1, (3, 3, 3), 0),       # blocks (2, 2), two tiles in z
    (32, 64, 2, (2, 3, 4), 1),       # blocks (4, 1)
    (64, 128, 1, (1, 4, 3), 0),      # several blocks each way
    (16, 16, 600, (2, 3, 3), 0),     # more tiles than splits: a ragged last split
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "c%d-%d_nb%d_lz%d_up%d" % (c[0], c[1], c[2], c[3][0], c[4]))
def test_weight_gradient_tiles_bit_exact(case):
    cin, cout, nb, (lz, ly, lx), up2 = case
    announce("wgrad tile %s" % (case,))
    rng = _rng(400 + cin + cout + nb)
    shape = (1 << lz, 1 << ly, 1 << lx)
    in_shape = tuple(s // 2 for s in shape) if up2 else shape
    # products are multiples of 1/16 of at most 1; sums of 153,600 stay below 2^24 of them
    x = rng.integers(-4, 5, size=(nb, cin) + in_shape) / 4.0
    g = rng.integers(-4, 5, size=(nb, cout) + shape) / 4.0
    gW, gb = N.conv3_weight_grad(g, N.up(x) if up2 else x)
    from paper_2605_28800_amd import proposal as PR
    grad = PR.nn_conv3_wgrad(dev_bf16(channels_last(g, cout)), dev_bf16(channels_last(x, cin)),
                             nb, lx, ly, lz, cin, cout, in_up2=up2)
    torch.cuda.synchronize()
    grad = grad.cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(grad[:cout * 27 * cin].reshape(cout, 27, cin), gW)
    np.testing.assert_array_equal(grad[cout * 27 * cin:], gb)
