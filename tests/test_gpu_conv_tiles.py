"""The tiled convolution at every tile its launcher chooses (channel blocks of 16
to 128 on grids small and large enough for each), bit for bit against the
oracle on inputs whose products and sums are exact in FP32, through the
single-layer entry point (plain weights); and the packed weights of a wide
network, all of whose levels take the tiled kernel, through its forward pass."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import tdgl_inputs as I  # noqa: E402
from oracle import nn_oracle as N  # noqa: E402
from tests.gpu_helpers import announce  # noqa: E402
from tests.test_gpu_net import (_rng, channels_last, dev_bf16, from_channels_last,  # noqa: E402
                                host_bf16, weights_dev)

# cin, cout, nb, (lz, ly, lx), up2: tiles of (channel blocks, rows) per wave
CASES = [
    (16, 16, 8, (3, 6, 6), 0),       # (1, 8): 512 groups
    (16, 32, 8, (3, 6, 6), 0),       # (2, 8)
    (32, 32, 2, (3, 5, 6), 1),       # (2, 2): 256 groups
    (16, 64, 16, (2, 6, 5), 0),      # (4, 4): 512 groups
    (16, 128, 2, (2, 6, 5), 0),      # (2, 4)
    (48, 16, 1, (2, 1, 4), 0),       # (1, 2): two rows in all, three chunks padded to four
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "c%d-%d_nb%d_up%d" % (c[0], c[1], c[2], c[4]))
def test_tiles_bit_exact(case):
    cin, cout, nb, (lz, ly, lx), up2 = case
    announce("conv tile %s" % (case,))
    cin_p = 1 << (cin - 1).bit_length()
    rng = _rng(300 + cin + cout + nb)
    shape = (1 << lz, 1 << ly, 1 << lx)
    in_shape = tuple(s // 2 for s in shape) if up2 else shape
    x = rng.integers(-4, 5, size=(nb, cin) + in_shape) / 4.0
    W = rng.integers(-4, 5, size=(cout, 27, cin)) / 8.0
    b = rng.integers(-8, 9, size=cout) / 16.0
    aux = rng.integers(-4, 5, size=(nb, cout) + shape) / 4.0
    acc = N.conv3(N.up(x) if up2 else x, W, np.zeros(cout))
    t = N.round_bf16(N.act(acc + b[None, :, None, None, None]))
    want = {0: (t, None), 1: (t, N.round_bf16(t + aux)),
            5: (N.round_bf16(acc), N.round_bf16(acc * N.act_slope(aux)))}
    from paper_2605_28800_amd import proposal as PR
    npos = nb * shape[0] * shape[1] * shape[2]
    din, dw = dev_bf16(channels_last(x, cin_p)), weights_dev(W, cin_p, cout)
    bias = torch.from_numpy(b.astype(np.float32)).cuda()
    daux = dev_bf16(channels_last(aux, cout))
    for epi, (w1, w2) in want.items():
        out = torch.full((npos, cout), 0x7FC0, dtype=torch.int16, device="cuda")
        out2 = torch.full((npos, cout), 0x7FC0, dtype=torch.int16, device="cuda")
        PR.nn_conv3(epi, din, dw, bias, nb, lx, ly, lz, cin_p, cout, out=out, out2=out2,
                    aux=daux, in_up2=up2)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(from_channels_last(host_bf16(out), nb, cout, shape), w1)
        if w2 is not None:
            np.testing.assert_array_equal(from_channels_last(host_bf16(out2), nb, cout, shape), w2)


def test_packed_weights_of_a_wide_network():
    """Width 64 (channel counts 64 to 256, all levels on the tiled kernel):
    the forward pass within the relative L2 that BF16 rounding flips of twelve
    layers allow, 5e-3 as the smaller networks' smoke check; a misplaced weight
    fragment moves the output by its own size."""
    from paper_2605_28800_amd.proposal import Net
    shape, width = (16, 16, 64), 64
    announce("packed weights, width %d" % width)
    T, th, noise = I.net_conditions(1, shape, 8, seed=2, thickness_range=(9, 16))
    theta = I.net_params(width, seed=2)
    net = Net(shape, width=width, noise_div=8, max_batch=1)
    try:
        net.set_params(theta)
        P = net.forward(*[torch.from_numpy(a).cuda() for a in (T, th, noise)]).cpu().numpy()
    finally:
        net.close()
    ref, _ = N.forward(theta.astype(np.float64), width, T, th, noise, shape, bf16=True)
    assert np.linalg.norm(P - ref) / np.linalg.norm(ref) <= 5e-3
