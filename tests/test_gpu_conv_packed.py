"""Every tile of the convolution with packed weights (the network's) and with plain
ones, and the kernel of small grids with both: bit for bit against the oracle on
inputs whose products and sums are exact in FP32, forward and with the mirrored
backward-data weights.  Each case asserts the tile that it is there for."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2605_28800_amd as T  # noqa: E402
from oracle import nn_oracle as N  # noqa: E402
from tests.gpu_helpers import announce  # noqa: E402
from tests.test_gpu_net import (_rng, channels_last, dev_bf16, from_channels_last,  # noqa: E402
                                host_bf16, weights_dev)

# cin, cout, nb, (lz, ly, lx), up2, tile (channel blocks, rows)
CASES = [
    (16, 16, 8, (3, 6, 6), 0, (1, 8)),       # 512 groups
    (5, 16, 7, (3, 6, 6), 1, (1, 2)),        # 448 groups of (1, 8); channels below their padding
    (16, 32, 8, (3, 6, 6), 0, (2, 8)),
    (32, 24, 7, (3, 6, 6), 0, (2, 4)),       # 448 groups of (2, 8)
    (16, 64, 16, (2, 6, 5), 0, (4, 4)),
    (48, 128, 4, (2, 6, 5), 0, (2, 4)),      # 256 groups of (4, 4), 512 of (2, 4)
    (16, 128, 2, (2, 6, 5), 1, (2, 2)),      # 256 groups of (2, 4)
    (128, 32, 1, (2, 1, 4), 0, (2, 2)),      # two rows in all, eight chunks
    (32, 64, 3, (2, 3, 3), 1, (0, 0)),       # rows of 8: the kernel of small grids
    (20, 130, 1, (2, 2, 2), 0, (0, 0)),      # two channel blocks
]


def pow2(n):
    return max(16, 1 << (n - 1).bit_length())


@pytest.mark.parametrize("case", CASES, ids=lambda c: "c%d-%d_nb%d_up%d" % (c[0], c[1], c[2], c[4]))
def test_forward_bit_exact(case):
    cin, cout, nb, (lz, ly, lx), up2, tile = case
    announce("conv tile %s" % (case,))
    cin_p, cout_p = pow2(cin), pow2(cout)
    assert T.lib().tdgl_internal_conv_tile(nb, lx, ly, lz, cin_p, cout_p) == 16 * tile[0] + tile[1]
    rng = _rng(600 + cin + cout + nb)
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
    for packed in (1, 0):
        run(packed, 0, W, b, x, aux, want, case)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "c%d-%d_nb%d_up%d" % (c[0], c[1], c[2], c[4]))
def test_backward_data_bit_exact(case):
    """The same layers from cout to cin channels with the mirrored weights."""
    cin, cout, nb, (lz, ly, lx), _, _ = case
    announce("conv tile %s mirrored" % (case,))
    rng = _rng(700 + cin + cout + nb)
    shape = (1 << lz, 1 << ly, 1 << lx)
    g = rng.integers(-4, 5, size=(nb, cout) + shape) / 4.0
    W = rng.integers(-4, 5, size=(cout, 27, cin)) / 8.0
    aux = rng.integers(-4, 5, size=(nb, cin) + shape) / 4.0
    acc = N.conv3(g, np.ascontiguousarray(W.transpose(2, 1, 0)[:, ::-1]), np.zeros(cin))
    want = {3: (N.round_bf16(acc), None), 4: (N.round_bf16(acc * N.act_slope(aux)), None)}
    run(1, 1, W, np.zeros(cout), g, aux, want, case)


def run(packed, mirror, W, b, x, aux, want, case):
    cin, cout, nb, (lz, ly, lx), up2, _ = case
    up2 = 0 if mirror else up2
    cin_p, cout_p = pow2(cin), pow2(cout)
    nin, nout = (cout_p, cin_p) if mirror else (cin_p, cout_p)
    channels = cin if mirror else cout
    shape = (1 << lz, 1 << ly, 1 << lx)
    npos = nb << (lz + ly + lx)
    din, daux = dev_bf16(channels_last(x, nin)), dev_bf16(channels_last(aux, nout))
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    bias = torch.zeros(cout_p, dtype=torch.float32, device="cuda")
    if packed:
        master = torch.from_numpy(np.concatenate([W.ravel(), b]).astype(np.float32)).cuda()
        w = [torch.full((28 * cin_p * cout_p,), 0x7FC0, dtype=torch.int16, device="cuda")
             for _ in range(2)]
    else:
        dw = weights_dev(W, cin_p, cout_p)
        bias[:cout] = torch.from_numpy(b.astype(np.float32)).cuda()
    from paper_2605_28800_amd import proposal as PR
    for epi, (w1, w2) in want.items():
        out = torch.full((npos, nout), 0x7FC0, dtype=torch.int16, device="cuda")
        out2 = torch.full((npos, nout), 0x7FC0, dtype=torch.int16, device="cuda")
        if packed:
            st = T.lib().tdgl_internal_conv3_packed(
                epi, ptr(din), up2, ptr(master), mirror, cin, cout, nb, lx, ly, lz, cin_p, cout_p,
                ptr(out), ptr(out2), ptr(daux), ptr(w[0]), ptr(w[1]), ptr(bias), stream)
            assert st == T.TDGL_OK
        else:
            PR.nn_conv3(epi, din, dw, bias, nb, lx, ly, lz, cin_p, cout_p, out=out, out2=out2,
                        aux=daux, in_up2=up2)
        torch.cuda.synchronize()
        got = from_channels_last(host_bf16(out), nb, channels, shape)
        np.testing.assert_array_equal(got, w1, err_msg="epilogue %d out" % epi)
        if w2 is not None:
            got2 = from_channels_last(host_bf16(out2), nb, channels, shape)
            np.testing.assert_array_equal(got2, w2, err_msg="epilogue %d out2" % epi)


def test_bias_at_any_float():
    """A bias that starts at any float of an array."""
    announce("conv with a bias at an odd offset")
    rng = _rng(11)
    for cin, cout, nb, (lz, ly, lx) in ((16, 32, 1, (2, 2, 4)), (16, 64, 2, (1, 2, 3))):
        shape = (1 << lz, 1 << ly, 1 << lx)
        x = rng.integers(-4, 5, size=(nb, cin) + shape) / 4.0
        W = rng.integers(-4, 5, size=(cout, 27, cin)) / 8.0
        b = rng.integers(-8, 9, size=cout) / 16.0
        acc = N.conv3(x, W, np.zeros(cout))
        want = N.round_bf16(N.act(acc + b[None, :, None, None, None]))
        from paper_2605_28800_amd import proposal as PR
        for offset in (1, 2, 3):
            store = torch.zeros(cout + 4, dtype=torch.float32, device="cuda")
            bias = store[offset:offset + cout]
            bias.copy_(torch.from_numpy(b.astype(np.float32)))
            out = torch.empty((nb << (lz + ly + lx), cout), dtype=torch.int16, device="cuda")
            PR.nn_conv3(0, dev_bf16(channels_last(x, cin)), weights_dev(W, cin, cout), bias, nb, lx,
                        ly, lz, cin, cout, out=out)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(from_channels_last(host_bf16(out), nb, cout, shape), want)
