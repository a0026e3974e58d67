"""The tiled weight gradient at each of its channel blocks, on both sides of the
256 groups below which it takes blocks of 16 x 16 channels, and in a workspace of
fewer splits than it asks for: bit for bit against the oracle on inputs whose
products and sums are exact in FP32."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2605_28800_amd as T  # noqa: E402
from oracle import nn_oracle as N  # noqa: E402
from tests.gpu_helpers import announce  # noqa: E402
from tests.test_gpu_net import _rng, channels_last, dev_bf16  # noqa: E402

# cin_p, cout_p, nb, (lz, ly, lx), up2
CASES = [
    (16, 16, 256, (0, 3, 3), 0), (16, 16, 255, (0, 3, 3), 0),     # (1, 1)
    (32, 16, 256, (0, 3, 3), 0), (32, 16, 255, (0, 3, 3), 0),     # (1, 2), (1, 1)
    (16, 32, 64, (1, 3, 5), 1), (16, 32, 63, (1, 3, 5), 1),       # (2, 1), repeated input
    (64, 32, 128, (2, 3, 3), 0), (64, 32, 127, (2, 3, 3), 0),     # (2, 2)
    (32, 64, 32, (3, 3, 4), 0), (32, 64, 31, (3, 3, 4), 0),       # (4, 1)
    (64, 128, 32, (2, 3, 3), 0), (64, 128, 31, (2, 3, 3), 0),     # several blocks each way
    (64, 64, 1, (2, 4, 4), 0),
]


def data(case):
    cin, cout, nb, (lz, ly, lx), up2 = case
    rng = _rng(500 + cin + cout + nb)
    shape = (1 << lz, 1 << ly, 1 << lx)
    in_shape = tuple(s // 2 for s in shape) if up2 else shape
    # products are multiples of 1/16 of at most 1; sums stay below 2^24 of them
    x = rng.integers(-4, 5, size=(nb, cin) + in_shape) / 4.0
    g = rng.integers(-4, 5, size=(nb, cout) + shape) / 4.0
    return x, g, N.conv3_weight_grad(g, N.up(x) if up2 else x)


def check(grad, cin, cout, want):
    grad = grad.cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(grad[:cout * 27 * cin].reshape(cout, 27, cin), want[0])
    np.testing.assert_array_equal(grad[cout * 27 * cin:], want[1])


def ident(c):
    return "c%d-%d_nb%d_lz%d_up%d" % (c[0], c[1], c[2], c[3][0], c[4])


@pytest.mark.parametrize("case", CASES, ids=ident)
def test_channel_blocks_bit_exact(case):
    cin, cout, nb, (lz, ly, lx), up2 = case
    announce("wgrad blocks %s" % (case,))
    x, g, want = data(case)
    from paper_2605_28800_amd import proposal as PR
    grad = PR.nn_conv3_wgrad(dev_bf16(channels_last(g, cout)), dev_bf16(channels_last(x, cin)),
                             nb, lx, ly, lz, cin, cout, in_up2=up2)
    torch.cuda.synchronize()
    check(grad, cin, cout, want)


@pytest.mark.parametrize("case", [(32, 64, 32, (3, 3, 4), 0), (16, 16, 256, (0, 3, 3), 0),
                                  (64, 64, 4, (2, 4, 4), 0), (16, 32, 64, (1, 3, 5), 1)], ids=ident)
def test_smaller_workspace_is_taken_with_fewer_splits(case):
    cin, cout, nb, (lz, ly, lx), up2 = case
    announce("wgrad workspace %s" % (case,))
    x, g, want = data(case)
    dg, dx = dev_bf16(channels_last(g, cout)), dev_bf16(channels_last(x, cin))
    full = ctypes.c_size_t()
    assert T.lib().tdgl_nn_wgrad_workspace(nb, lx, ly, lz, cin, cout, ctypes.byref(full)) == T.TDGL_OK
    split = 4 * cout * (27 * cin + 1)
    npos = nb << (lz + ly + lx)
    small = min(-(-1024 // -(-27 * cin // 64)), -(-npos // 256))     # splits of the other kernel
    chunk = -(-(-(-npos // small)) // 128) * 128
    least = min(-(-npos // chunk), full.value // split)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    for splits in sorted({least, (least + full.value // split) // 2, full.value // split}):
        guard = 1024
        ws = torch.full((splits * split // 4 + guard,), 7.0, dtype=torch.float32, device="cuda")
        grad = torch.empty(cout * 27 * cin + cout, dtype=torch.float32, device="cuda")
        call = lambda nbytes: T.lib().tdgl_nn_conv3_wgrad(
            ptr(dg), ptr(dx), up2, nb, lx, ly, lz, cin, cout, ptr(ws), ctypes.c_size_t(nbytes),
            ptr(grad), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert call(splits * split) == T.TDGL_OK
        torch.cuda.synchronize()
        check(grad, cin, cout, want)
        assert (ws[-guard:] == 7.0).all()
        if splits == least:
            assert call(splits * split - 1) == T.TDGL_E_ARG
