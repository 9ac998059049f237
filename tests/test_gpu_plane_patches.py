"""Channel-major activations read as they are (patches turned on their way into LDS): the limb-pair kernel, forced through the
test hook, and the kernels of split channels, as the library picks them.  Bit for bit against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


SHAPES = [  # N, C, K, H, W
    (1, 8, 5, 1, 1),        # eight bytes: one load, moved for every channel but the first
    (1, 7, 5, 1, 1),        # fewer: the other kernels
    (1, 3, 4, 2, 3),        # rows shorter than a patch
    (1, 4, 1, 1, 9),        # the tensor's last row ends inside a load
    (2, 5, 33, 5, 2),
    (1, 16, 16, 16, 16),
    (3, 21, 40, 7, 13),     # odd channels, rows at any alignment, tiles of three images in a block
    (1, 64, 96, 8, 20),
    (1, 65, 32, 9, 6),      # a second block of one channel
    (2, 130, 36, 10, 12),   # three blocks
    (1, 16, 72, 131, 67),   # more workgroups than compute units
]


@pytest.mark.parametrize("shape", SHAPES)
def test_limb_pair_kernel(shape):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, seed=5)
    x[0, 0], g[0] = -128, -128
    want = oracle.direct_conv2d(x, g)
    packed = wg.winograd_filter_transform(_dev(g), wg.NCHW, wg.LOSSLESS)
    wg.lossless_variant(1)
    try:
        y = wg.winograd_conv2d_int8(_dev(x), packed, wg.NCHW)
        got = [(False, False, wg.winograd_conv2d_int8_requant(_dev(x), packed, 9, False, False, wg.NCHW))]
        if H % 2 == 0 and W % 2 == 0:
            got.append((True, True, wg.winograd_conv2d_int8_requant(_dev(x), packed, 9, True, True, wg.NCHW)))
    finally:
        wg.lossless_variant(0)
    assert np.array_equal(y.cpu().numpy(), want)
    for relu, pool, q in got:
        assert np.array_equal(q.cpu().numpy(), oracle.requant_relu_pool(want, 9, relu, pool))


@pytest.mark.parametrize("mode", ["lossless", "scaled"])
@pytest.mark.parametrize("shape", [(1, 256, 16, 10, 10), (1, 200, 40, 9, 7), (1, 512, 64, 14, 14)])
def test_split_channels(shape, mode):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="relu", wgt="gauss", seed=6)
    want = oracle.direct_conv2d(x, g) if mode == "lossless" else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(_dev(g), wg.NCHW, wg.LOSSLESS if mode == "lossless" else wg.SCALED)
    assert np.array_equal(wg.winograd_conv2d_int8(_dev(x), packed, wg.NCHW).cpu().numpy(), want)
    q = wg.winograd_conv2d_int8_requant(_dev(x), packed, 11, True, False, wg.NCHW)
    assert np.array_equal(q.cpu().numpy(), oracle.requant_relu_pool(want, 11, True, False))
