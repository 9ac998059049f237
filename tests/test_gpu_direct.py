"""The direct convolution's kernels and the requantisation kernels at the edges of their tiles, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, C, K, H, W: each form of the linear-pixel kernel (128 x 512, 64 x 512, 64 x 256, 64 x 128 filters x pixels), pixel counts at
# and next to a multiple of a workgroup's, several channel blocks with a partial last one, one-pixel images, rows too long
# for its LDS
SHAPES = [(1, 16, 64, 16, 32), (1, 64, 65, 1, 129), (3, 80, 130, 7, 7), (130, 16, 8, 1, 1), (4, 130, 64, 33, 31),
          (2, 16, 257, 91, 113), (8, 64, 192, 56, 56), (33, 48, 640, 28, 28), (1, 20, 36, 3, 700), (1, 5, 3, 2, 600),
          # rows too long: the patch kernel with 16-byte loads (C % 16 = 0, K % 4 = 0), a partial last block, two filter blocks
          (1, 32, 36, 3, 700), (2, 80, 68, 9, 650)]


@pytest.mark.parametrize("layout", [wg.NCHW, wg.NHWC])
@pytest.mark.parametrize("shape", SHAPES)
def test_direct_convolution(shape, layout):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=3)
    nhwc = layout == wg.NHWC
    y = wg.direct_conv2d_int8(torch.from_numpy(wl.to_nhwc(x) if nhwc else x).cuda(), torch.from_numpy(wl.to_krsc(g) if nhwc else g).cuda(), layout)
    got = y.cpu().numpy()
    assert np.array_equal(wl.from_nhwc(got) if nhwc else got, oracle.direct_conv2d(x, g))


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("layout", [wg.NCHW, wg.NHWC])
@pytest.mark.parametrize("shape", [(2, 64, 8, 16), (1, 6, 4, 10), (3, 7, 2, 2), (1, 4, 6, 24), (1, 1, 2, 2)])
def test_requantisation_of_any_int32(shape, layout, pool):
    N, K, H, W = shape
    rng = np.random.default_rng(7)
    y = rng.integers(-2 ** 31, 2 ** 31, (N, K, H, W), dtype=np.int64).astype(np.int32)
    y[0, 0, 0, :2] = (2 ** 31 - 1, -2 ** 31)
    nhwc = layout == wg.NHWC
    yd = torch.from_numpy(wl.to_nhwc(y) if nhwc else y).cuda()
    for shift in (0, 1, 24, 31):
        got = wg.requant_relu_pool_int8(yd, shift, False, pool, layout).cpu().numpy()
        v = (y.astype(np.int64) + (1 << shift >> 1)) >> shift
        v = np.clip(v, -128, 127)
        if pool:
            v = v.reshape(N, K, H // 2, 2, W // 2, 2).max(axis=(3, 5))
        assert np.array_equal(wl.from_nhwc(got) if nhwc else got, v.astype(np.int8))


# N, C, K, H, W: deep layers of few pixels
@pytest.mark.parametrize("shape", [(96, 128, 128, 8, 16), (97, 128, 128, 8, 16), (16, 176, 36, 19, 50), (104, 256, 256, 7, 16), (105, 256, 200, 8, 15),
                                   (1, 496, 68, 13, 21), (5, 256, 4, 1, 1)])
def test_few_patches_of_deep_layers(shape):
    """Both layouts run the linear-pixel kernel, channel-major through copies of both operands: the two against each other, and the
    first and the last image against the oracle."""
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=4)
    got = wg.direct_conv2d_int8(torch.from_numpy(wl.to_nhwc(x)).cuda(), torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC)
    other = wg.direct_conv2d_int8(torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda(), wg.NCHW)
    assert torch.equal(got.permute(0, 3, 1, 2), other)
    for n in {0, N - 1}:
        assert np.array_equal(other[n:n + 1].cpu().numpy(), oracle.direct_conv2d(x[n:n + 1], g))
