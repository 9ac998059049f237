"""The linear-pixel direct convolution over several channel blocks: its pixel buffers and the halves of a block alternate."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu


# N, C, K, H, W: 1 to 6 channel blocks, last ones of 16 to 64 channels, in each of the four forms; the last pixel of the batch
# beside every edge of a workgroup
@pytest.mark.parametrize("C", [64, 112, 192, 208, 320, 336])
@pytest.mark.parametrize("shape", [(1, 24, 9, 11), (5, 72, 51, 1), (7, 64, 60, 61), (9, 130, 61, 60), (17, 200, 33, 61)])
def test_channel_blocks(C, shape):
    N, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=C)
    y = wg.direct_conv2d_int8(torch.from_numpy(wl.to_nhwc(x)).cuda(), torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC)
    assert np.array_equal(wl.from_nhwc(y.cpu().numpy()), oracle.direct_conv2d(x, g))


# sums that go to memory by way of LDS: K whole quads and not, one filter more and less than the lines (64, 33) in a workgroup's first and
# last wave, the last pixel of the batch in the middle of a wave's 32
@pytest.mark.parametrize("K", [32, 33, 60, 64, 65, 97, 124, 128, 161, 196, 257])
@pytest.mark.parametrize("shape", [(1, 16, 3, 7), (2, 32, 37, 41), (17, 16, 59, 60)])
def test_sums_by_way_of_lds(K, shape):
    N, C, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=K)
    y = wg.direct_conv2d_int8(torch.from_numpy(wl.to_nhwc(x)).cuda(), torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC)
    assert np.array_equal(wl.from_nhwc(y.cpu().numpy()), oracle.direct_conv2d(x, g))


# the forms of 512 pixels per workgroup (64 and 128 filters), which take layers of three and more, or two, channel blocks on a full
# chip: filters that end with, before and behind a workgroup's 64 or 128, in whole quads and not, rows short and long, ragged last blocks
@pytest.mark.parametrize("shape", [(6, 144, 65, 72, 76), (17, 144, 129, 21, 61), (11, 144, 200, 22, 68), (16, 208, 191, 22, 62),
                                   (15, 80, 193, 41, 80), (14, 144, 129, 39, 80), (7, 144, 257, 57, 80), (21, 144, 196, 22, 80)])
def test_wide_forms(shape):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=K + W)
    y = wg.direct_conv2d_int8(torch.from_numpy(wl.to_nhwc(x)).cuda(), torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC)
    assert np.array_equal(wl.from_nhwc(y.cpu().numpy()), oracle.direct_conv2d(x, g))
