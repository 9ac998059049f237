"""GPU parity of the streaming kernel with eight product waves of 8 filters each (limb-pair operand; lossless mode, one channel block),
forced through the test hooks on small shapes: bit for bit against the oracle's direct convolution."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu

ZX, ZW, SHIFT = 255, 0, 9


@pytest.fixture(autouse=True)
def pairs():
    wg.stream_variant(4)
    wg.scaled_variant(2)
    yield
    wg.stream_variant(0)
    wg.scaled_variant(0)
    wg.stream_workgroups(0)


def _in(a, layout, transposed):
    return torch.from_numpy(np.ascontiguousarray(transposed(a) if layout == wg.NHWC else a)).cuda()


def _nchw(t, layout):
    a = t.cpu().numpy()
    return wl.from_nhwc(a) if layout == wg.NHWC else a


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("shape,workgroups", [
    ((1, 16, 64, 4, 4), 1),        # one tile
    ((2, 64, 64, 8, 32), 1),       # two full tile blocks, one after the other in one workgroup
    ((3, 64, 40, 18, 22), 3),      # ragged tiles, a last tile block that is not full, filters beyond K
    ((3, 20, 97, 9, 13), 2),       # odd everything: bytes stored one by one, a copy in channel-major layout
    ((1, 33, 130, 20, 36), 4),     # three filter blocks, the last with two filters; channels that are no multiple of four
])
def test_equals_the_oracle(shape, workgroups, layout):
    N, C, K, H, W = shape
    rng = np.random.default_rng(31)
    xb, gb = rng.integers(0, 256, (N, C, H, W), dtype=np.uint8), rng.integers(0, 256, (K, C, 3, 3), dtype=np.uint8)
    xb[0, :, : max(1, H // 2)], gb[0] = 0x80, 0x80      # -128 times -128 as signed bytes
    xi, gi = xb.view(np.int8), gb.view(np.int8)
    want = oracle.direct_conv2d(xi, gi)
    packed = wg.winograd_filter_transform(_in(gi, layout, wl.to_krsc), layout, wg.LOSSLESS)
    wg.stream_workgroups(workgroups)
    assert np.array_equal(_nchw(wg.winograd_conv2d_int8(_in(xi, layout, wl.to_nhwc), packed, layout), layout), want)
    for relu, pool in ((False, False), (True, True)):
        if pool and (H | W) & 1:
            continue
        got = wg.winograd_conv2d_int8_requant(_in(xi, layout, wl.to_nhwc), packed, SHIFT, relu, pool, layout)
        assert np.array_equal(_nchw(got, layout), oracle.requant_relu_pool(want, SHIFT, relu, pool))
    packed = wg.winograd_filter_transform_u8(_in(gb, layout, wl.to_krsc), ZW, layout, wg.LOSSLESS)
    got = wg.winograd_conv2d_u8(_in(xb, layout, wl.to_nhwc), ZX, packed, layout)
    assert np.array_equal(_nchw(got, layout), oracle.direct_conv2d_i16(xb.astype(np.int16) - ZX, gb.astype(np.int16) - ZW))
