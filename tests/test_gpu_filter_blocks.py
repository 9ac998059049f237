"""Filter counts that fill a 64-filter block at most half, on grids of one and of several rounds of the compute units (the
library's own choice of form), and grids whose size is no multiple of the eight XCDs.  Bit for bit against the CPU oracle."""
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
    (1, 16, 16, 260, 260),    # one channel block, 265 workgroups of 32 filters
    (1, 16, 96, 190, 190),    # 144 tile blocks: 432 workgroups of 32 filters, 288 of 64
    (1, 12, 161, 96, 96),     # 216 workgroups of 32 filters (one filter in the last block): the rule for more than a round does not apply
    (1, 72, 32, 260, 259),    # two channel blocks
    (1, 72, 96, 150, 150),    # 91 tile blocks
    (1, 72, 330, 96, 96),     # 216 workgroups of 64 filters
    (3, 72, 330, 9, 9),       # 22 of 32
    (1, 264, 80, 20, 36),     # split channels
    (1, 224, 16, 24, 24), (1, 224, 16, 48, 48),   # at most 32 filters: split in either mode, and in lossless mode alone
    (1, 116, 16, 80, 96),     # in one kernel in either mode, by 4-byte loads
]


@pytest.mark.parametrize("mode", ["lossless", "scaled"])
@pytest.mark.parametrize("shape", [(1, 224, 16, 48, 48), (4, 240, 20, 19, 19), (1, 116, 16, 80, 96)])
def test_few_filters_from_channel_major(shape, mode):   # split without a copy, with either kernel's sums
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="relu", wgt="gauss", seed=8)
    want = oracle.direct_conv2d(x, g) if mode == "lossless" else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(_dev(g), wg.NCHW, wg.LOSSLESS if mode == "lossless" else wg.SCALED)
    assert np.array_equal(wg.winograd_conv2d_int8(_dev(x), packed, wg.NCHW).cpu().numpy(), want)


@pytest.mark.parametrize("mode", ["lossless", "scaled"])
@pytest.mark.parametrize("shape", SHAPES)
def test_equals_oracle(shape, mode):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="relu", wgt="gauss", seed=8)
    want = oracle.direct_conv2d(x, g) if mode == "lossless" else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(_dev(wl.to_krsc(g)), wg.NHWC, wg.LOSSLESS if mode == "lossless" else wg.SCALED)
    xd = _dev(wl.to_nhwc(x))
    y = wg.winograd_conv2d_int8(xd, packed, wg.NHWC)
    assert np.array_equal(wl.from_nhwc(y.cpu().numpy()), want)
    q = wg.winograd_conv2d_int8_requant(xd, packed, 10, True, False, wg.NHWC)
    assert np.array_equal(wl.from_nhwc(q.cpu().numpy()), oracle.requant_relu_pool(want, 10, True, False))


# One channel block, more than one round of 32 filters: what the rule takes for signed channels-last tensors, scaled / lossless
ONE_BLOCK = [
    (1, 16, 96, 160, 160),    # 100 tile blocks: eight product waves / whole entries
    (1, 16, 80, 210, 210),    # 176: whole entries in either mode
    (1, 16, 16, 364, 364),    # 518: halves in either mode
    (1, 12, 90, 150, 150),    # 91, int8 outputs byte by byte: eight product waves / the limb-pair kernel
    (1, 9, 23, 262, 259),     # 269, the same: halves / the limb-pair kernel
]


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("mode", ["lossless", "scaled"])
@pytest.mark.parametrize("shape", ONE_BLOCK)
def test_one_channel_block(shape, mode, layout):
    N, C, K, H, W = shape
    nhwc, lossless = layout == wg.NHWC, mode == "lossless"
    blob_mode = wg.LOSSLESS if lossless else wg.SCALED
    put = lambda a: _dev(wl.to_nhwc(a) if nhwc else a)
    get = lambda t: wl.from_nhwc(t.cpu().numpy()) if nhwc else t.cpu().numpy()
    filters = lambda g: _dev(wl.to_krsc(g) if nhwc else g)
    x, g = wl.make_custom(N, C, K, H, W, act="relu", wgt="gauss", seed=10)
    want = oracle.direct_conv2d(x, g) if lossless else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(filters(g), layout, blob_mode)
    assert np.array_equal(get(wg.winograd_conv2d_int8(put(x), packed, layout)), want)
    for pool in (False, True) if H % 2 == 0 and W % 2 == 0 else (False,):
        q = wg.winograd_conv2d_int8_requant(put(x), packed, 10, True, pool, layout)
        assert np.array_equal(get(q), oracle.requant_relu_pool(want, 10, True, pool))
    rng = np.random.default_rng(K)
    xq, gq = rng.integers(0, 256, x.shape, dtype=np.uint8), rng.integers(0, 256, g.shape, dtype=np.uint8)
    x9, g9 = xq.astype(np.int16) - 117, gq.astype(np.int16) - 131
    want = oracle.direct_conv2d_i16(x9, g9) if lossless else oracle.winograd_conv2d_i16(x9, g9, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform_u8(filters(gq), 131, layout, blob_mode)
    assert np.array_equal(get(wg.winograd_conv2d_u8(put(xq), 117, packed, layout)), want)


@pytest.mark.parametrize("shape", [
    (1, 72, 16, 40, 33), (2, 40, 97, 30, 30), (1, 130, 330, 22, 18),
    (1, 20, 80, 256, 260),    # 260 tile blocks: four rounds of 32 filters, three of 64
    (1, 12, 16, 280, 280),    # 307: two and two
])
def test_activations_scaled_as_well(shape):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="relu", wgt="gauss", seed=9)
    want = oracle.winograd_conv2d(x, g, oracle.BOTH_SCALED, 127)[0]
    packed = wg.winograd_filter_transform(_dev(wl.to_krsc(g)), wg.NHWC, wg.SCALED)
    y = wg.winograd_conv2d_int8_act_scaled(_dev(wl.to_nhwc(x)), packed, wg.NHWC)
    assert np.array_equal(wl.from_nhwc(y.cpu().numpy()), want)
