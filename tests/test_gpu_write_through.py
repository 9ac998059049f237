"""Outputs and partial sums that are written through the L2, on either side of the rule (writes_through in wg_internal.h: 512 Ki outputs
and more, up to 16 Mi, or 6 Mi where K is no multiple of 32; channel-major rows of 16 and more): bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _in(a, layout, transposed):
    return torch.from_numpy(np.ascontiguousarray(transposed(a) if layout == wg.NHWC else a)).cuda()


def _nchw(t, layout):
    a = t.cpu().numpy()
    return wl.from_nhwc(a) if layout == wg.NHWC else a


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("shape", [
    (6, 16, 64, 37, 37),     # 525,696 outputs: just through; partial tiles
    (6, 16, 64, 36, 37),     # 511,488: just not
    (7, 80, 75, 32, 32),     # lines written in parts, two channel blocks, K odd
    (9, 48, 68, 49, 21),     # K a multiple of four only
    (42, 16, 64, 14, 14),    # channel-major rows that are too short
    (128, 64, 64, 9, 9),     # more than a round of tile blocks
])
def test_convolutions_equal_the_oracle(shape, layout):
    N, C, K, H, W = shape
    rng = np.random.default_rng(77)
    x, g = rng.integers(-128, 128, (N, C, H, W)).astype(np.int8), rng.integers(-128, 128, (K, C, 3, 3)).astype(np.int8)
    xd, gd = _in(x, layout, wl.to_nhwc), _in(g, layout, wl.to_krsc)
    want = oracle.direct_conv2d(x, g)
    ends = [0, N - 1]
    packed = wg.winograd_filter_transform(gd, layout, wg.LOSSLESS)
    assert np.array_equal(_nchw(wg.winograd_conv2d_int8(xd, packed, layout), layout), want)
    assert np.array_equal(_nchw(wg.direct_conv2d_int8(xd, gd, layout), layout), want)
    assert np.array_equal(_nchw(wg.f2x2_conv2d_int8(xd, wg.f2x2_filter_transform(gd, layout, wg.LOSSLESS), layout), layout), want)
    scaled = wg.winograd_filter_transform(gd, layout, wg.SCALED)
    got = _nchw(wg.winograd_conv2d_int8(xd, scaled, layout), layout)
    assert np.array_equal(got[ends], oracle.winograd_conv2d(x[ends], g, oracle.SCALED, 127)[0])
    both = _nchw(wg.winograd_conv2d_int8_act_scaled(xd, scaled, layout), layout)
    alone = [_nchw(wg.winograd_conv2d_int8_act_scaled(_in(x[n:n + 1], layout, wl.to_nhwc), scaled, layout), layout)[0] for n in ends]   # few outputs
    assert np.array_equal(both[ends], np.stack(alone))


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("shape", [(1, 512, 256, 14, 14), (1, 512, 64, 8, 8)])   # partial sums of 1 - 5 MB and of less than one
def test_split_channels_equal_the_oracle(shape, mode):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, seed=78)
    packed = wg.winograd_filter_transform(_in(g, wg.NHWC, wl.to_krsc), wg.NHWC, mode)
    for _ in range(2):   # in turn, so that nothing a call left in the scratch memory can stand in for what the next one writes
        for image in (x, x[..., ::-1]):
            want = oracle.direct_conv2d(np.ascontiguousarray(image), g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(np.ascontiguousarray(image), g, oracle.SCALED, 127)[0]
            assert np.array_equal(_nchw(wg.winograd_conv2d_int8(_in(image, wg.NHWC, wl.to_nhwc), packed, wg.NHWC), wg.NHWC), want)


@pytest.mark.parametrize("N,K,pool", [(24, 96, False), (23, 96, False), (96, 48, True)])   # 33.7, 32.3 and, pooled, 34.0 million: parts of lines beyond 32 Mi, below, beyond
def test_first_layers_with_many_int8_outputs_equal_the_oracle(N, K, pool):
    rng = np.random.default_rng(79)
    H, W = (120, 122) if not pool else (180, 164)
    x, g = rng.integers(-128, 128, (N, 3, H, W)).astype(np.int8), rng.integers(-128, 128, (K, 3, 3, 3)).astype(np.int8)
    some = [0, N // 2, N - 1]
    for mode in (wg.LOSSLESS, wg.SCALED):
        packed = wg.winograd_filter_transform(_in(g, wg.NHWC, wl.to_krsc), wg.NHWC, mode)
        got = _nchw(wg.winograd_conv2d_int8_requant(_in(x, wg.NHWC, wl.to_nhwc), packed, 9, True, pool, wg.NHWC)[some], wg.NHWC)
        want = oracle.direct_conv2d(x[some], g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x[some], g, oracle.SCALED, 127)[0]
        assert np.array_equal(got, oracle.requant_relu_pool(want, 9, True, pool))
