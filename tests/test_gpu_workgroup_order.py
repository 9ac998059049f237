"""Every kernel whose workgroups are dealt to the XCDs in an order of their own, in both orders (by tiles, by filters), on grids
that are no multiple of the eight XCDs and smaller than eight: bit for bit against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu

ZX, ZW = 117, 131


@pytest.fixture(autouse=True)
def hooks_off_afterwards():
    yield
    wg.stream_variant(0)
    wg.scaled_variant(0)
    wg.lossless_variant(0)
    wg.stream_workgroups(0)


def _in(a, layout):
    return torch.from_numpy(np.ascontiguousarray(wl.to_nhwc(a) if layout == wg.NHWC else a)).cuda()


def _filters(g, layout):
    return torch.from_numpy(np.ascontiguousarray(wl.to_krsc(g) if layout == wg.NHWC else g)).cuda()


def _nchw(t, layout):
    a = t.cpu().numpy()
    return wl.from_nhwc(a) if layout == wg.NHWC else a


def _set_form(form):
    if form in ("halves", "whole", "eight"):
        wg.stream_variant({"halves": 2, "whole": 1, "eight": 3}[form])
        wg.stream_workgroups(5)
    elif form == "roles, 64 filters":
        wg.scaled_variant(1)
    elif form == "roles, 32 filters":
        wg.scaled_variant(2)
    else:
        wg.lossless_variant(2)


# N, C, K, H, W: 3, 6, 2, 9, 2 and 2 tile blocks; four and eight filter blocks in the fourth; the planes of the last two outweigh the
# activations
SHAPES = [(1, 72, 75, 30, 22), (2, 72, 161, 30, 22), (1, 60, 130, 22, 18), (3, 40, 225, 30, 22), (1, 264, 330, 22, 18), (1, 136, 364, 21, 18)]


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("form", ["halves", "whole", "eight", "roles, 64 filters", "roles, 32 filters", "four waves"])
@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("shape", SHAPES)
def test_equals_oracle(shape, mode, form, layout):
    N, C, K, H, W = shape
    if form == "whole" and mode == wg.SCALED and C > 64:
        pytest.skip("in scaled mode the form with whole entries exists for one channel block only")
    _set_form(form)
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=K)
    want = oracle.direct_conv2d(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(_filters(g, layout), layout, mode)
    assert np.array_equal(_nchw(wg.winograd_conv2d_int8(_in(x, layout), packed, layout), layout), want)
    q = wg.winograd_conv2d_int8_requant(_in(x, layout), packed, 10, True, False, layout)
    assert np.array_equal(_nchw(q, layout), oracle.requant_relu_pool(want, 10, True, False))
    if C > wg.MAX_CHANNELS_U8:
        return
    rng = np.random.default_rng(K)
    xq, gq = rng.integers(0, 256, x.shape, dtype=np.uint8), rng.integers(0, 256, g.shape, dtype=np.uint8)
    x9, g9 = xq.astype(np.int16) - ZX, gq.astype(np.int16) - ZW
    want = oracle.direct_conv2d_i16(x9, g9) if mode == wg.LOSSLESS else oracle.winograd_conv2d_i16(x9, g9, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform_u8(_filters(gq, layout), ZW, layout, mode)
    assert np.array_equal(_nchw(wg.winograd_conv2d_u8(_in(xq, layout), ZX, packed, layout), layout), want)


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("shape", SHAPES + [(2, 24, 97, 100, 90)])   # 75 tile blocks: 300 workgroups of 32 filters, 150 of 64
def test_activations_scaled_as_well(shape, layout):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="relu", wgt="gauss", seed=K)
    packed = wg.winograd_filter_transform(_filters(g, layout), layout, wg.SCALED)
    y = wg.winograd_conv2d_int8_act_scaled(_in(x, layout), packed, layout)
    assert np.array_equal(_nchw(y, layout), oracle.winograd_conv2d(x, g, oracle.BOTH_SCALED, 127)[0])
