"""Every form of the streaming kernel with every input, output and filter count it takes: signed bytes to int32 and to int8,
uint8 with a zero point, both layouts, K that is no multiple of four, against the oracle; forced through the test hooks on
small shapes, and by the library's own choice at ordinary sizes."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu

HALVES, WHOLE, EIGHT = 2, 1, 3   # of stream_variant
ZX, ZW, SHIFT = 77, 201, 9


@pytest.fixture(autouse=True)
def hooks_off_afterwards():
    yield
    wg.stream_variant(0)
    wg.scaled_variant(0)
    wg.stream_workgroups(0)


def _in(a, layout):
    return torch.from_numpy(wl.to_nhwc(a) if layout == wg.NHWC else a).cuda()


def _filters(g, layout):
    return torch.from_numpy(wl.to_krsc(g) if layout == wg.NHWC else g).cuda()


def _nchw(t, layout):
    a = t.cpu().numpy()
    return wl.from_nhwc(a) if layout == wg.NHWC else a


def _signed(x, g, mode):
    return oracle.direct_conv2d(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]


def _unsigned(x, g, mode):
    x, g = x.astype(np.int16) - ZX, g.astype(np.int16) - ZW
    return oracle.direct_conv2d_i16(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d_i16(x, g, oracle.SCALED, 127)[0]


def _bytes(shape, seed):
    return np.random.default_rng(seed).integers(0, 256, shape, dtype=np.uint8)


CASES = [  # (N, C, K, H, W), workgroups per filter block: several tile blocks for each
    ((2, 64, 40, 18, 22), 3),       # one channel block
    ((1, 100, 75, 14, 26), 2),      # two, the last one not full; odd K
    ((1, 130, 66, 12, 20), 1),      # three, an odd channel count (a copy in either layout)
    ((3, 20, 97, 9, 13), 2),        # one that is not full, odd everything
]


# (in scaled mode the form with whole entries exists for one channel block only)
FORMS = [(case, mode, form) for case in CASES for mode in (wg.LOSSLESS, wg.SCALED) for form in (HALVES, WHOLE, EIGHT)
         if form != WHOLE or mode == wg.LOSSLESS or case[0][1] <= 64]


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("case,mode,form", FORMS)
def test_forced_forms_equal_the_oracle(case, mode, form, layout):
    (N, C, K, H, W), workgroups = case
    xb, gb = _bytes((N, C, H, W), 21), _bytes((K, C, 3, 3), 22)
    xi, gi = xb.view(np.int8), gb.view(np.int8)
    want, want_u8 = _signed(xi, gi, mode), _unsigned(xb, gb, mode)
    packed = wg.winograd_filter_transform(_filters(gi, layout), layout, mode)
    packed_u8 = wg.winograd_filter_transform_u8(_filters(gb, layout), ZW, layout, mode)
    wg.stream_variant(form)
    wg.scaled_variant(2)
    wg.stream_workgroups(workgroups)
    assert np.array_equal(_nchw(wg.winograd_conv2d_int8(_in(xi, layout), packed, layout), layout), want)
    assert np.array_equal(_nchw(wg.winograd_conv2d_u8(_in(xb, layout), ZX, packed_u8, layout), layout), want_u8)
    for relu, pool in ((False, False), (True, True)):
        if pool and (H | W) & 1:
            continue
        got = wg.winograd_conv2d_int8_requant(_in(xi, layout), packed, SHIFT, relu, pool, layout)
        assert np.array_equal(_nchw(got, layout), oracle.requant_relu_pool(want, SHIFT, relu, pool))


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("shape,layout", [((32, 128, 128, 56, 56), wg.NHWC), ((32, 128, 126, 56, 56), wg.NCHW), ((24, 64, 64, 56, 56), wg.NCHW),
                                          ((24, 64, 63, 56, 56), wg.NHWC)])
def test_the_librarys_choice_at_ordinary_sizes(shape, layout, mode):
    """Sizes at which the library streams by itself, with 64 filters per workgroup; the first and the last image."""
    N, C, K, H, W = shape
    xb, gb = _bytes((N, C, H, W), 23), _bytes((K, C, 3, 3), 24)
    xi, gi = xb.view(np.int8), gb.view(np.int8)
    packed = wg.winograd_filter_transform(_filters(gi, layout), layout, mode)
    y = wg.winograd_conv2d_int8(_in(xi, layout), packed, layout)
    q = wg.winograd_conv2d_int8_requant(_in(xi, layout), packed, SHIFT, True, True, layout)
    u = wg.winograd_conv2d_u8(_in(xb, layout), ZX, wg.winograd_filter_transform_u8(_filters(gb, layout), ZW, layout, mode), layout)
    for at in (0, N - 1):
        image = slice(at, at + 1)
        want = _signed(xi[image], gi, mode)
        assert np.array_equal(_nchw(y[image], layout), want)
        assert np.array_equal(_nchw(q[image], layout), oracle.requant_relu_pool(want, SHIFT, True, True))
        assert np.array_equal(_nchw(u[image], layout), _unsigned(xb[image], gb, mode))
