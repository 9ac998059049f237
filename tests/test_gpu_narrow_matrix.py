"""First layers (at most four channels, channels-last) on the matrix cores in half precision: every integer has to come out exactly, so
the extremes matter, with odd numbers beside them; and by the kernel of one wave per workgroup.  Either is forced by a test hook, so that
no line between them decides what is tested.  Several groups of 16 tiles per workgroup, a last one that is partly empty, ragged images,
filter counts stored four and sixteen at a time."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu
FORMS = {"matrix cores": 1, "one wave": 2}


@pytest.fixture(params=FORMS)
def form(request):
    wg.narrow_variant(FORMS[request.param])
    yield request.param
    wg.narrow_variant(0)


SHAPES = [(2, 3, 64, 128, 128), (1, 4, 132, 148, 126), (1, 1, 20, 200, 182), (5, 2, 80, 97, 110), (1, 4, 68, 460, 450)]


def _operands(N, C, K, H, W, values):
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=C + K)
    if values == "extreme":
        rng = np.random.default_rng(K)
        x = rng.choice(np.array([-128, -128, -128, -127, 127], np.int8), x.shape)
        g = rng.choice(np.array([-128, -128, 127], np.int8), g.shape)
        x[:, :, :H // 2] = -128
        g[::3] = -128
    elif values == "checkerboard":
        x[...] = np.where(np.indices(x.shape[2:]).sum(0) & 1, 127, -128)
        g[...] = np.where(np.indices((3, 3)).sum(0) & 1, -128, 127)
    return x, g


def _want(x, g, mode):
    return oracle.direct_conv2d(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("values", ["uniform", "extreme", "checkerboard"])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_output_form(shape, values, mode, form):
    x, g = _operands(*shape, values)
    want = _want(x, g, mode)
    packed = wg.winograd_filter_transform(torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC, mode)
    xd = torch.from_numpy(wl.to_nhwc(x)).cuda()
    assert np.array_equal(wl.from_nhwc(wg.winograd_conv2d_int8(xd, packed, wg.NHWC).cpu().numpy()), want)
    for shift, relu, pool in ((9, True, False), (11, False, False), (10, False, True), (0, True, True), (31, False, True)):
        if pool and (shape[3] % 2 or shape[4] % 2):
            continue
        got = wg.winograd_conv2d_int8_requant(xd, packed, shift, relu, pool, wg.NHWC)
        assert np.array_equal(wl.from_nhwc(got.cpu().numpy()), oracle.requant_relu_pool(want, shift, relu, pool)), (shift, relu, pool)


@pytest.mark.parametrize("values", ["uniform", "extreme"])
def test_lossless_int32_outputs(values):
    """(int32 outputs of lossless mode come from the matrix cores by themselves only in larger layers.)"""
    x, g = _operands(1, 4, 1000, 180, 178, values)
    packed = wg.winograd_filter_transform(torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC, wg.LOSSLESS)
    y = wg.winograd_conv2d_int8(torch.from_numpy(wl.to_nhwc(x)).cuda(), packed, wg.NHWC)
    assert np.array_equal(wl.from_nhwc(y.cpu().numpy()), oracle.direct_conv2d(x, g))


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("offset", [4, 8])
@pytest.mark.parametrize("K", [16, 64, 80])
def test_outputs_that_start_off_a_16_byte_boundary(K, offset, mode, form):
    """K % 16 = 0 would be stored 16 filters at a time; the buffer allows four."""
    shape = (1, 3, K, 38, 50)
    x, g = _operands(*shape, "uniform")
    want = _want(x, g, mode)
    packed = wg.winograd_filter_transform(torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC, mode)
    xd = torch.from_numpy(wl.to_nhwc(x)).cuda()
    for pool in (False, True):
        half = 2 if pool else 1
        size = (1, 38 // half, 50 // half, K)
        buffer = torch.full((size[1] * size[2] * K + 32,), 86, dtype=torch.int8, device="cuda")
        out = buffer[offset:offset + size[1] * size[2] * K].view(size)
        assert out.data_ptr() % 16 == offset
        wg.winograd_conv2d_int8_requant(xd, packed, 9, True, pool, wg.NHWC, out=out)
        assert np.array_equal(wl.from_nhwc(out.cpu().numpy()), oracle.requant_relu_pool(want, 9, True, pool)), pool
        assert (buffer[:offset] == 86).all() and (buffer[offset + out.numel():] == 86).all()
