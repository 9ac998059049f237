"""Outputs and partial sums that are written through the L2, on either side of the rules (write_through.h): bit for bit against the oracle.
(tests/test_write_through_rule.py asks the rules themselves.)"""
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


def _calls(gd, layout):
    """Every call with int32 outputs, and the oracle's answer to it."""
    lossless, scaled = wg.winograd_filter_transform(gd, layout, wg.LOSSLESS), wg.winograd_filter_transform(gd, layout, wg.SCALED)
    f2 = wg.f2x2_filter_transform(gd, layout, wg.LOSSLESS)
    return [(lambda x, out=None: wg.winograd_conv2d_int8(x, lossless, layout, out=out), oracle.direct_conv2d),
            (lambda x, out=None: wg.direct_conv2d_int8(x, gd, layout, out=out), oracle.direct_conv2d),
            (lambda x, out=None: wg.f2x2_conv2d_int8(x, f2, layout, out=out), oracle.direct_conv2d),
            (lambda x, out=None: wg.winograd_conv2d_int8(x, scaled, layout, out=out), lambda x, g: oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]),
            (lambda x, out=None: wg.winograd_conv2d_int8_act_scaled(x, scaled, layout, out=out), lambda x, g: oracle.winograd_conv2d(x, g, oracle.BOTH_SCALED, 127)[0])]


def _operands(shape):
    N, C, K, H, W = shape
    rng = np.random.default_rng(77)
    return rng.integers(-128, 128, (N, C, H, W)).astype(np.int8), rng.integers(-128, 128, (K, C, 3, 3)).astype(np.int8)


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("shape", [
    (6, 16, 64, 37, 37),     # 525,696 outputs: just through; partial tiles
    (6, 16, 64, 36, 37),     # 511,488: just not
    (7, 80, 75, 32, 32),     # K odd: channels-last outputs stored one by one; two channel blocks
    (9, 48, 68, 49, 21),     # channels-last lines in parts, rows of 21
    (42, 16, 64, 14, 14),    # channel-major rows that are too short
    (128, 64, 64, 9, 9),     # more than a round of tile blocks
])
def test_convolutions_equal_the_oracle(shape, layout):
    x, g = _operands(shape)
    xd, ends, answers = _in(x, layout, wl.to_nhwc), [0, len(x) - 1], {}
    for call, answer in _calls(_in(g, layout, wl.to_krsc), layout):
        whole = answer is oracle.direct_conv2d
        if answer not in answers:
            answers[answer] = answer(x if whole else x[ends], g)
        got = call(xd) if whole else call(xd)[ends]
        assert np.array_equal(_nchw(got, layout), answers[answer])


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("shape", [
    (13, 16, 100, 56, 56), (14, 16, 100, 56, 56),   # parts of lines, 4.08 and 4.39 million outputs (4 Mi); direct: 160 and 172 pixel blocks
    (17, 16, 100, 56, 56),                          # 5.33 (5 Mi)
    (20, 16, 64, 56, 56), (21, 16, 64, 56, 56),     # channel-major rows in parts, 4.01 and 4.21 (4 Mi)
    (41, 16, 48, 56, 56), (42, 16, 48, 56, 56),     # whole 64-byte units, 6.17 and 6.32 (6 Mi)
    (20, 16, 64, 112, 112), (21, 16, 64, 112, 112), # whole lines, 16.1 and 16.9 (16 Mi)
    (32, 64, 84, 32, 32),                           # direct: two filter blocks of one XCD write a line
])
def test_many_outputs_equal_the_oracle(shape, layout):
    x, g = _operands(shape)
    some = [0, len(x) // 2, len(x) - 1]
    xd, answers = _in(x, layout, wl.to_nhwc), {}
    for call, answer in _calls(_in(g, layout, wl.to_krsc), layout):
        if answer not in answers:
            answers[answer] = answer(x[some], g)
        assert np.array_equal(_nchw(call(xd)[some], layout), answers[answer])


@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("offset", [4, 16, 64])
@pytest.mark.parametrize("shape", [(6, 16, 64, 37, 37), (4, 48, 96, 64, 32), (14, 64, 68, 28, 28)])
def test_outputs_off_a_boundary_are_the_same(shape, offset, layout):
    x, g = _operands(shape)
    xd, gd = _in(x, layout, wl.to_nhwc), _in(g, layout, wl.to_krsc)
    for call, _ in _calls(gd, layout):
        want = call(xd)
        assert want.data_ptr() % 128 == 0
        room = torch.full((want.numel() + 64,), 97531, dtype=torch.int32, device="cuda")
        out = room[offset // 4:offset // 4 + want.numel()].view(want.shape)
        call(xd, out=out)
        assert torch.equal(out, want)
        assert bool((room[:offset // 4] == 97531).all()) and bool((room[offset // 4 + want.numel():] == 97531).all())


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
