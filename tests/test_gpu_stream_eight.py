"""GPU parity of the streaming kernel's form with eight product waves (two waves per 16 filters; one stages, the other adds to
it), forced through the test hooks on small shapes: bit for bit against the CPU oracle, int32 and int8 outputs."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def eight_wave_stream():
    wg.stream_variant(3)
    yield
    wg.stream_variant(0)
    wg.stream_workgroups(0)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


CASES = [  # (N, C, K, H, W), workgroups per filter block
    ((1, 128, 64, 4, 4), 1),        # one tile, two channel blocks
    ((2, 64, 40, 18, 22), 3),       # one channel block, filters padded from 40 to 64, ragged tiles
    ((2, 132, 72, 30, 18), 2),      # three channel blocks, the last with four channels, two filter blocks
    ((1, 256, 128, 20, 12), 1),     # four channel blocks, every tile block through one workgroup
]


@pytest.mark.parametrize("mode", [wg.SCALED, wg.LOSSLESS])
@pytest.mark.parametrize("case", CASES)
def test_equals_oracle(case, mode):
    (N, C, K, H, W), slots = case
    x, g = wl.make_custom(N, C, K, H, W, act="relu", wgt="gauss", seed=17)
    if mode == wg.LOSSLESS:
        want = oracle.direct_conv2d(x, g)
    else:
        want, flags = oracle.winograd_conv2d(x, g, oracle.SCALED, 127)
        assert (flags & 5) == 0
    wg.stream_workgroups(slots)
    packed = wg.winograd_filter_transform(_dev(wl.to_krsc(g)), wg.NHWC, mode)
    xd = _dev(wl.to_nhwc(x))
    got = wg.winograd_conv2d_int8(xd, packed, wg.NHWC)
    assert np.array_equal(wl.from_nhwc(got.cpu().numpy()), want)
    shift = max(0, int(np.abs(want).max()).bit_length() - 7)
    for pool in (False, True):
        got = wg.winograd_conv2d_int8_requant(xd, packed, shift, True, pool, wg.NHWC)
        assert np.array_equal(wl.from_nhwc(got.cpu().numpy()), oracle.requant_relu_pool(want, shift, True, pool))
    packed = wg.winograd_filter_transform(_dev(g), wg.NCHW, mode)
    got = wg.winograd_conv2d_int8(_dev(x), packed, wg.NCHW)
    assert np.array_equal(got.cpu().numpy(), want)
