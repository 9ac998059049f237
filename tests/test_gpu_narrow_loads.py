"""First-layer kernel (at most four channels, channels-last): one dword per pixel, shifted where it would run past the tensor's
end, in tensors of one to a few pixels and at the last tiles of larger ones, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("N,H,W", [(1, 1, 1), (1, 1, 2), (1, 3, 1), (2, 1, 1), (1, 4, 5), (3, 13, 2), (2, 9, 21)])
@pytest.mark.parametrize("C", [1, 2, 3, 4])
def test_narrow_patch_loads(C, N, H, W, mode):
    x, g = wl.make_custom(N, C, 70, H, W, act="uniform", wgt="uniform", seed=C)
    packed = wg.winograd_filter_transform(torch.from_numpy(wl.to_krsc(g)).cuda(), wg.NHWC, mode)
    y = wg.winograd_conv2d_int8(torch.from_numpy(wl.to_nhwc(x)).cuda(), packed, wg.NHWC)
    want = oracle.direct_conv2d(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    assert np.array_equal(wl.from_nhwc(y.cpu().numpy()), want)
