"""Which int32 outputs are written through the L2 (write_through.h): the rule's choice, asked on the host, on either side of each of its lines."""
import os

import pytest

import paper_1901_01965_amd as wg
from paper_1901_01965_amd import binding

ROWS, PLANES, F2, DIRECT, FIRST, FIRST_INT8, FIRST_POOLED, PAIR_PLANES = range(8)
BASE = 1 << 20


@pytest.fixture(scope="module")
def through():
    if not os.path.exists(binding.LIB_PATH):
        from paper_1901_01965_amd import build
        build.build()
    lib = wg.load_library()

    def ask(kernel, N, K, H, W, offset=0, C=64):   # (C matters to direct convolution alone)
        r = lib.winograd_debug_writes_through(kernel, N, C, H, W, K, BASE + offset)
        assert r in (0, 1)
        return bool(r)

    return ask


@pytest.mark.parametrize("kernel", [ROWS, PLANES, F2, DIRECT])
def test_few_and_many_outputs_are_left_to_the_l2(through, kernel):
    assert not through(kernel, 1, 64, 64, 127) and through(kernel, 1, 64, 64, 128)            # 512 Ki outputs
    assert through(kernel, 64, 64, 64, 64) and not through(kernel, 65, 64, 64, 64)            # 16 Mi outputs


@pytest.mark.parametrize("kernel", [ROWS, PLANES, F2, DIRECT])
@pytest.mark.parametrize("offset", [4, 16, 48])
def test_outputs_off_a_64_byte_boundary_are_written_in_parts(through, kernel, offset):
    """64 outputs per pixel, rows of 64: whole lines on the boundary, none off it."""
    assert through(kernel, 4, 64, 256, 256) and through(kernel, 4, 64, 256, 256, 64)          # 16 Mi outputs
    assert not through(kernel, 4, 64, 256, 256, offset)
    assert through(kernel, 4, 64, 64, 64, offset) == (kernel != ROWS)                         # 1 Mi


@pytest.mark.parametrize("kernel,most", [(ROWS, 4), (F2, 5), (DIRECT, 5)])
def test_channels_last_lines_in_parts_are_few(through, kernel, most):
    """Mi outputs: K a multiple of 32, of 16, of neither; and of 32, but off a 64-byte boundary."""
    for K, offset, limit in ((96, 0, 16), (48, 0, 6), (16, 0, 6 if kernel == ROWS else most), (36, 0, most), (60, 0, most), (64, 16, 0 if kernel == ROWS else most)):
        pixels = (limit << 20) // K
        if limit == 0:
            assert not through(kernel, 1, K, 16384, 1, offset)
            continue
        assert through(kernel, 1, K, pixels, 1, offset) and not through(kernel, 1, K, pixels + 1, 1, offset), (K, offset)


def test_channel_major_rows_in_parts_are_few_and_not_narrow(through):
    """Mi outputs: rows of whole 64-byte units; of parts from 28, from 20 outputs on, and narrower; off a 64-byte boundary."""
    for W, offset, limit in ((16, 0, 16), (48, 0, 16), (224, 0, 16), (56, 0, 4), (53, 0, 4), (28, 0, 4), (27, 0, 2), (20, 0, 2), (19, 0, 0), (15, 0, 0),
                             (7, 0, 0), (64, 16, 2), (56, 4, 2), (16, 4, 0)):
        for K in (64, 75):
            rows = (limit << 20) // (K * W)
            assert limit == 0 or through(PLANES, 1, K, rows, W, offset), (W, offset, K)
            assert not through(PLANES, 1, K, max(rows + 1, (1 << 20) // (K * W)), W, offset), (W, offset, K)


@pytest.mark.parametrize("C,K,N,H,W", [(64, 84, 16, 32, 32), (64, 100, 32, 32, 32), (128, 72, 4, 64, 64), (64, 84, 13, 56, 56), (64, 80, 15, 56, 56),
                                       (64, 132, 16, 32, 32)])
def test_direct_filter_blocks_of_one_xcd_do_not_share_lines(through, C, K, N, H, W):
    """Pixel blocks a multiple of eight, so that the filter blocks of one go to one XCD: lines that two of them write stay in its L2."""
    assert not through(DIRECT, N, K, H, W, 0, C)
    assert through(DIRECT, N, K // 32 * 32, H, W, 0, C)                    # whole lines
    assert through(F2, N, K, H, W, 0, C)


def test_direct_lines_of_different_xcds_or_of_one_workgroup(through):
    assert through(DIRECT, 12, 84, 56, 56) and through(DIRECT, 14, 84, 56, 56)      # 147 and 172 pixel blocks
    assert through(DIRECT, 32, 48, 32, 32) and through(DIRECT, 32, 36, 32, 32)      # one filter block
    assert not through(DIRECT, 16, 96, 32, 32, 64)                                  # a base in the middle of a line


@pytest.mark.parametrize("kernel,K,W,offset", [
    (FIRST, 100, 224, 0), (FIRST, 132, 224, 0), (FIRST, 36, 225, 0), (FIRST, 52, 226, 0), (FIRST, 64, 224, 16), (FIRST, 48, 224, 16),
    (FIRST_INT8, 96, 224, 0), (FIRST_INT8, 48, 225, 0), (FIRST_INT8, 64, 224, 16), (FIRST_POOLED, 16, 224, 0), (FIRST_POOLED, 48, 224, 0), (FIRST_POOLED, 32, 226, 0)])
def test_first_layers_in_parts_are_few(through, kernel, K, W, offset):
    limit, per_row = (5 if kernel == FIRST else 32) << 20, K * W // (4 if kernel == FIRST_POOLED else 1)
    H = limit // per_row // 2 * 2
    assert through(kernel, 1, K, H, W, offset, 3) and not through(kernel, 1, K, H + 2, W, offset, 3)


@pytest.mark.parametrize("kernel,K,W", [
    (FIRST, 64, 223), (FIRST, 36, 224), (FIRST, 52, 56), (FIRST, 96, 225), (FIRST, 256, 224), (FIRST_INT8, 16, 224), (FIRST_INT8, 48, 224),
    (FIRST_INT8, 128, 225), (FIRST_POOLED, 32, 224), (FIRST_POOLED, 64, 226)])
def test_first_layers_of_whole_units_are_written_through(through, kernel, K, W):
    assert through(kernel, 1, K, 224, W, 0, 3) and through(kernel, 64, K, 224, W, 0, 3)


def test_narrow_channel_major_rows_of_the_limb_pair_kernel_are_left_to_the_l2(through):
    for W in (7, 13, 14, 15, 17, 19):
        assert not through(PAIR_PLANES, 4, 64, 14, W)
    for W in (16, 20, 28, 53, 56):
        assert through(PAIR_PLANES, 1, 16, 14, W) and through(PAIR_PLANES, 4, 64, 14, W)
    assert not through(PAIR_PLANES, 4, 64, 14, 16, 16) and through(PAIR_PLANES, 4, 64, 14, 28, 16)
