"""Paths that use scratch memory: channels-last copies of channel-major and odd-channel inputs, channel blocks dealt to
several workgroups, and the stores of any K in either layout, against the oracle; and the same calls through the C ABI,
which gives the int8 entry point no scratch."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, C, K, H, W: split channels with one and several blocks per workgroup, a last split that is shorter, a last block that
# is not full; ragged tiles; K at and around multiples of 4, 16, 32 and 64; images of one to four pixels
SPLIT = [(1, 512, 40, 14, 14), (1, 320, 96, 8, 10), (1, 896, 31, 6, 6), (2, 500, 65, 4, 14), (1, 448, 512, 14, 9),
         (4, 820, 250, 14, 14), (4, 448, 512, 14, 14)]   # (these two: two blocks per workgroup, one in the last)
COPY = [(2, 5, 7, 9, 11), (1, 130, 33, 3, 5), (3, 67, 66, 1, 1), (2, 64, 100, 1, 3), (1, 3, 64, 10, 6), (2, 31, 130, 21, 20)]


def _inputs(shape, layout):
    N, C, K, H, W = shape
    x, g = wl.make_custom(N, C, K, H, W, act="uniform", wgt="uniform", seed=5)
    nhwc = layout == wg.NHWC
    return x, g, torch.from_numpy(wl.to_nhwc(x) if nhwc else x).cuda(), torch.from_numpy(wl.to_krsc(g) if nhwc else g).cuda()


def _nchw(t, layout):
    a = t.cpu().numpy()
    return wl.from_nhwc(a) if layout == wg.NHWC else a


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("layout", [wg.NCHW, wg.NHWC])
@pytest.mark.parametrize("shape", SPLIT + COPY)
def test_int32_and_int8_outputs(shape, layout, mode):
    x, g, xd, gd = _inputs(shape, layout)
    want = oracle.direct_conv2d(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(gd, layout, mode)
    assert np.array_equal(_nchw(wg.winograd_conv2d_int8(xd, packed, layout), layout), want)
    N, C, K, H, W = shape
    for relu, pool in ((True, False), (False, True)):
        if pool and (H | W) & 1:
            continue
        got = wg.winograd_conv2d_int8_requant(xd, packed, 9, relu, pool, layout)
        expect = oracle.requant_relu_pool(want, 9, relu, pool)
        assert np.array_equal(_nchw(got, layout), expect)
        # the C ABI's entry point has no scratch memory to offer
        bare = torch.full_like(got, 77)
        p = lambda t: ctypes.c_void_p(t.data_ptr())
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert wg.load_library().winograd_conv2d_int8_requant(p(xd), p(packed.blob), p(bare), N, C, H, W, K, layout, mode, 9,
                                                              int(relu), int(pool), stream) == 0
        assert np.array_equal(_nchw(bare, layout), expect)


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("C", [256, 576, 640])
@pytest.mark.parametrize("K, H, W", [(32, 6, 10), (33, 10, 6), (100, 2, 14), (68, 4, 4)])
def test_splits_are_finished_whatever_their_number(C, K, H, W, mode):
    """Four splits, nine and ten (more than a thread reads at once); tiles cut by the image's edge and windows of them;
    filters just into and just short of a block of 32, channels-last outputs stored by fours and one by one."""
    x, g, xd, gd = _inputs((1, C, K, H, W), wg.NHWC)
    want = oracle.direct_conv2d(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(gd, wg.NHWC, mode)
    assert np.array_equal(_nchw(wg.winograd_conv2d_int8(xd, packed, wg.NHWC), wg.NHWC), want)
    for relu, pool in ((True, True), (False, False)):
        got = wg.winograd_conv2d_int8_requant(xd, packed, 10, relu, pool, wg.NHWC)
        assert np.array_equal(_nchw(got, wg.NHWC), oracle.requant_relu_pool(want, 10, relu, pool))


@pytest.mark.parametrize("mode", [wg.LOSSLESS, wg.SCALED])
@pytest.mark.parametrize("layout", [wg.NCHW, wg.NHWC])
@pytest.mark.parametrize("shape", [(2, 64, 64, 9, 10), (2, 6, 70, 5, 5), (1, 200, 33, 14, 7), (40, 32, 128, 14, 14), (9, 128, 72, 28, 28)])
def test_uint8_inputs(shape, layout, mode):
    """Padding pixels read as the zero point on every form that takes uint8 tensors."""
    N, C, K, H, W = shape
    rng = np.random.default_rng(11)
    x, g = rng.integers(0, 256, (N, C, H, W), dtype=np.uint8), rng.integers(0, 256, (K, C, 3, 3), dtype=np.uint8)
    zx, zw = 201, 117
    xi, gi = x.astype(np.int16) - zx, g.astype(np.int16) - zw
    want = oracle.direct_conv2d_i16(xi, gi) if mode == wg.LOSSLESS else oracle.winograd_conv2d_i16(xi, gi, oracle.SCALED, 127)[0]
    nhwc = layout == wg.NHWC
    xd = torch.from_numpy(wl.to_nhwc(x) if nhwc else x).cuda()
    packed = wg.winograd_filter_transform_u8(torch.from_numpy(wl.to_krsc(g) if nhwc else g).cuda(), zw, layout, mode)
    assert np.array_equal(_nchw(wg.winograd_conv2d_u8(xd, zx, packed, layout), layout), want)


def test_mismatched_filters_leave_the_output_untouched_with_split_channels():
    """The kernels find a blob of another layer on the device and write nothing, in both halves of a split convolution."""
    x, g, xd, gd = _inputs((1, 512, 64, 8, 8), wg.NHWC)
    for mode in (wg.LOSSLESS, wg.SCALED):
        packed = wg.winograd_filter_transform(gd, wg.NHWC, mode)
        packed.blob[8] += 1            # K in the header
        out = torch.full((1, 8, 8, 64), 123, dtype=torch.int32, device="cuda")
        wg.winograd_conv2d_int8(xd, packed, wg.NHWC, out=out)
        assert bool((out == 123).all())


@pytest.mark.parametrize("layout", [wg.NCHW, wg.NHWC])
@pytest.mark.parametrize("shape", [(1, 5, 33, 7, 6), (2, 130, 65, 10, 9), (40, 64, 160, 14, 14), (1, 896, 20, 4, 5),
                                   # one round of workgroups and a little more, one and two channel blocks: both sides of the
                                   # rule that keeps the two passes in one kernel
                                   (32, 64, 250, 16, 16), (33, 64, 250, 16, 16), (43, 100, 150, 14, 13), (32, 128, 256, 15, 14), (2, 192, 33, 9, 9)])
def test_both_sides_scaled_with_and_without_scratch(shape, layout):
    """32 and 64 filters per workgroup, one to fourteen channel blocks, against the oracle; the C ABI's entry point has no
    scratch memory and runs both passes in one kernel."""
    N, C, K, H, W = shape
    x, g, xd, gd = _inputs(shape, layout)
    want = oracle.winograd_conv2d(x, g, 2, 127)[0]
    packed = wg.winograd_filter_transform(gd, layout, wg.SCALED)
    got, table = wg.winograd_conv2d_int8_act_scaled(xd, packed, layout, want_table=True)
    assert np.array_equal(_nchw(got, layout), want)
    bare, bare_table = torch.full_like(got, 77), torch.zeros_like(table)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert wg.load_library().winograd_conv2d_int8_act_scaled(p(xd), p(packed.blob), p(bare), N, C, H, W, K, layout, p(bare_table), stream) == 0
    assert torch.equal(bare, got) and torch.equal(bare_table, table)


def test_calls_run_without_the_memory_they_would_like_and_outputs_without_memory_raise_torchs_error():
    """Channel-major tensors with an odd channel count: every call would like a copy of 29 MB.  With no memory left they
    write the caller's output as they can; without a caller's output they raise torch.cuda.OutOfMemoryError."""
    N, C, K, H, W = 8, 67, 48, 224, 224
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    bytes_like = lambda *shape: torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda", generator=gen)
    x, w = bytes_like(N, C, H, W), bytes_like(K, C, 3, 3)
    y = lambda dtype: torch.zeros((N, K, H, W), dtype=dtype, device="cuda")
    packed = {m: wg.winograd_filter_transform(w, wg.NCHW, m) for m in (wg.LOSSLESS, wg.SCALED)}
    packed_u8 = wg.winograd_filter_transform_u8(w.view(torch.uint8), 100, wg.NCHW, wg.SCALED)
    packed_f2 = wg.f2x2_filter_transform(w, wg.NCHW, wg.LOSSLESS)
    calls = [(torch.int32, lambda out: wg.winograd_conv2d_int8(x, packed[wg.LOSSLESS], wg.NCHW, out=out)),
             (torch.int8, lambda out: wg.winograd_conv2d_int8_requant(x, packed[wg.SCALED], 12, layout=wg.NCHW, out=out)),
             (torch.int32, lambda out: wg.winograd_conv2d_u8(x.view(torch.uint8), 90, packed_u8, wg.NCHW, out=out)),
             (torch.int32, lambda out: wg.winograd_conv2d_int8_act_scaled(x, packed[wg.SCALED], wg.NCHW, out=out)),
             (torch.int32, lambda out: wg.f2x2_conv2d_int8(x, packed_f2, wg.NCHW, out=out)),
             (torch.int8, lambda out: wg.f2x2_conv2d_int8_requant(x, packed_f2, 12, layout=wg.NCHW, out=out)),
             (torch.int32, lambda out: wg.direct_conv2d_int8(x, w, wg.NCHW, out=out))]
    wanted = [call(None) for _, call in calls]
    outs = [y(dtype) for dtype, _ in calls]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    try:
        torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / torch.cuda.get_device_properties(0).total_memory)
        held = []   # what the allocator holds in reserve from earlier work, in pieces down to 2 MB
        for mb in (1024, 256, 64, 16, 4, 2):
            try:
                while True:
                    held.append(torch.empty(mb << 20, dtype=torch.uint8, device="cuda"))
            except torch.cuda.OutOfMemoryError:
                pass
        for (_, call), out in zip(calls, outs):
            call(out)
        for _, call in calls:
            with pytest.raises(torch.cuda.OutOfMemoryError):
                call(None)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    for out, want in zip(outs, wanted):
        assert torch.equal(out, want)


@pytest.mark.parametrize("mode, layout, shape, splits", [
    # two to three channel blocks per workgroup, fewer in the last split.  Lossless mode, up to ten tile blocks: splits are dealt out first
    (wg.LOSSLESS, wg.NHWC, (1, 320, 192, 40, 64), 3), (wg.LOSSLESS, wg.NHWC, (1, 516, 250, 38, 40), 3),   # the second: C no multiple of 16
    (wg.LOSSLESS, wg.NHWC, (1, 320, 160, 44, 64), 3),                                                     # eleven tile blocks: those first
    # the same with 16 filters per workgroup, its waves sharing the entries in quarters
    (wg.LOSSLESS, wg.NHWC, (1, 580, 75, 40, 64), 5), (wg.LOSSLESS, wg.NHWC, (1, 324, 100, 52, 56), 3),
    (wg.LOSSLESS, wg.NHWC, (2, 512, 9, 56, 112), 4), (wg.LOSSLESS, wg.NHWC, (1, 320, 48, 80, 84), 3),
    (wg.LOSSLESS, wg.NCHW, (1, 512, 16, 84, 112), 4),
    (wg.SCALED, wg.NHWC, (1, 640, 60, 60, 64), 5),
    # one block per workgroup, C no multiple of 16
    (wg.LOSSLESS, wg.NHWC, (1, 600, 20, 49, 66), 10), (wg.SCALED, wg.NHWC, (1, 600, 20, 49, 66), 10), (wg.SCALED, wg.NHWC, (1, 580, 130, 32, 40), 10)])
def test_split_channels_in_either_order_of_the_grid(mode, layout, shape, splits):
    N, C, K, H, W = shape
    wanted = wg.load_library()._ZN2wg20conv2d_scratch_bytesEiiiiiiii
    wanted.restype, wanted.argtypes = ctypes.c_size_t, [ctypes.c_int] * 8
    tiles = (N * ((H + 3) // 4) * ((W + 3) // 4) + 15) // 16 * 16
    sums = (16 if mode == wg.LOSSLESS else 36) * tiles * ((K + 63) // 64 * 64) * 4
    assert wanted(N, C, H, W, K, layout, mode, 0) == splits * sums   # as many splits as this shape is here for, and no copy
    x, g, xd, gd = _inputs(shape, layout)
    want = oracle.direct_conv2d(x, g) if mode == wg.LOSSLESS else oracle.winograd_conv2d(x, g, oracle.SCALED, 127)[0]
    packed = wg.winograd_filter_transform(gd, layout, mode)
    for _ in range(2):
        assert np.array_equal(_nchw(wg.winograd_conv2d_int8(xd, packed, layout), layout), want)
    for pool in (False, True) if (H | W) % 2 == 0 else (False,):
        got = wg.winograd_conv2d_int8_requant(xd, packed, 10, True, pool, layout)
        assert np.array_equal(_nchw(got, layout), oracle.requant_relu_pool(want, 10, True, pool)), pool
