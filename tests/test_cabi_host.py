"""Host-side checks of the C ABI that need no GPU: the library loads, exports every function the header
declares, sizes are consistent, and every validation error path returns its code before any launch."""
import ctypes
import os
import re

import pytest

import paper_1901_01965_amd as wg
from paper_1901_01965_amd import binding, workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "winograd_c.h")

OK, EINVAL, EUNSUPPORTED, ESMALLBUF = 0, -1, -2, -3


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.LIB_PATH):
        from paper_1901_01965_amd import build
        build.build()
    return wg.load_library()


def _declared_functions():
    text = re.sub(r"/\*.*?\*/", "", open(HEADER).read(), flags=re.S)
    return sorted(set(re.findall(r"\b(winograd_\w+|direct_conv2d_int8|requant_relu_pool_int8)\s*\(", text)))


def test_every_declared_function_is_exported(lib):
    names = _declared_functions()
    assert len(names) >= 12
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(binding.EXPORTED_SYMBOLS) == names


def test_status_strings(lib):
    for code in range(-6, 1):
        assert wg.binding.status_string(code)
    assert "blob" in wg.binding.status_string(-4)


def test_size_queries(lib):
    assert wg.packed_filter_bytes(0, 4, 0) == 0 and lib.winograd_packed_filter_bytes(4, 4, 7) == 0
    assert wg.packed_filter_bytes(4, 897, 0) == 0            # beyond WG_MAX_CHANNELS
    lossless, scaled = wg.packed_filter_bytes(64, 64, wg.LOSSLESS), wg.packed_filter_bytes(64, 64, wg.SCALED)
    assert lossless > 138 * 64 * 64 and scaled > 46 * 64 * 64 and lossless > scaled
    assert lossless % 256 == 0
    # padding: K up to 64, C up to 64
    assert wg.packed_filter_bytes(1, 5, 0) == wg.packed_filter_bytes(64, 64, 0)
    # up to four input channels: the blob also carries the 36 values of each filter as int16 x 4 channel slots
    assert wg.packed_filter_bytes(1, 1, 0) == wg.packed_filter_bytes(64, 4, 0) == wg.packed_filter_bytes(64, 64, 0) + 64 * 36 * 4 * 2
    assert wg.workspace_bytes(0, 1, 1, 1, 1, 0) == 0
    c = wl.CASES["cfg2"]
    ws = wg.workspace_bytes(c.N, c.C, c.H, c.W, c.K, wg.LOSSLESS)
    assert ws >= 138 * c.tiles * c.C + 36 * 4 * c.tiles * c.K
    assert lib.winograd_num_activation_planes(0) == 138 and lib.winograd_num_activation_planes(1) == 72
    assert lib.winograd_num_filter_planes(0) == 138 and lib.winograd_num_filter_planes(1) == 46
    assert lib.winograd_num_filter_planes(5) == 0


def test_path_query(lib):
    assert wg.conv2d_path(8, 64, 56, 56, 64, wg.LOSSLESS) == wg.FUSED
    assert wg.conv2d_path(64, 512, 7, 7, 512, wg.SCALED) == wg.FUSED
    assert lib.winograd_debug_force_path(wg.STAGED) == OK
    assert wg.conv2d_path(8, 64, 56, 56, 64, wg.LOSSLESS) == wg.STAGED
    assert lib.winograd_debug_force_path(wg.AUTO) == OK
    assert lib.winograd_conv2d_path(8, 64, 56, 56, 64, 9) == EINVAL
    assert lib.winograd_debug_force_path(3) == EINVAL
    assert lib.winograd_debug_force_path(0) == OK


def test_validation_errors_return_before_any_launch(lib):
    """Fake but well-aligned addresses: every call must be rejected on the host (nothing dereferences them)."""
    p = ctypes.c_void_p
    good, good2, good3 = p(0x10000), p(0x20000), p(0x30000)
    odd = p(0x10001)
    big = 1 << 40
    ft = lib.winograd_filter_transform
    assert ft(None, 4, 4, 0, 0, good, big, None) == EINVAL
    assert ft(good, 4, 4, 0, 0, None, big, None) == EINVAL
    assert ft(good, 0, 4, 0, 0, good2, big, None) == EINVAL
    assert ft(good, 4, -1, 0, 0, good2, big, None) == EINVAL
    assert ft(good, 4, 4, 2, 0, good2, big, None) == EINVAL          # unknown layout
    assert ft(good, 4, 4, 0, 2, good2, big, None) == EINVAL          # unknown mode
    assert ft(good, 4, 897, 0, 0, good2, big, None) == EUNSUPPORTED  # int32 exactness bound
    assert ft(odd, 4, 4, 0, 0, good2, big, None) == EINVAL           # misaligned filters
    assert ft(good, 4, 4, 0, 0, p(0x20010), big, None) == EINVAL     # misaligned blob
    assert ft(good, 4, 4, 0, 0, good2, 100, None) == ESMALLBUF

    conv = lib.winograd_conv2d_int8
    args = dict(N=1, C=4, H=8, W=8, K=4)
    ws_bytes = wg.workspace_bytes(1, 4, 8, 8, 4, 0)

    def call(x=good, blob=good2, y=good3, N=1, C=4, H=8, W=8, K=4, layout=0, mode=0, ws=p(0x40000), wsb=ws_bytes):
        return conv(x, blob, y, N, C, H, W, K, layout, mode, ws, wsb, None)

    assert call(x=None) == EINVAL and call(blob=None) == EINVAL and call(y=None) == EINVAL and call(ws=None) == EINVAL
    assert call(N=0) == EINVAL and call(H=-3) == EINVAL and call(K=0) == EINVAL
    assert call(layout=5) == EINVAL and call(mode=-1) == EINVAL
    assert call(C=1000) == EUNSUPPORTED
    assert call(N=1 << 20, H=1 << 10, W=1 << 10) == EUNSUPPORTED      # beyond 32-bit indexing
    assert call(wsb=ws_bytes - 1) == ESMALLBUF
    assert call(x=odd) == EINVAL and call(ws=p(0x40010)) == EINVAL

    direct = lib.direct_conv2d_int8
    assert direct(None, good, good2, 1, 4, 8, 8, 4, 0, None) == EINVAL
    assert direct(good, good2, good3, 1, 4, 8, 8, 4, 3, None) == EINVAL
    assert direct(good, good2, good3, 1, 900, 8, 8, 4, 0, None) == EUNSUPPORTED

    rq = lib.requant_relu_pool_int8
    assert rq(None, good, 1, 4, 8, 8, 0, 3, 1, 0, None) == EINVAL
    assert rq(good, good2, 1, 4, 8, 8, 0, 32, 1, 0, None) == EINVAL   # shift out of range
    assert rq(good, good2, 1, 4, 7, 8, 0, 3, 1, 1, None) == EUNSUPPORTED   # odd H with pooling

    cq = lib.winograd_conv2d_int8_requant
    assert cq(good, good2, None, 1, 4, 8, 8, 4, 0, 0, 3, 1, 0, None) == EINVAL
    assert cq(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, -1, 1, 0, None) == EINVAL     # shift out of range
    assert cq(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, 32, 1, 0, None) == EINVAL
    assert cq(good, good2, good3, 1, 4, 8, 8, 4, 0, 2, 3, 1, 0, None) == EINVAL      # unknown mode
    assert cq(good, good2, odd, 1, 4, 8, 8, 4, 0, 0, 3, 1, 0, None) == EINVAL        # misaligned output
    assert cq(good, good2, good3, 1, 4, 8, 7, 4, 0, 0, 3, 1, 1, None) == EUNSUPPORTED   # odd W with pooling
    assert cq(good, good2, good3, 1, 1000, 8, 8, 4, 0, 0, 3, 1, 0, None) == EUNSUPPORTED

    # rational F(2x2,3x3) entry points
    assert lib.winograd_f2x2_packed_filter_bytes(0, 4, 0) == 0 and lib.winograd_f2x2_packed_filter_bytes(4, 4, 5) == 0
    f2_bytes = lib.winograd_f2x2_packed_filter_bytes(4, 4, 0)
    assert f2_bytes > 32 * 64 * 64 and f2_bytes % 256 == 0
    assert lib.winograd_f2x2_packed_filter_bytes(4, 4, 1) < f2_bytes          # one operand plane per entry instead of two
    f2t = lib.winograd_f2x2_filter_transform
    assert f2t(None, 4, 4, 0, 0, good2, f2_bytes, None) == EINVAL
    assert f2t(good, 4, 4, 0, 0, good2, f2_bytes - 1, None) == ESMALLBUF
    assert f2t(good, 4, 1000, 0, 0, good2, big, None) == EUNSUPPORTED
    assert f2t(good, 4, 4, 0, 0, p(0x20010), big, None) == EINVAL             # misaligned blob
    f2c = lib.winograd_f2x2_conv2d_int8
    assert f2c(good, good2, None, 1, 4, 8, 8, 4, 0, 0, None) == EINVAL
    assert f2c(good, good2, good3, 1, 4, 8, 8, 4, 7, 0, None) == EINVAL       # unknown layout
    assert f2c(good, good2, good3, 0, 4, 8, 8, 4, 0, 0, None) == EINVAL
    assert f2c(odd, good2, good3, 1, 4, 8, 8, 4, 0, 0, None) == EINVAL
    assert f2c(good, good2, good3, 1, 1000, 8, 8, 4, 0, 0, None) == EUNSUPPORTED
    assert lib.winograd_f2x2_debug_filter_operands(good2, 4, 4, 0, None, good3, None) == EINVAL
    f2tu, f2cu = lib.winograd_f2x2_filter_transform_u8, lib.winograd_f2x2_conv2d_u8
    assert f2tu(good, 256, 4, 4, 0, 0, good2, f2_bytes, None) == EINVAL      # zero point beyond a byte
    assert f2tu(good, -1, 4, 4, 0, 0, good2, f2_bytes, None) == EINVAL
    assert f2tu(None, 3, 4, 4, 0, 0, good2, f2_bytes, None) == EINVAL
    assert f2cu(good, 300, good2, good3, 1, 4, 8, 8, 4, 0, 0, None) == EINVAL
    assert f2cu(good, 3, good2, None, 1, 4, 8, 8, 4, 0, 0, None) == EINVAL
    f2q = lib.winograd_f2x2_conv2d_int8_requant
    assert f2q(good, good2, None, 1, 4, 8, 8, 4, 0, 0, 3, 1, 0, None) == EINVAL
    assert f2q(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, 32, 1, 0, None) == EINVAL        # shift out of range
    assert f2q(good, good2, good3, 1, 4, 8, 8, 4, 0, 2, 3, 1, 0, None) == EINVAL         # unknown mode
    assert f2q(good, good2, good3, 1, 4, 8, 7, 4, 0, 0, 3, 1, 1, None) == EUNSUPPORTED   # odd W with pooling
    f2a = lib.winograd_f2x2_conv2d_int8_act_scaled
    assert f2a(good, good2, None, 1, 4, 8, 8, 4, 0, None, None) == EINVAL
    assert f2a(good, None, good3, 1, 4, 8, 8, 4, 0, None, None) == EINVAL
    assert f2a(good, good2, good3, 1, 4, 8, 8, 4, 9, None, None) == EINVAL       # unknown layout
    assert f2a(good, good2, good3, 1, 4, 8, 8, 4, 0, odd, None) == EINVAL        # misaligned table export
    assert f2a(good, good2, good3, 1, 1000, 8, 8, 4, 0, None, None) == EUNSUPPORTED

    st = lib.winograd_conv2d_int8_enqueue_stage
    assert st(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, p(0x40000), ws_bytes, None, 0, 0) == EINVAL    # iters < 1
    assert st(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, p(0x40000), ws_bytes, None, 4, 1) == EINVAL    # unknown stage
    assert st(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, None, ws_bytes, None, 0, 1) == EINVAL          # no workspace
    assert st(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, p(0x40000), ws_bytes - 1, None, 0, 1) == ESMALLBUF
    assert lib.winograd_packed_filter_check(None, 4, 4, 0, None) == EINVAL
    assert lib.winograd_debug_input_operands(None, good, 1, 4, 8, 8, 0, 0, good2, big, None) == EINVAL
    assert lib.winograd_debug_filter_operands(good2, 4, 4, 3, good, good3, None) == EINVAL
    assert lib.winograd_debug_contraction(good, good2, good3, 1, 4, 8, 8, 4, 0, 0, None, big, None) == EINVAL


def test_binding_refuses_cpu_tensors(lib):
    import torch
    x = torch.zeros((1, 4, 8, 8), dtype=torch.int8)
    with pytest.raises(TypeError):
        wg.direct_conv2d_int8(x, torch.zeros((4, 4, 3, 3), dtype=torch.int8))


def test_vgg_shift_constants_match_the_generated_fixture():
    with open(os.path.join(ROOT, "tests", "golden", "vgg16_shifts.txt")) as f:
        line = [l for l in f if not l.startswith("#")][0]
    assert [int(t) for t in line.split()] == wl.VGG16_SHIFTS


def test_tile_decode_by_multiply_and_shift_matches_division(lib):
    """The kernels split a tile index with precomputed multiply-and-shift constants; compare with divmod
    over awkward tile grids, at the ends of every row and image."""
    out = (ctypes.c_int * 3)()
    shapes = [(1, 1, 1), (3, 4, 4), (5, 9, 7), (2, 56, 56), (16, 224, 224), (7, 13, 1021), (4000, 29, 31),
              (1, 4093, 4099), (65536, 8, 8)]
    for N, H, W in shapes:
        TH, TW = (H + 3) // 4, (W + 3) // 4
        T = N * TH * TW
        picks = {0, T - 1, T // 2, TW - 1, TW, TH * TW - 1, TH * TW, T - TW, max(0, T - TH * TW - 1)}
        picks |= {(i * 2654435761) % T for i in range(200)}
        for t in sorted(x for x in picks if 0 <= x < T):
            assert lib.winograd_debug_tile_decode(N, 4, H, W, 4, t, out) == 0
            n, rem = divmod(t, TH * TW)
            ty, tx = divmod(rem, TW)
            assert (out[0], out[1], out[2]) == (n, ty, tx), (N, H, W, t)
    assert lib.winograd_debug_tile_decode(1, 4, 8, 8, 4, 4, out) == EINVAL      # only 4 tiles


def _f2_fast_offsets_hold(N, C, H, W):
    """The F(2x2,3x3) fast kernel's load offsets in exact integers: a pixel's whole offset (vector part plus scalar part) from a
    base one row and one pixel before the tensor has to stay inside the descriptor's range, which is at most 2^31 bytes,
    and the scalar part is a signed 32-bit number."""
    before = (W + 1) * C
    farthest = (3 * W + 3) * C + (C - 1) // 64 * 64        # scalar part: patch pixel (3, 3), last channel block
    last = N * H * W * C - 4 + before                      # the last four channels of the tensor
    return farthest < 2 ** 31 and last + 4 <= min(N * H * W * C + before, 2 ** 31)


@pytest.mark.parametrize("N,C,H,W", [
    (1, 512, 1, 3_000_000), (1, 512, 1, 2_097_150), (1, 512, 1, 2_097_152), (1, 512, 1, 1_048_574), (1, 512, 1, 1_048_577),
    (2, 512, 1, 1_398_101), (1, 64, 3, 11_184_810), (1, 896, 2, 1_198_371), (1, 16, 1, 60_000_000), (37, 512, 336, 336), (38, 512, 332, 332),
    (1, 16, 1, 1), (8, 64, 56, 56), (256, 64, 112, 112)])
def test_f2x2_fast_kernel_only_where_its_offsets_hold(lib, N, C, H, W):
    K = 1
    route = lib.winograd_f2x2_debug_route
    assert N * C * H * W < 2 ** 31
    got = route(N, C, H, W, K, wg.NHWC, 0)
    assert got in (0, 1)
    if got == 1:
        assert _f2_fast_offsets_hold(N, C, H, W)
    else:   # what is turned away is large: nothing ordinary loses the fast kernel
        assert N * H * W * C + 4 * (W + 1) * C > 2 ** 31
    for layout, channels in ((wg.NCHW, C), (wg.NCHW, C - 1), (wg.NHWC, C - 1)):
        padded = 4 if channels <= 4 else (channels + 15) // 16 * 16
        with_memory, without = route(N, channels, H, W, K, layout, 1), route(N, channels, H, W, K, layout, 0)
        assert without == 0 and with_memory in (0, 2)
        if with_memory == 2:
            assert N * H * W * padded < 2 ** 31 and _f2_fast_offsets_hold(N, padded, H, W)
    assert route(N, C, H, W, K, 7, 0) == EINVAL and route(0, C, H, W, K, 0, 0) == EINVAL


@pytest.mark.parametrize("hook,value,modes", [
    ("lossless_variant", 1, (wg.LOSSLESS,)), ("lossless_variant", 2, (wg.LOSSLESS,)), ("scaled_variant", 1, (0, 1)), ("scaled_variant", 2, (0, 1)),
    ("stream_variant", 1, (0, 1)), ("stream_variant", 2, (0, 1)), ("stream_variant", 3, (0, 1)), ("stream_workgroups", 2, (0, 1))])
def test_a_forced_form_runs_in_one_kernel(lib, hook, value, modes):
    """The channel blocks of a deep layer with few tiles are dealt to several workgroups, which takes scratch memory; a test
    hook that asks for a form, or for never the limb-pair form (which the lossless split is), gets one kernel without."""
    wanted = lib._ZN2wg20conv2d_scratch_bytesEiiiiiiii    # what the extension asks before such a call
    wanted.restype, wanted.argtypes = ctypes.c_size_t, [ctypes.c_int] * 8
    sizes = lambda: [wanted(1, 512, 14, 14, 64, wg.NHWC, mode, 0) for mode in (wg.LOSSLESS, wg.SCALED)]
    by_itself = sizes()
    assert min(by_itself) > 0
    try:
        getattr(binding, hook)(value)
        forced = sizes()
    finally:
        getattr(binding, hook)(0)
    assert forced == [0 if mode in modes else by_itself[mode] for mode in (wg.LOSSLESS, wg.SCALED)]
    assert sizes() == by_itself


@pytest.mark.parametrize("N,C,K,HW,splits", [
    # channel blocks dealt to this many workgroups (lossless, scaled); 1: one kernel
    (1, 512, 512, 14, (8, 8)), (1, 512, 512, 28, (4, 1)), (4, 512, 512, 14, (4, 1)), (1, 256, 256, 56, (1, 1)), (2, 256, 512, 28, (1, 1)),
    (1, 256, 512, 28, (4, 1)), (4, 820, 250, 14, (7, 7)), (2, 324, 512, 28, (1, 1)), (1, 128, 64, 14, (1, 1)), (8, 512, 512, 28, (1, 1)),
    (1, 176, 64, 8, (3, 1))])
def test_which_layers_deal_their_channel_blocks_to_several_workgroups(lib, N, C, K, HW, splits):
    """The scratch memory that the extension asks for holds the splits' partial sums: 16 outputs (lossless) or 36 channel sums
    (scaled) per tile and filter, tiles padded to 16 and filters to 64."""
    wanted = lib._ZN2wg20conv2d_scratch_bytesEiiiiiiii
    wanted.restype, wanted.argtypes = ctypes.c_size_t, [ctypes.c_int] * 8
    tiles = (N * ((HW + 3) // 4) ** 2 + 15) // 16 * 16
    for mode, sums in ((wg.LOSSLESS, 16), (wg.SCALED, 36)):
        per_split = sums * tiles * ((K + 63) // 64 * 64) * 4
        assert wanted(N, C, HW, HW, K, wg.NHWC, mode, 0) == (0 if splits[mode] == 1 else splits[mode] * per_split), mode


@pytest.mark.parametrize("N,C,K,H,W", [(3, 224, 32, 82, 98), (59, 208, 48, 16, 16), (2, 196, 92, 63, 63), (5, 193, 56, 39, 74)])
def test_channel_major_layers_that_are_split_are_not_copied(lib, N, C, K, H, W):
    """Up to two channel blocks per workgroup: the scratch memory is the splits' sums and no channels-last copy, with which these took
    up to a quarter longer."""
    wanted = lib._ZN2wg20conv2d_scratch_bytesEiiiiiiii
    wanted.restype, wanted.argtypes = ctypes.c_size_t, [ctypes.c_int] * 8
    tiles = (N * ((H + 3) // 4) * ((W + 3) // 4) + 15) // 16 * 16
    per_split = 16 * tiles * ((K + 63) // 64 * 64) * 4
    assert wanted(N, C, H, W, K, wg.NCHW, wg.LOSSLESS, 0) == 2 * per_split


@pytest.mark.parametrize("mode,int8_out,most", [(wg.SCALED, True, 64), (wg.SCALED, False, 70), (wg.LOSSLESS, True, 128), (wg.LOSSLESS, False, 1999)])
def test_first_layers_of_few_tiles_stay_on_the_vector_alu(lib, mode, int8_out, most):
    """Groups of 16 tiles x 64 filters up to which the one-wave kernel takes a first layer: where it measured faster (scaled, 64 groups
    7.3 us against 7.7)."""
    takes = lib._ZN2wg22narrow_on_matrix_coresEiiib
    takes.restype, takes.argtypes = ctypes.c_bool, [ctypes.c_int] * 3 + [ctypes.c_bool]
    for filter_blocks in (1, 2, 3):
        groups = most // filter_blocks
        assert not takes(16 * groups, 64 * filter_blocks, mode, int8_out)
        assert takes(16 * groups + 1, 64 * filter_blocks, mode, int8_out)
    try:
        for variant in (1, 2):
            binding.narrow_variant(variant)
            assert [takes(t, 64, mode, int8_out) for t in (1, 10 ** 6)] == [variant == 1] * 2
    finally:
        binding.narrow_variant(0)
    assert lib.winograd_debug_narrow_variant(3) == EINVAL and lib.winograd_debug_narrow_variant(-1) == EINVAL
