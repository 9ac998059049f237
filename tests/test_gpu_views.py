"""Operands and outputs that are views into larger buffers, 4, 8 and 12 bytes after a 16-byte boundary, through every call:
the same results as with tensors of their own, and nothing written beside the output."""
import pytest
import torch

import paper_1901_01965_amd as wg

pytestmark = pytest.mark.gpu

CANARY = 86


def _at(t, offset):
    """t's values in a view that starts `offset` bytes after a 16-byte boundary."""
    buffer = torch.zeros(t.numel() * t.element_size() + 64, dtype=torch.uint8, device="cuda")
    view = buffer[offset:offset + t.numel() * t.element_size()].view(t.dtype).view(t.shape)
    assert view.data_ptr() % 16 == offset
    view.copy_(t)
    return view


# channel blocks dealt to several workgroups; 16-byte pieces where aligned; 4-byte pieces; neither; few channels; one that streams
SHAPES = [(1, 512, 40, 14, 14), (2, 64, 64, 18, 22), (2, 100, 76, 10, 10), (1, 67, 33, 8, 6), (2, 3, 20, 12, 10), (24, 64, 64, 56, 56)]


@pytest.mark.parametrize("offset", [4, 8, 12])
@pytest.mark.parametrize("layout", [wg.NHWC, wg.NCHW])
@pytest.mark.parametrize("shape", SHAPES)
def test_views_give_the_same_results(shape, layout, offset):
    N, C, K, H, W = shape
    nhwc = layout == wg.NHWC
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    x = torch.randint(-128, 128, (N, H, W, C) if nhwc else (N, C, H, W), dtype=torch.int8, device="cuda", generator=gen)
    w = torch.randint(-128, 128, (K, 3, 3, C) if nhwc else (K, C, 3, 3), dtype=torch.int8, device="cuda", generator=gen)
    xv, wv = _at(x, offset), _at(w, offset)
    u8, u8v = x.view(torch.uint8), xv.view(torch.uint8)
    calls = []
    for mode in (wg.LOSSLESS, wg.SCALED):
        packed, f2 = wg.winograd_filter_transform(wv, layout, mode), wg.f2x2_filter_transform(wv, layout, mode)
        assert torch.equal(packed.blob, wg.winograd_filter_transform(w, layout, mode).blob)
        assert torch.equal(f2.blob, wg.f2x2_filter_transform(w, layout, mode).blob)
        calls += [(x, xv, lambda a, out, p=packed: wg.winograd_conv2d_int8(a, p, layout, out=out)),
                  (x, xv, lambda a, out, p=packed: wg.winograd_conv2d_int8_requant(a, p, 10, False, False, layout, out=out)),
                  (x, xv, lambda a, out, p=packed: wg.winograd_conv2d_int8_requant(a, p, 10, True, True, layout, out=out)),
                  (x, xv, lambda a, out, p=f2: wg.f2x2_conv2d_int8(a, p, layout, out=out)),
                  (u8, u8v, lambda a, out, p=f2: wg.f2x2_conv2d_int8(a, p, layout, out=out, zero_point=33)),
                  (x, xv, lambda a, out, p=f2: wg.f2x2_conv2d_int8_requant(a, p, 10, True, True, layout, out=out))]
        if C <= wg.MAX_CHANNELS_U8:
            p8 = wg.winograd_filter_transform_u8(wv.view(torch.uint8), 140, layout, mode)
            calls.append((u8, u8v, lambda a, out, p=p8: wg.winograd_conv2d_u8(a, 33, p, layout, out=out)))
    calls += [(x, xv, lambda a, out, p=packed: wg.winograd_conv2d_int8_act_scaled(a, p, layout, out=out)),
              (x, xv, lambda a, out, p=f2: wg.f2x2_conv2d_int8_act_scaled(a, p, layout, out=out)),
              (x, xv, lambda a, out: wg.direct_conv2d_int8(a, w if a is x else wv, layout, out=out))]
    y = wg.direct_conv2d_int8(x, w, layout)
    calls += [(y, _at(y, offset), lambda a, out, pool=pool: wg.requant_relu_pool_int8(a, 10, True, pool, layout, out=out)) for pool in (False, True)]
    for i, (own, view, call) in enumerate(calls):
        want = call(own, None)
        size = want.numel() * want.element_size()
        buffer = torch.full((size + 64,), CANARY, dtype=torch.uint8, device="cuda")
        out = buffer[offset:offset + size].view(want.dtype).view(want.shape)
        call(view, out)
        assert torch.equal(out, want), i
        assert bool((buffer[:offset] == CANARY).all()) and bool((buffer[offset + size:] == CANARY).all()), i
