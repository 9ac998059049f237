"""Host side of the CPython extension's calls, without a GPU: what a call does with tensors that look like GPU tensors but
have no storage."""
import threading

import pytest
import torch

import paper_1901_01965_amd as wg
from paper_1901_01965_amd import binding


class NoStorage(torch.Tensor):
    """A tensor that says it is on the GPU and holds nothing."""

    @staticmethod
    def __new__(cls, shape, dtype):
        return torch.Tensor._make_wrapper_subclass(cls, shape, dtype=dtype, device="cuda:0")

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise NotImplementedError(func)


def _gpu_like(shape, dtype):
    return NoStorage(shape, dtype)


I8, U8, I32, X, Y = torch.int8, torch.uint8, torch.int32, (1, 8, 8, 16), (1, 8, 8, 32)
BLOB = (U8, (4096,))
CALLS = {   # name: (arguments by role, call)
    "winograd_conv2d_int8": ({"x": (I8, X), "blob": BLOB, "out": (I32, Y)},
                             lambda x, blob, out: wg.winograd_conv2d_int8(x, wg.PackedFilter(blob, 32, 16, 0), wg.NHWC, out=out)),
    "winograd_conv2d_int8 with a workspace": (
        {"x": (I8, X), "blob": BLOB, "out": (I32, Y), "workspace": BLOB},
        lambda x, blob, out, workspace: wg.winograd_conv2d_int8(x, wg.PackedFilter(blob, 32, 16, 0), wg.NHWC, out=out, workspace=workspace)),
    "winograd_conv2d_int8_requant": (
        {"x": (I8, X), "blob": BLOB, "out": (I8, Y)},
        lambda x, blob, out: wg.winograd_conv2d_int8_requant(x, wg.PackedFilter(blob, 32, 16, 0), 8, layout=wg.NHWC, out=out)),
    "winograd_conv2d_u8": ({"x": (U8, X), "blob": BLOB, "out": (I32, Y)},
                           lambda x, blob, out: wg.winograd_conv2d_u8(x, 3, wg.PackedFilterU8(blob, 32, 16, 0), wg.NHWC, out=out)),
    "winograd_conv2d_int8_act_scaled": (
        {"x": (I8, X), "blob": BLOB, "out": (I32, Y)},
        lambda x, blob, out: wg.winograd_conv2d_int8_act_scaled(x, wg.PackedFilter(blob, 32, 16, 1), wg.NHWC, out=out)),
    "f2x2_conv2d_int8": ({"x": (I8, X), "blob": BLOB, "out": (I32, Y)},
                         lambda x, blob, out: wg.f2x2_conv2d_int8(x, wg.F2x2PackedFilter(blob, 32, 16, 0), wg.NHWC, out=out)),
    "direct_conv2d_int8": ({"x": (I8, X), "w": (I8, (32, 3, 3, 16)), "out": (I32, Y)},
                           lambda x, w, out: wg.direct_conv2d_int8(x, w, wg.NHWC, out=out)),
    "requant_relu_pool_int8": ({"y": (I32, Y), "out": (I8, Y)}, lambda y, out: wg.requant_relu_pool_int8(y, 8, layout=wg.NHWC, out=out)),
}


@pytest.mark.parametrize("name,role", [(n, r) for n, (roles, _) in CALLS.items() for r in roles])
def test_a_tensor_without_a_data_pointer_is_refused(name, role):
    """A vmap batch passes the checks of device, type and layout and has no data pointer.  Asking for one throws, which
    has to happen while the interpreter lock is held and before anything is asked of the device: a RuntimeError that says
    so, and an interpreter that goes on, in this thread and in another."""
    roles, call = CALLS[name]
    tensors = {r: _gpu_like(shape, dtype) for r, (dtype, shape) in roles.items()}
    dtype, shape = roles[role]
    binding._native()

    def body(batched):
        with pytest.raises(RuntimeError, match="data pointer"):
            call(**dict(tensors, **{role: batched}))
        return torch.zeros(1)

    torch.vmap(body)(_gpu_like((2,) + shape, dtype))
    ran = []
    t = threading.Thread(target=lambda: ran.append(sum(range(1000))))
    t.start()
    t.join()
    assert ran == [499500]
