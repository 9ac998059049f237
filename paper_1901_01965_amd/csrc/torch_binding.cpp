// CPython extension over the C ABI: takes torch tensors, checks them, allocates outputs from torch's caching allocator
// and enqueues on torch's current stream.  A convolution of the smaller layers takes 5 to 15 us on the GPU, which is
// what marshalling the same call through ctypes cost the interpreter (12 us); through here a call costs about 4 us, most
// of it the launch itself.  No arithmetic lives here.
//
// Every function takes positional arguments only (binding.py keeps the public signatures) and returns the output tensor,
// or the C ABI's negative status as an int, which binding.py turns into WinogradError.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "host_api.h"

namespace {

struct PyError {};   // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw PyError();
}

const char* type_name(at::ScalarType t) {
    return t == at::kChar ? "torch.int8" : t == at::kByte ? "torch.uint8" : "torch.int32";
}

const at::Tensor& tensor(PyObject* o, at::ScalarType dtype, const char* what) {
    if (THPVariable_Check(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.scalar_type() == dtype && t.is_contiguous()) return t;
    }
    PyErr_Format(PyExc_TypeError, "%s must be a contiguous CUDA tensor of %s", what, type_name(dtype));
    throw PyError();
}

template <class T>
T* data(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }

int integer(PyObject* o) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyError();
    if (v != (int)v) fail(PyExc_OverflowError, "integer argument out of range");
    return (int)v;
}

struct Dims {
    int N, C, H, W;
};
Dims dims(const at::Tensor& x, int layout) {
    if (x.dim() != 4) fail(PyExc_ValueError, "activations and outputs have four dimensions");
    for (int i = 0; i < 4; ++i)
        if (x.size(i) > 0x7fffffff) fail(PyExc_ValueError, "dimension too large");
    const int a = (int)x.size(1), b = (int)x.size(2), c = (int)x.size(3);
    return layout == WG_NCHW ? Dims{(int)x.size(0), a, b, c} : Dims{(int)x.size(0), c, a, b};
}

// A fresh output tensor, or the caller's after a check of its shape, type and contiguity: a kernel writes every element
// of the shape wherever the pointer leads.
at::Tensor output(PyObject* out, int N, int K, int H, int W, int layout, at::ScalarType dtype, const at::Tensor& like) {
    const int64_t nchw[4] = {N, K, H, W}, nhwc[4] = {N, H, W, K};
    const at::IntArrayRef shape(layout == WG_NCHW ? nchw : nhwc, 4);
    if (out == Py_None) return at::Tensor(at::detail::empty_cuda(shape, dtype, like.device(), std::nullopt));
    const at::Tensor& t = tensor(out, dtype, "out");
    if (t.sizes() != shape) {
        PyErr_Format(PyExc_ValueError, "out has another shape than the call writes, (%d, %d, %d, %d)", (int)shape[0], (int)shape[1],
                     (int)shape[2], (int)shape[3]);
        throw PyError();
    }
    return t;
}

// Scratch memory of one call, from torch's caching allocator (which hands it out again only to work queued behind it).
// Where it only makes the call faster (`needed` false), a device without room for it leaves the call without.
struct ScratchTensor {
    at::Tensor t;
    void* p = nullptr;
    size_t bytes = 0;
    ScratchTensor(size_t wanted, const at::Tensor& like, bool needed = false) {
        if (wanted == 0) return;
        try {
            t = at::Tensor(at::detail::empty_cuda({(int64_t)wanted}, at::kByte, like.device(), std::nullopt));
        } catch (const c10::OutOfMemoryError&) {
            if (needed) throw;
            return;
        }
        p = t.data_ptr();
        bytes = wanted;
    }
};

void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

void need_channels(int packed_for, int C, const char* what) {
    if (packed_for == C) return;
    PyErr_Format(PyExc_ValueError, "%s: the filters were packed for C = %d, the activations have C = %d", what, packed_for, C);
    throw PyError();
}

// The interpreter lock given up for as long as one of these lives, also when an exception ends that.
struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// The enqueueing call itself runs without the interpreter lock, like a ctypes call.  It is given plain pointers: asking a
// tensor for its data can throw (a vmap batch, a wrapper subclass: tensors without storage), and a call that is refused for
// that is refused before anything is allocated or asked of the device.
template <class F>
PyObject* finish(const at::Tensor& y, F&& enqueue) {
    int status;
    {
        const Unlocked unlocked;
        status = enqueue();
    }
    return status == WG_OK ? THPVariable_Wrap(y) : PyLong_FromLong(status);
}

template <class F>
PyObject* guarded(Py_ssize_t got, Py_ssize_t want, F&& body) {
    if (got != want) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        return body();
    } catch (const PyError&) {
        return nullptr;
    } catch (...) {   // torch's own errors become the Python exceptions that torch's functions raise for them
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

// (x, blob, K, C, mode, layout, out, workspace)
PyObject* conv2d_int8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 8, [&]() -> PyObject* {
        const int K = integer(a[2]), packed_c = integer(a[3]), mode = integer(a[4]), layout = integer(a[5]);
        const at::Tensor& x = tensor(a[0], at::kChar, "x");
        const Dims d = dims(x, layout);
        need_channels(packed_c, d.C, "winograd_conv2d_int8");
        const int8_t* const xp = data<int8_t>(x);
        const void* const blob = data<void>(tensor(a[1], at::kByte, "blob"));
        void* given = nullptr;   // a caller's workspace
        size_t given_bytes = 0;
        if (a[7] != Py_None) {
            const at::Tensor& t = tensor(a[7], at::kByte, "workspace");
            given = data<void>(t);
            given_bytes = (size_t)t.numel();
        }
        const at::Tensor y = output(a[6], d.N, K, d.H, d.W, layout, at::kInt, x);
        int32_t* const yp = data<int32_t>(y);
        void* const s = stream();
        // the staged pipeline, or a caller's workspace: the C ABI's entry point
        const bool staged = a[7] == Py_None && winograd_conv2d_path(d.N, d.C, d.H, d.W, K, mode) == 1;
        if (staged || a[7] != Py_None) {
            const ScratchTensor own(staged ? winograd_workspace_bytes(d.N, d.C, d.H, d.W, K, mode) : 0, x, true);
            void* const ws = staged ? own.p : given;
            const size_t ws_bytes = staged ? own.bytes : given_bytes;
            return finish(y, [&] { return winograd_conv2d_int8(xp, blob, yp, d.N, d.C, d.H, d.W, K, layout, mode, ws, ws_bytes, s); });
        }
        const ScratchTensor scratch(wg::conv2d_scratch_bytes(d.N, d.C, d.H, d.W, K, layout, mode, 0), x);
        return finish(y, [&] {
            return wg::conv2d_int8_with_scratch(xp, blob, yp, d.N, d.C, d.H, d.W, K, layout, mode, scratch.p, scratch.bytes, s);
        });
    });
}

// (x, blob, K, C, mode, layout, out, shift, relu, pool, f2x2)
PyObject* conv2d_int8_requant(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 11, [&]() -> PyObject* {
        const int K = integer(a[2]), packed_c = integer(a[3]), mode = integer(a[4]), layout = integer(a[5]);
        const int shift = integer(a[7]), relu = integer(a[8]), pool = integer(a[9]), f2x2 = integer(a[10]);
        const at::Tensor& x = tensor(a[0], at::kChar, "x");
        const Dims d = dims(x, layout);
        need_channels(packed_c, d.C, f2x2 ? "f2x2_conv2d_int8_requant" : "winograd_conv2d_int8_requant");
        const int8_t* const xp = data<int8_t>(x);
        const void* const blob = data<void>(tensor(a[1], at::kByte, "blob"));
        const at::Tensor y = output(a[6], d.N, K, pool ? d.H / 2 : d.H, pool ? d.W / 2 : d.W, layout, at::kChar, x);
        int8_t* const yp = data<int8_t>(y);
        void* const s = stream();
        const ScratchTensor scratch(f2x2 ? wg::f2x2_conv2d_scratch_bytes(d.N, d.C, d.H, d.W, K, layout)
                                         : wg::conv2d_scratch_bytes(d.N, d.C, d.H, d.W, K, layout, mode, 0), x);
        return finish(y, [&] {
            if (f2x2)
                return wg::f2x2_conv2d_int8_requant_with_scratch(xp, blob, yp, d.N, d.C, d.H, d.W, K, layout, mode, shift, relu, pool,
                                                                 scratch.p, scratch.bytes, s);
            return wg::conv2d_int8_requant_with_scratch(xp, blob, yp, d.N, d.C, d.H, d.W, K, layout, mode, shift, relu, pool, scratch.p,
                                                        scratch.bytes, s);
        });
    });
}

// (x, zero_point or None, blob, K, C, mode, layout, out, f2x2): uint8 activations, or (F(2x2,3x3) only) int8 without a zero point
PyObject* conv2d_bytes(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 9, [&]() -> PyObject* {
        const bool is_unsigned = a[1] != Py_None;
        const int zero = is_unsigned ? integer(a[1]) : 0;
        const int K = integer(a[3]), packed_c = integer(a[4]), mode = integer(a[5]), layout = integer(a[6]), f2x2 = integer(a[8]);
        const at::Tensor& x = tensor(a[0], is_unsigned ? at::kByte : at::kChar, "x");
        const Dims d = dims(x, layout);
        need_channels(packed_c, d.C, f2x2 ? "f2x2_conv2d_int8" : "winograd_conv2d_u8");
        const void* const xp = data<void>(x);
        const void* const blob = data<void>(tensor(a[2], at::kByte, "blob"));
        const at::Tensor y = output(a[7], d.N, K, d.H, d.W, layout, at::kInt, x);
        int32_t* const yp = data<int32_t>(y);
        void* const s = stream();
        const ScratchTensor scratch(f2x2 ? wg::f2x2_conv2d_scratch_bytes(d.N, d.C, d.H, d.W, K, layout)
                                         : wg::conv2d_scratch_bytes(d.N, d.C, d.H, d.W, K, layout, mode, 1), x);
        return finish(y, [&] {
            if (f2x2)
                return wg::f2x2_conv2d_with_scratch(xp, is_unsigned, zero, blob, yp, d.N, d.C, d.H, d.W, K, layout, mode, scratch.p,
                                                    scratch.bytes, s);
            return wg::conv2d_u8_with_scratch(static_cast<const uint8_t*>(xp), zero, blob, yp, d.N, d.C, d.H, d.W, K, layout, mode, scratch.p,
                                              scratch.bytes, s);
        });
    });
}

// (x, blob, K, C, layout, out, table or None, f2x2)
PyObject* conv2d_act_scaled(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 8, [&]() -> PyObject* {
        const int K = integer(a[2]), packed_c = integer(a[3]), layout = integer(a[4]), f2x2 = integer(a[7]);
        const at::Tensor& x = tensor(a[0], at::kChar, "x");
        const Dims d = dims(x, layout);
        need_channels(packed_c, d.C, f2x2 ? "f2x2_conv2d_int8_act_scaled" : "winograd_conv2d_int8_act_scaled");
        const int8_t* const xp = data<int8_t>(x);
        const void* const blob = data<void>(tensor(a[1], at::kByte, "blob"));
        int32_t* const table = a[6] == Py_None ? nullptr : data<int32_t>(tensor(a[6], at::kInt, "table"));
        const at::Tensor y = output(a[5], d.N, K, d.H, d.W, layout, at::kInt, x);
        int32_t* const yp = data<int32_t>(y);
        void* const s = stream();
        const ScratchTensor scratch(f2x2 ? 0 : wg::act_scaled_scratch_bytes(d.N, d.C, d.H, d.W, K, layout), x);
        return finish(y, [&] {
            if (f2x2)
                return winograd_f2x2_conv2d_int8_act_scaled(xp, blob, yp, d.N, d.C, d.H, d.W, K, layout, table, s);
            return wg::conv2d_int8_act_scaled_with_scratch(xp, blob, yp, d.N, d.C, d.H, d.W, K, layout, table, scratch.p, scratch.bytes, s);
        });
    });
}

// (x, w, layout, out)
PyObject* direct_conv2d(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 4, [&]() -> PyObject* {
        const int layout = integer(a[2]);
        const at::Tensor &x = tensor(a[0], at::kChar, "x"), &w = tensor(a[1], at::kChar, "w");
        const Dims d = dims(x, layout);
        const bool fits = w.dim() == 4 && (layout == WG_NCHW ? w.size(1) == d.C && w.size(2) == 3 && w.size(3) == 3
                                                             : w.size(1) == 3 && w.size(2) == 3 && w.size(3) == d.C);
        if (!fits || w.size(0) > 0x7fffffff) {
            PyErr_Format(PyExc_ValueError, "w does not have the shape of 3x3 filters for activations with C = %d", d.C);
            throw PyError();
        }
        const int K = (int)w.size(0);
        const int8_t *const xp = data<int8_t>(x), *const wp = data<int8_t>(w);
        const at::Tensor y = output(a[3], d.N, K, d.H, d.W, layout, at::kInt, x);
        int32_t* const yp = data<int32_t>(y);
        void* const s = stream();
        const ScratchTensor scratch(wg::direct_conv2d_scratch_bytes(d.N, d.C, d.H, d.W, K, layout), x);
        return finish(y, [&] {
            return wg::direct_conv2d_with_scratch(xp, wp, yp, d.N, d.C, d.H, d.W, K, layout, scratch.p, scratch.bytes, s);
        });
    });
}

// (y, layout, out, shift, relu, pool)
PyObject* requant_relu_pool(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 6, [&]() -> PyObject* {
        const int layout = integer(a[1]), shift = integer(a[3]), relu = integer(a[4]), pool = integer(a[5]);
        const at::Tensor& y = tensor(a[0], at::kInt, "y");
        const Dims d = dims(y, layout);
        const int32_t* const yp = data<int32_t>(y);
        const at::Tensor out = output(a[2], d.N, d.C, pool ? d.H / 2 : d.H, pool ? d.W / 2 : d.W, layout, at::kChar, y);
        int8_t* const op = data<int8_t>(out);
        void* const s = stream();
        return finish(out, [&] {
            return requant_relu_pool_int8(yp, op, d.N, d.C, d.H, d.W, layout, shift, relu, pool, s);
        });
    });
}

#define WG_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {WG_METHOD(conv2d_int8),   WG_METHOD(conv2d_int8_requant), WG_METHOD(conv2d_bytes), WG_METHOD(conv2d_act_scaled),
                         WG_METHOD(direct_conv2d), WG_METHOD(requant_relu_pool),   {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_winograd_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__winograd_torch() { return PyModule_Create(&module); }
