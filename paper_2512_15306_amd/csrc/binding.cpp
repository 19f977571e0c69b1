// Python module _binding: the calls of a training step without ctypes.  A call of llmq.py takes 11.4 us on the host in
// ctypes with three launches, of which the launches are 7.8: the checks of nine tensors and the conversion of thirteen arguments in
// Python are most of the rest.  Here they are reads of the tensors' fields.
//
// Every function takes the arguments of its namesake in llmq.py and returns the library's status, or None for whatever is not the
// plain case (a tensor subclass, another type, layout, device or size, a number out of range): the caller then takes the ctypes
// path, which does or refuses what it always has.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <limits>
#include <optional>
#include <utility>

#include "../../include/llmq.h"

namespace {

PyObject *g_get_device, *g_get_stream;          // torch._C functions

constexpr at::ScalarType kBf16 = at::kBFloat16, kF32 = at::kFloat, kU8 = at::kByte;

// The arguments of one call; ok turns false at the first one that is not the plain case.
struct Args {
    PyObject* const* a;
    bool ok;

    const at::Tensor* tensor(int i, at::ScalarType type) {
        if (!THPVariable_CheckExact(a[i])) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(a[i]);
        if (!t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != type || !t.is_contiguous()) { ok = false; return nullptr; }
        return &t;
    }
    // Device pointer of a tensor or NULL for None; numel: how many elements it has to have (-1: any)
    template <class T>
    T* ptr(int i, at::ScalarType type, int64_t numel = -1) {
        if (a[i] == Py_None) return nullptr;
        const at::Tensor* t = tensor(i, type);
        if (!t) return nullptr;
        if (numel >= 0 && t->numel() != numel) { ok = false; return nullptr; }
        return static_cast<T*>(t->data_ptr());
    }
    void* bf16(int i, int64_t numel = -1) { return ptr<void>(i, kBf16, numel); }
    float* f32(int i, int64_t numel = -1) { return ptr<float>(i, kF32, numel); }
    uint8_t* u8(int i, int64_t numel = -1) { return ptr<uint8_t>(i, kU8, numel); }
    uint8_t* some_u8(int i, int64_t numel) {                     // not None
        if (a[i] == Py_None) ok = false;
        return ok ? u8(i, numel) : nullptr;
    }
    void* some_bf16(int i, int64_t numel) {
        if (a[i] == Py_None) ok = false;
        return ok ? bf16(i, numel) : nullptr;
    }
    float* some_f32(int i, int64_t numel) {
        if (a[i] == Py_None) ok = false;
        return ok ? f32(i, numel) : nullptr;
    }
    // A workspace and its size
    void* workspace(int i, size_t& bytes) {
        const at::Tensor* t = tensor(i, kU8);
        if (!t) return nullptr;
        bytes = (size_t)t->numel();
        return t->data_ptr();
    }
    // [rows, cols] of a matrix
    bool dims(int i, at::ScalarType type, int64_t& rows, int64_t& cols) {
        const at::Tensor* t = tensor(i, type);
        if (!t || t->dim() != 2) { ok = false; return false; }
        rows = t->size(0);
        cols = t->size(1);
        return true;
    }
    int64_t i64(int i) {
        if (!PyLong_CheckExact(a[i])) { ok = false; return 0; }
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(a[i], &over);
        if (over) ok = false;
        return v;
    }
    int i32(int i) {
        const int64_t v = i64(i);
        if (v < std::numeric_limits<int>::min() || v > std::numeric_limits<int>::max()) ok = false;
        return (int)v;
    }
    int truth(int i) {
        if (!PyLong_Check(a[i])) { ok = false; return 0; }       // bool or int
        return PyObject_IsTrue(a[i]) == 1;
    }
};

// The current device's current stream
bool current_stream(void** stream) {
    PyObject* dev = PyObject_CallNoArgs(g_get_device);
    if (!dev) return false;
    PyObject* s = PyObject_CallOneArg(g_get_stream, dev);
    Py_DECREF(dev);
    if (!s) return false;
    *stream = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !PyErr_Occurred();
}

// N arguments read by `read` into a call, which `read` returns: a callable that takes the stream
template <class Read>
auto read_arguments(PyObject* const* args, Read read) -> std::optional<decltype(read(std::declval<Args&>()))> {
    Args a{args, true};
    try {
        auto call = read(a);
        if (a.ok) return call;
    } catch (...) {                                              // a tensor without storage, say
    }
    return std::nullopt;
}
template <class Read>
PyObject* run(PyObject* const* args, Py_ssize_t n, Py_ssize_t want, Read read) {
    if (n != want) Py_RETURN_NONE;
    const auto call = read_arguments(args, read);
    if (!call) Py_RETURN_NONE;
    void* stream = nullptr;
    if (!current_stream(&stream)) return nullptr;
    int status = 0;
    Py_BEGIN_ALLOW_THREADS                                       // (as ctypes does: a launch may wait for room in the queue)
    status = (*call)(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

#define LLMQ_BINDING(name) PyObject* name(PyObject*, PyObject* const* args, Py_ssize_t n)

LLMQ_BINDING(linear_fwd) {
    return run(args, n, 11, [](Args& a) {
        size_t bytes = 0;
        void *X = a.bf16(0), *W = a.bf16(1);
        const int64_t M = a.i64(2), N = a.i64(3), K = a.i64(4);
        float *sx = a.f32(5), *sw = a.f32(6);
        void* Y = a.bf16(7);
        float* amax = a.f32(8);
        void* ws = a.workspace(9, bytes);
        const int flags = a.i32(10);
        return [=](void* s) { return llmq_fp8_linear_fwd(X, W, M, N, K, sx, sw, Y, amax, ws, bytes, flags, s); };
    });
}

LLMQ_BINDING(linear_dgrad) {
    return run(args, n, 12, [](Args& a) {
        size_t bytes = 0;
        void *dY = a.bf16(0), *W = a.bf16(1);
        const int64_t M = a.i64(2), N = a.i64(3), K = a.i64(4);
        float *sdy = a.f32(5), *sw = a.f32(6);
        const int fmt = a.i32(7);
        void* dX = a.bf16(8);
        float* amax = a.f32(9);
        void* ws = a.workspace(10, bytes);
        const int flags = a.i32(11);
        return [=](void* s) { return llmq_fp8_linear_dgrad(dY, W, M, N, K, sdy, sw, fmt, dX, amax, ws, bytes, flags, s); };
    });
}

LLMQ_BINDING(linear_wgrad) {
    return run(args, n, 12, [](Args& a) {
        size_t bytes = 0;
        void *dY = a.bf16(0), *X = a.bf16(1);
        const int64_t M = a.i64(2), N = a.i64(3), K = a.i64(4);
        float *sdy = a.f32(5), *sx = a.f32(6);
        const int fmt = a.i32(7);
        void* dW = a.bf16(8);
        const int accumulate = a.truth(9);
        void* ws = a.workspace(10, bytes);
        const int flags = a.i32(11);
        return [=](void* s) { return llmq_fp8_linear_wgrad(dY, X, M, N, K, sdy, sx, fmt, dW, accumulate, ws, bytes, flags, s); };
    });
}

LLMQ_BINDING(amax) {
    return run(args, n, 5, [](Args& a) {
        size_t bytes = 0;
        const at::Tensor* t = a.tensor(0, kBf16);
        const size_t count = t ? (size_t)t->numel() : 0;
        void* x = t ? t->data_ptr() : nullptr;
        const int fmt = a.i32(1);
        float *am = a.f32(2), *sc = a.f32(3);
        void* ws = a.workspace(4, bytes);
        return [=](void* s) { return llmq_amax(x, count, fmt, am, sc, ws, bytes, s); };
    });
}

template <bool SLABS>
PyObject* quantize(PyObject* const* args, Py_ssize_t n) {
    return run(args, n, 5, [](Args& a) {
        int64_t rows = 0, cols = 0;
        a.dims(0, kBf16, rows, cols);
        void* x = a.ok ? a.bf16(0) : nullptr;
        float* sc = a.f32(1);
        const int fmt = a.i32(2);
        uint8_t *q = a.some_u8(3, rows * cols), *qt = SLABS ? a.some_u8(4, rows * cols) : a.u8(4, rows * cols);
        return [=](void* s) { return SLABS ? llmq_quantize_fp8_slabs(x, rows, cols, sc, fmt, q, qt, s) : llmq_quantize_fp8(x, rows, cols, sc, fmt, q, qt, s); };
    });
}
LLMQ_BINDING(quantize_fp8) { return quantize<false>(args, n); }
LLMQ_BINDING(quantize_fp8_slabs) { return quantize<true>(args, n); }

LLMQ_BINDING(bf16_gemm_tn) {
    return run(args, n, 4, [](Args& a) {
        int64_t R = 0, T = 0, C = 0, T2 = 0, R2 = 0, C2 = 0;
        a.dims(0, kBf16, R, T);
        a.dims(1, kBf16, C, T2);
        a.dims(2, kBf16, R2, C2);
        if (T != T2 || R2 != R || C2 != C) a.ok = false;
        void *A = a.ok ? a.bf16(0) : nullptr, *B = a.ok ? a.bf16(1) : nullptr, *c = a.ok ? a.bf16(2) : nullptr;
        const int accumulate = a.truth(3);
        return [=](void* s) { return llmq_bf16_gemm_tn(A, B, R, C, T, c, accumulate, s); };
    });
}

// (M, I) of a gate + up tensor
void swiglu_dims(Args& a, int i, int64_t& M, int64_t& I) {
    if (a.dims(i, kBf16, M, I) && I % 2) a.ok = false;
    I /= 2;
}

LLMQ_BINDING(swiglu_fwd) {
    return run(args, n, 6, [](Args& a) {
        int64_t M = 0, I = 0;
        size_t bytes = 0;
        swiglu_dims(a, 0, M, I);
        void *gu = a.ok ? a.bf16(0) : nullptr, *h = a.some_bf16(1, M * I);
        const int fmt = a.i32(2);
        float *am = a.f32(3), *sc = a.f32(4);
        void* ws = a.workspace(5, bytes);
        return [=](void* s) { return llmq_swiglu_fwd(gu, M, I, h, fmt, am, sc, ws, bytes, s); };
    });
}

template <bool SLABS>
PyObject* swiglu_codes(PyObject* const* args, Py_ssize_t n) {
    return run(args, n, 6, [](Args& a) {
        int64_t M = 0, I = 0;
        swiglu_dims(a, 0, M, I);
        void* gu = a.ok ? a.bf16(0) : nullptr;
        float* sc = a.f32(1);
        const int fmt = a.i32(2);
        uint8_t *q = a.some_u8(3, M * I), *qt = SLABS ? a.some_u8(4, M * I) : a.u8(4, M * I);
        void* h = a.bf16(5, M * I);
        return [=](void* s) { return SLABS ? llmq_swiglu_fwd_fp8_slabs(gu, M, I, sc, fmt, q, qt, h, s) : llmq_swiglu_fwd_fp8(gu, M, I, sc, fmt, q, qt, h, s); };
    });
}
LLMQ_BINDING(swiglu_fwd_fp8) { return swiglu_codes<false>(args, n); }
LLMQ_BINDING(swiglu_fwd_fp8_slabs) { return swiglu_codes<true>(args, n); }

LLMQ_BINDING(swiglu_bwd) {
    return run(args, n, 7, [](Args& a) {
        int64_t M = 0, I = 0;
        size_t bytes = 0;
        swiglu_dims(a, 1, M, I);
        void *dh = a.some_bf16(0, M * I), *gu = a.ok ? a.bf16(1) : nullptr, *dgu = a.some_bf16(2, 2 * M * I);
        const int fmt = a.i32(3);
        float *am = a.f32(4), *sc = a.f32(5);
        void* ws = a.workspace(6, bytes);
        return [=](void* s) { return llmq_swiglu_bwd(dh, gu, M, I, dgu, fmt, am, sc, ws, bytes, s); };
    });
}

LLMQ_BINDING(rmsnorm_fwd) {
    return run(args, n, 11, [](Args& a) {
        int64_t M = 0, C = 0;
        size_t bytes = 0;
        a.dims(0, kBf16, M, C);
        void *res = a.ok ? a.bf16(0) : nullptr, *x = a.bf16(1, M * C), *w = a.some_bf16(2, C);
        if (!PyFloat_CheckExact(a.a[3])) a.ok = false;
        const float eps = a.ok ? (float)PyFloat_AS_DOUBLE(a.a[3]) : 0.0f;
        void *res_out = a.bf16(4, M * C), *y = a.some_bf16(5, M * C);
        float* rstd = a.some_f32(6, M);
        const int fmt = a.i32(7);
        float *am = a.f32(8), *sc = a.f32(9);
        void* ws = a.workspace(10, bytes);
        return [=](void* s) { return llmq_rmsnorm_fwd(res, x, w, M, C, eps, res_out, y, rstd, fmt, am, sc, ws, bytes, s); };
    });
}

template <bool SLABS>
PyObject* rmsnorm_codes(PyObject* const* args, Py_ssize_t n) {
    return run(args, n, 8, [](Args& a) {
        int64_t M = 0, C = 0;
        a.dims(0, kBf16, M, C);
        void *res = a.ok ? a.bf16(0) : nullptr, *w = a.some_bf16(1, C);
        float *rstd = a.some_f32(2, M), *sc = a.f32(3);
        const int fmt = a.i32(4);
        uint8_t *q = a.some_u8(5, M * C), *qt = SLABS ? a.some_u8(6, M * C) : a.u8(6, M * C);
        void* y = a.bf16(7, M * C);
        return [=](void* s) {
            return SLABS ? llmq_rmsnorm_apply_fp8_slabs(res, w, rstd, M, C, sc, fmt, q, qt, y, s) : llmq_rmsnorm_apply_fp8(res, w, rstd, M, C, sc, fmt, q, qt, y, s);
        };
    });
}
LLMQ_BINDING(rmsnorm_apply_fp8) { return rmsnorm_codes<false>(args, n); }
LLMQ_BINDING(rmsnorm_apply_fp8_slabs) { return rmsnorm_codes<true>(args, n); }

#define LLMQ_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {LLMQ_METHOD(linear_fwd), LLMQ_METHOD(linear_dgrad), LLMQ_METHOD(linear_wgrad), LLMQ_METHOD(amax), LLMQ_METHOD(quantize_fp8),
                           LLMQ_METHOD(quantize_fp8_slabs), LLMQ_METHOD(bf16_gemm_tn), LLMQ_METHOD(swiglu_fwd), LLMQ_METHOD(swiglu_fwd_fp8),
                           LLMQ_METHOD(swiglu_fwd_fp8_slabs), LLMQ_METHOD(swiglu_bwd), LLMQ_METHOD(rmsnorm_fwd), LLMQ_METHOD(rmsnorm_apply_fp8),
                           LLMQ_METHOD(rmsnorm_apply_fp8_slabs), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
    PyObject* c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_get_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    g_get_stream = g_get_device ? PyObject_GetAttrString(c, "_cuda_getCurrentRawStream") : nullptr;
    Py_DECREF(c);
    if (!g_get_stream) {                                          // a PyTorch without GPUs
        PyErr_SetString(PyExc_ImportError, "torch._C has no device functions");
        return nullptr;
    }
    return PyModule_Create(&g_module);
}
