// The layer calls of the Python binding for their ordinary case, without the interpreter between the checks: plain tensors of
// the documented types, outputs and workspace made here.  Every function returns None where an argument is anything else, an
// allocation fails or the library refuses; the Python code then does the call (and raises what there is to raise).  The library's
// entry points come in as addresses, so that this module depends on no particular build of it.
//
// What it saves is host time, which is what a call with less than 20 us of GPU work takes: a quantizer call 8.5 to 12 -> 5.2 to
// 5.9 us, a product 8.8 -> 4.9; a normalised layer at 64 tokens x 4096 x 12288 (two calls) 21.4 -> 18.1 us, the one-call layer at
// one token x 4096 x 4096 8.6 -> 7.8.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

#include <cstring>

#include "../../include/zqfp.h"

namespace {

using at::Tensor;

struct Library {
    decltype(&zqfp_quantize_act_fp8) quantize;
    decltype(&zqfp_rmsnorm_quantize_act_fp8) rmsnorm;
    decltype(&zqfp_layernorm_quantize_act_fp8) layernorm;
    decltype(&zqfp_add_rmsnorm_quantize_act_fp8) add_rmsnorm;
    decltype(&zqfp_add_layernorm_quantize_act_fp8) add_layernorm;
    decltype(&zqfp_relu_quantize_act_fp8) relu;
    decltype(&zqfp_swiglu_quantize_act_fp8) swiglu;
    decltype(&zqfp_packed_weight_bytes) blob_bytes;
    decltype(&zqfp_packed_weight_fp8_bytes) blob_bytes_fp8;
    decltype(&zqfp_gemm_workspace_bytes) workspace_bytes;
    decltype(&zqfp_w4a8_gemm) gemm;
    decltype(&zqfp_w4a8_gemm_lorc) gemm_lorc;
    decltype(&zqfp_w8a8_gemm) gemm_w8;
    decltype(&zqfp_w4a8_linear) linear;
} lib;

// a plain CUDA tensor of this type (no subclass, which might want to see the call), or nullptr
const Tensor* tensor(PyObject* o, at::ScalarType type, int64_t dims)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || t.dim() != dims || t.layout() != at::kStrided) return nullptr;
    return &t;
}
const Tensor* dense(PyObject* o, at::ScalarType type, int64_t dims)
{
    const Tensor* t = tensor(o, type, dims);
    return t != nullptr && t->is_contiguous() ? t : nullptr;
}
const Tensor* rows(PyObject* o, at::ScalarType type)
{
    const Tensor* t = tensor(o, type, 2);
    return t != nullptr && t->stride(1) == 1 ? t : nullptr;
}
bool size(PyObject* o, int64_t& v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool output_type(PyObject* o, at::ScalarType& type, int& code)
{
    if (!THPDtype_Check(o)) return false;
    type = reinterpret_cast<THPDtype*>(o)->scalar_type;
    code = type == at::kFloat ? ZQFP_OUT_F32 : ZQFP_OUT_BF16;
    return type == at::kFloat || type == at::kBFloat16;
}
Tensor make(at::IntArrayRef shape, at::ScalarType type, at::Device device) { return at::empty(shape, at::TensorOptions().dtype(type).device(device)); }
void* stream_of(at::Device device) { return c10::hip::getCurrentHIPStream(device.index()).stream(); }
void* ptr(const Tensor& t) { return t.data_ptr(); }

// Without the interpreter lock: allocations may wait for the device, and a launch for room in its queue or for code to be loaded, while
// other threads of the interpreter go on (and may be what the queue waits for).  Whatever is read from the arguments is read before.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

template <class F>
PyObject* guarded(F&& f)
{
    try {
        if (!at::impl::torch_function_mode_enabled())
            if (PyObject* r = f()) return r;
    } catch (const std::exception&) {  // a failed allocation, a tensor without storage: the Python code meets it again and reports it
    }
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

template <class... T>
PyObject* tuple_of(const T&... t)
{
    PyObject* items[] = {THPVariable_Wrap(t)...};
    PyObject* r = PyTuple_New(sizeof...(T));
    for (size_t i = 0; i < sizeof...(T); ++i) {
        if (r == nullptr || items[i] == nullptr) {
            Py_XDECREF(items[i]);
            continue;
        }
        PyTuple_SET_ITEM(r, i, items[i]);
    }
    return r;
}

// quantize(kind, X, other, gain, bias, eps, U): kind 0 plain, 1 RMS norm, 2 layer norm, 3 ReLU, 4 gated SiLU; other: residual (1, 2) or
// up values (4).  Returns the tuple of the Python function of that kind.
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int64_t kind;
        if (n != 7 || !size(a[0], kind)) return nullptr;
        const bool other = a[2] != Py_None, norm = kind == 1 || kind == 2;
        const Tensor* X = (kind >= 3 || other) ? rows(a[1], at::kBFloat16) : dense(a[1], at::kBFloat16, 2);
        if (X == nullptr) return nullptr;
        const int64_t M = X->size(0), K = X->size(1);
        const Tensor *R = nullptr, *g = nullptr, *b = nullptr, *U = nullptr;
        if (other) {
            R = rows(a[2], at::kBFloat16);
            if (R == nullptr || R->size(0) != M || R->size(1) != K) return nullptr;
        }
        if (norm) {
            g = dense(a[3], at::kBFloat16, 1);
            if (g == nullptr || g->size(0) != K || !PyFloat_CheckExact(a[5])) return nullptr;
        }
        if (kind == 2) {
            b = dense(a[4], at::kBFloat16, 1);
            if (b == nullptr || b->size(0) != K) return nullptr;
        }
        int r = 0;
        if (a[6] != Py_None) {
            U = dense(a[6], at::kHalf, 2);
            if (U == nullptr || U->size(0) != K || U->size(1) < 1 || U->size(1) > 64) return nullptr;
            r = (int)U->size(1);
        }
        const float eps = norm ? (float)PyFloat_AS_DOUBLE(a[5]) : 0.0f;
        auto address = [](const Tensor* t) -> const void* { return t != nullptr ? ptr(*t) : nullptr; };
        const void *x = ptr(*X), *o = address(R), *gain = address(g), *bias = address(b), *u = address(U);
        const int64_t ldx = X->stride(0), ldo = R != nullptr ? R->stride(0) : 0;
        const at::Device device = X->device();
        Tensor H, Xq, sx, T;
        int rc = ZQFP_E_SHAPE;
        {
            Unlocked unlocked;
            if (norm && other) H = make({M, K}, at::kBFloat16, device);
            Xq = make({M, K}, at::kByte, device);
            sx = make({M}, at::kFloat, device);
            if (r) T = make({M, r}, at::kFloat, device);
            uint8_t* q = static_cast<uint8_t*>(ptr(Xq));
            float *s = static_cast<float*>(ptr(sx)), *t = r ? static_cast<float*>(ptr(T)) : nullptr;
            void* st = stream_of(device);
            if (kind == 0) rc = lib.quantize(x, M, K, ldx, q, s, u, r, t, st);
            else if (kind == 3) rc = lib.relu(x, M, K, ldx, q, s, u, r, t, st);
            else if (kind == 4) rc = lib.swiglu(x, o, ldo, nullptr, M, K, ldx, q, s, u, r, t, st);
            else if (kind == 1 && !other) rc = lib.rmsnorm(x, gain, eps, M, K, ldx, q, s, u, r, t, st);
            else if (kind == 2 && !other) rc = lib.layernorm(x, gain, bias, eps, M, K, ldx, q, s, u, r, t, st);
            else if (kind == 1) rc = lib.add_rmsnorm(x, o, ldo, ptr(H), gain, eps, M, K, ldx, q, s, u, r, t, st);
            else if (kind == 2) rc = lib.add_layernorm(x, o, ldo, ptr(H), gain, bias, eps, M, K, ldx, q, s, u, r, t, st);
        }
        if (rc != ZQFP_OK) return nullptr;
        if (H.defined()) return r ? tuple_of(H, Xq, sx, T) : tuple_of(H, Xq, sx);
        return r ? tuple_of(Xq, sx, T) : tuple_of(Xq, sx);
    });
}

// gemm(wbits, Xq, sx, packed, N, G, T, V, out_dtype, accum): w4a8_gemm, w4a8_gemm_lorc, w8a8_gemm with their own output and workspace
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int64_t wbits, N, G, accum;
        at::ScalarType type;
        int code, r = 0;
        if (n != 10 || !size(a[0], wbits) || !size(a[4], N) || !size(a[5], G) || !size(a[9], accum) || !output_type(a[8], type, code)) return nullptr;
        const Tensor *Xq = dense(a[1], at::kByte, 2), *sx = dense(a[2], at::kFloat, 1), *packed = dense(a[3], at::kByte, 1);
        if (!Xq || !sx || !packed || G < 1 || G > INT32_MAX || accum < 0 || accum > 1) return nullptr;
        const int64_t M = Xq->size(0), K = Xq->size(1);
        const Tensor *T = nullptr, *V = nullptr;
        if (a[6] != Py_None) {
            T = dense(a[6], at::kFloat, 2);
            V = dense(a[7], at::kHalf, 2);
            if (!T || !V || T->size(0) != M || T->size(1) < 1 || T->size(1) > 64 || V->size(0) != T->size(1) || V->size(1) != N) return nullptr;
            r = (int)T->size(1);
        }
        const size_t need = wbits == 8 ? lib.blob_bytes_fp8(K, N, (int)G) : lib.blob_bytes(K, N, (int)G);
        if (need == 0 || (size_t)packed->numel() != need || sx->size(0) != M) return nullptr;
        const uint8_t* q = static_cast<const uint8_t*>(ptr(*Xq));
        const float *s = static_cast<const float*>(ptr(*sx)), *t = r ? static_cast<const float*>(ptr(*T)) : nullptr;
        const void *p = ptr(*packed), *v = r ? ptr(*V) : nullptr;
        const at::Device device = Xq->device();
        Tensor Y;
        int rc;
        {
            Unlocked unlocked;
            Y = make({M, N}, type, device);
            void *st = stream_of(device), *y = ptr(Y);
            const int64_t ldy = Y.stride(0);
            if (wbits == 8) {
                rc = lib.gemm_w8(q, s, M, K, p, N, (int)G, t, v, r, y, ldy, code, (int)accum, st);
            } else {
                const size_t bytes = lib.workspace_bytes(M, K, N);
                Tensor ws;
                if (bytes) ws = make({(int64_t)bytes}, at::kByte, device);
                void* w = bytes ? ptr(ws) : nullptr;
                rc = r ? lib.gemm_lorc(q, s, M, K, p, N, (int)G, t, v, r, y, ldy, code, (int)accum, w, bytes, st)
                       : lib.gemm(q, s, M, K, p, N, (int)G, y, ldy, code, (int)accum, w, bytes, st);
            }
        }
        return rc == ZQFP_OK ? THPVariable_Wrap(Y) : nullptr;
    });
}

// linear(X, packed, N, G, U, V, out_dtype, accum): w4a8_linear without the codes
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int64_t N, G, accum;
        at::ScalarType type;
        int code, r = 0;
        if (n != 8 || !size(a[2], N) || !size(a[3], G) || !size(a[7], accum) || !output_type(a[6], type, code)) return nullptr;
        const Tensor *X = rows(a[0], at::kBFloat16), *packed = dense(a[1], at::kByte, 1);
        if (!X || !packed || G < 1 || G > INT32_MAX || accum < 0 || accum > 1) return nullptr;
        const int64_t M = X->size(0), K = X->size(1);
        const Tensor *U = nullptr, *V = nullptr;
        if (a[4] != Py_None) {
            U = dense(a[4], at::kHalf, 2);
            V = dense(a[5], at::kHalf, 2);
            if (!U || !V || U->size(0) != K || U->size(1) < 1 || U->size(1) > 64 || V->size(0) != U->size(1) || V->size(1) != N) return nullptr;
            r = (int)U->size(1);
        }
        const size_t need = lib.blob_bytes(K, N, (int)G);
        if (need == 0 || (size_t)packed->numel() != need) return nullptr;
        const void *x = ptr(*X), *w = ptr(*packed), *u = r ? ptr(*U) : nullptr, *v = r ? ptr(*V) : nullptr;
        const int64_t ldx = X->stride(0);
        const at::Device device = X->device();
        Tensor Y;
        int rc;
        {
            Unlocked unlocked;
            Y = make({M, N}, type, device);
            Tensor Xq, sx, T, ws;
            size_t bytes = 0;
            if (!(M >= 1 && M <= 16 && K <= 4096 && r == 0)) {  // not the one-kernel form
                Xq = make({M, K}, at::kByte, device);
                sx = make({M}, at::kFloat, device);
                bytes = lib.workspace_bytes(M, K, N);
                if (bytes) ws = make({(int64_t)bytes}, at::kByte, device);
            }
            if (r) T = make({M, r}, at::kFloat, device);
            auto p = [](const Tensor& t) { return t.defined() ? ptr(t) : nullptr; };
            rc = lib.linear(x, ldx, M, K, w, N, (int)G, u, v, r, static_cast<uint8_t*>(p(Xq)), static_cast<float*>(p(sx)), static_cast<float*>(p(T)), ptr(Y),
                            Y.stride(0), code, (int)accum, p(ws), bytes, stream_of(device));
        }
        return rc == ZQFP_OK ? THPVariable_Wrap(Y) : nullptr;
    });
}

// use(addresses): the library's entry points, in the order of `Library`
PyObject* use(PyObject*, PyObject* o)
{
    void* addresses[sizeof(Library) / sizeof(void*)];
    constexpr Py_ssize_t count = sizeof(addresses) / sizeof(addresses[0]);
    if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != count) {
        PyErr_SetString(PyExc_TypeError, "a tuple with the address of every entry point");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < count; ++i) {
        addresses[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(o, i));
        if (addresses[i] == nullptr) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    std::memcpy(&lib, addresses, sizeof lib);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"use", use, METH_O, nullptr},
                         {"quantize", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(quantize)), METH_FASTCALL, nullptr},
                         {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gemm)), METH_FASTCALL, nullptr},
                         {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
