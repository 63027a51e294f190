// Plain calls of the Python binding in native code: argument checks, raw pointers, current stream, call.
//
// In Python these cost about twice what the smallest launches take on the GPU (8B O projection, M = 1: 9.9 us a call
// among others for a kernel of 4.4 us; through this module 4.3 us).  A call that is not plain -- an argument that is no ordinary
// CUDA tensor, or that any check of the binding would refuse -- is answered with -1 before anything is done, and the
// binding's own code takes it from there (and says what is wrong with it).
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/core/DispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "lutq.h"

namespace {

decltype(&lutq_packed_bytes) packed_bytes = nullptr;
decltype(&lutq_matmul) matmul = nullptr;
decltype(&lutq_matmul_static) matmul_static = nullptr;
decltype(&lutq_matmul_channel) matmul_channel = nullptr;
decltype(&lutq_matmul_pairs) matmul_pairs = nullptr;
decltype(&lutq_matmul_quads) matmul_quads = nullptr;
decltype(&lutq_quantize) quantize = nullptr;
decltype(&lutq_dequant) dequant = nullptr;

// the functions of liblutq.so by address, in the order of the declarations above
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    void* p[8];
    if (n != 8) { PyErr_SetString(PyExc_TypeError, "eight addresses"); return nullptr; }
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (!p[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address"); return nullptr; }
    }
    packed_bytes = reinterpret_cast<decltype(packed_bytes)>(p[0]);
    matmul = reinterpret_cast<decltype(matmul)>(p[1]);
    matmul_static = reinterpret_cast<decltype(matmul_static)>(p[2]);
    matmul_channel = reinterpret_cast<decltype(matmul_channel)>(p[3]);
    matmul_pairs = reinterpret_cast<decltype(matmul_pairs)>(p[4]);
    matmul_quads = reinterpret_cast<decltype(matmul_quads)>(p[5]);
    quantize = reinterpret_cast<decltype(quantize)>(p[6]);
    dequant = reinterpret_cast<decltype(dequant)>(p[7]);
    Py_RETURN_NONE;
}

// an ordinary dense CUDA tensor (no subclass, no functorch or functionalisation wrapper) that is contiguous, or null
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    static const c10::DispatchKeySet wrappers({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                               c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize});
    if (!t.defined() || t.layout() != c10::kStrided || t.unsafeGetTensorImpl()->key_set().has_any(wrappers)) return nullptr;
    return t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

int dtype_code(const at::Tensor& t) {
    return t.scalar_type() == at::kHalf ? LUTQ_F16 : t.scalar_type() == at::kBFloat16 ? LUTQ_BF16 : -1;
}

bool small_int(PyObject* o, long lo, long hi, int* out) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < lo || v > hi) return false;
    *out = (int)v;
    return true;
}

bool shape_is(const at::Tensor& t, int64_t a, int64_t b) { return t.dim() == 2 && t.size(0) == a && t.size(1) == b; }

void* current_stream() { return static_cast<void*>(c10::hip::getCurrentHIPStream().stream()); }

// A torch call that throws (a nested tensor asked for an irregular size, storage that may not be read, no device) makes the call one
// that is not plain: no exception leaves through the C entry, and the binding's own code meets the same refusal and raises it.
template <typename F> PyObject* answer(F f) {
    try { return f(); } catch (...) { return PyLong_FromLong(-1); }
}

struct WithoutGil {
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

enum Kind { kMatmul = 0, kStatic = 1, kChannel = 2, kPairs = 3, kQuads = 4 };

// (kind, X, packed, scales, lut, bits, group_size, Y, workspace or None) -> status, or -1
PyObject* mm(PyObject*, PyObject* const* args, Py_ssize_t n) { return answer([&]() -> PyObject* {
    int kind, bits, group;
    if (!matmul || n != 9 || !small_int(args[0], 0, 4, &kind) || !small_int(args[5], 2, 4, &bits) || !small_int(args[6], 1, 1 << 16, &group))
        return PyLong_FromLong(-1);
    const at::Tensor *X = plain(args[1]), *packed = plain(args[2]), *scales = plain(args[3]), *lut = plain(args[4]),
                     *Y = plain(args[7]), *ws = kind == kStatic ? nullptr : plain(args[8]);
    if (!X || !packed || !scales || !lut || !Y || (kind != kStatic && !ws)) return PyLong_FromLong(-1);
    const int code = dtype_code(*X);
    if (code < 0 || dtype_code(*scales) != code || dtype_code(*lut) != code || dtype_code(*Y) != code || X->dim() != 2 || scales->dim() != 2)
        return PyLong_FromLong(-1);
    const int64_t M = X->size(0), K = X->size(1), N = scales->size(0);
    const bool table = kind == kChannel ? shape_is(*lut, N, 1 << bits)
                     : kind == kPairs   ? bits == 4 && shape_is(*lut, 256, 2)
                     : kind == kQuads   ? bits == 2 && shape_is(*lut, 256, 4)
                                        : lut->numel() == (1 << bits);
    if (!table || scales->size(1) * group != K || !shape_is(*Y, M, N) || packed->numel() != (int64_t)packed_bytes(N, K, bits, group))
        return PyLong_FromLong(-1);
    const void *x = X->data_ptr(), *p = packed->data_ptr(), *s = scales->data_ptr(), *l = lut->data_ptr();
    void *y = Y->data_ptr(), *w = ws ? ws->data_ptr() : nullptr, *stream = current_stream();
    const size_t wb = ws ? (size_t)ws->numel() * ws->element_size() : 0;
    const lutq_dtype dt = (lutq_dtype)code;
    lutq_status st = LUTQ_OK;
    {
        WithoutGil released;
        switch (kind) {
            case kMatmul: st = matmul(x, p, s, l, bits, group, M, N, K, dt, y, w, wb, stream); break;
            case kStatic: st = matmul_static(x, p, s, l, bits, group, M, N, K, dt, y, stream, nullptr); break;
            case kChannel: st = matmul_channel(x, p, s, l, bits, group, M, N, K, dt, y, w, wb, stream); break;
            case kPairs: st = matmul_pairs(x, p, s, l, group, M, N, K, dt, y, w, wb, stream); break;
            case kQuads: st = matmul_quads(x, p, s, l, group, M, N, K, dt, y, w, wb, stream); break;
        }
    }
    return PyLong_FromLong((long)st);
}); }

// (W, lut, bits, group_size, scales_out, packed_out) -> status, or -1
PyObject* quant(PyObject*, PyObject* const* args, Py_ssize_t n) { return answer([&]() -> PyObject* {
    int bits, group;
    if (!quantize || n != 6 || !small_int(args[2], 2, 4, &bits) || !small_int(args[3], 1, 1 << 16, &group)) return PyLong_FromLong(-1);
    const at::Tensor *W = plain(args[0]), *lut = plain(args[1]), *scales = plain(args[4]), *packed = plain(args[5]);
    if (!W || !lut || !scales || !packed) return PyLong_FromLong(-1);
    const int code = dtype_code(*lut);
    const bool f32 = W->scalar_type() == at::kFloat;
    if (code < 0 || (!f32 && dtype_code(*W) != code) || dtype_code(*scales) != code || W->dim() != 2) return PyLong_FromLong(-1);
    const int64_t N = W->size(0), K = W->size(1);
    if (!shape_is(*scales, N, K / group) || lut->numel() != (1 << bits) ||
        packed->numel() * packed->element_size() != (int64_t)packed_bytes(N, K, bits, group))
        return PyLong_FromLong(-1);
    const void *w = W->data_ptr(), *l = lut->data_ptr();
    void *s = scales->data_ptr(), *p = packed->data_ptr(), *stream = current_stream();
    lutq_status st;
    {
        WithoutGil released;
        st = quantize(w, f32 ? 1 : 0, l, bits, group, N, K, (lutq_dtype)code, s, p, stream);
    }
    return PyLong_FromLong((long)st);
}); }

// (packed, scales, lut, bits, group_size, W_out) -> status, or -1
PyObject* dequantise(PyObject*, PyObject* const* args, Py_ssize_t n) { return answer([&]() -> PyObject* {
    int bits, group;
    if (!dequant || n != 6 || !small_int(args[3], 2, 4, &bits) || !small_int(args[4], 1, 1 << 16, &group)) return PyLong_FromLong(-1);
    const at::Tensor *packed = plain(args[0]), *scales = plain(args[1]), *lut = plain(args[2]), *W = plain(args[5]);
    if (!W || !lut || !scales || !packed) return PyLong_FromLong(-1);
    const int code = dtype_code(*W);
    if (code < 0 || dtype_code(*lut) != code || dtype_code(*scales) != code || W->dim() != 2 || scales->dim() != 2) return PyLong_FromLong(-1);
    const int64_t N = W->size(0), K = W->size(1);
    if (scales->size(0) != N || scales->size(1) * group != K || lut->numel() != (1 << bits) ||
        packed->numel() != (int64_t)packed_bytes(N, K, bits, group))
        return PyLong_FromLong(-1);
    const void *p = packed->data_ptr(), *s = scales->data_ptr(), *l = lut->data_ptr();
    void *w = W->data_ptr(), *stream = current_stream();
    lutq_status st;
    {
        WithoutGil released;
        st = dequant(p, s, l, bits, group, N, K, (lutq_dtype)code, w, stream);
    }
    return PyLong_FromLong((long)st);
}); }

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {"mm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(mm)), METH_FASTCALL, nullptr},
    {"quantize", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(quant)), METH_FASTCALL, nullptr},
    {"dequant", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(dequantise)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lutq_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lutq_torch() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", LUTQ_TORCH_VERSION) != 0) { Py_DECREF(m); return nullptr; }
    return m;
}
