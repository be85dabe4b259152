// Argument marshalling of the Python binding, natively: checks that the tensors are what the C entry point will index
// (device, layout, shape, element type), reads their addresses and makes the call.  A call whose arguments do not pass
// is not made here (None comes back) and goes through the Python form of the same checks, which names what is wrong.
//
// Why: an entry point enqueues a kernel of a few microseconds, and marshalling its ten tensors in Python took 12 - 15 us
// a call, so a program that calls the subgraphs one by one waited for the interpreter.  Here it takes about 1 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <initializer_list>
#include <new>
#include "../../include/ago.h"

namespace {

// One marshalled call: everything the C entry point needs, as plain values.
struct Launch {
    int (*run)(const Launch&);
    const void* p[11];            // tensors in the entry point's order
    int d[8];                     // sizes
    int k[3];                     // stride / depthwise size / residual / activation ...
    long long s[3];
    float f;
    ago_dtype dt;
    void* ws;
    size_t ws_bytes;
    void* stream;
};

typedef const at::Tensor* T;
struct Args {
    PyObject* const* a;           // one slot per declared argument, NULL where the caller gave none
    bool ok = true;

    bool given(int i) const { return a[i] && a[i] != Py_None; }
    T any(int i) {                // a tensor of any shape
        if (!given(i) || !THPVariable_Check(a[i])) { ok = false; return nullptr; }
        return &THPVariable_Unpack(a[i]);
    }
    T like(int i, std::initializer_list<int64_t> shape, at::ScalarType st) {      // contiguous, on the device, of this shape and type
        T t = any(i);
        if (!t) return nullptr;
        const auto sz = t->sizes();
        bool same = t->is_cuda() && t->is_contiguous() && t->scalar_type() == st && sz.size() == shape.size();
        size_t q = 0;
        for (int64_t v : shape) same = same && sz[q++] == v;
        ok = ok && same;
        return t;
    }
    T first(int i, size_t rank) { // the tensor the sizes are read from
        T t = any(i);
        if (!t) return nullptr;
        if (t->dim() != (int64_t)rank || !t->is_cuda() || !t->is_contiguous() ||
            (t->scalar_type() != at::kBFloat16 && t->scalar_type() != at::kFloat)) { ok = false; return nullptr; }
        for (int64_t v : t->sizes()) ok = ok && v < (1LL << 31);
        return ok ? t : nullptr;
    }
    int64_t size(int i, size_t rank, size_t q) {
        T t = any(i);
        if (!t || t->dim() != (int64_t)rank) { ok = false; return 0; }
        ok = ok && t->sizes()[q] < (1LL << 31);
        return t->sizes()[q];
    }
    const void* ptr(int i, std::initializer_list<int64_t> shape, at::ScalarType st) {
        T t = like(i, shape, st);
        return ok ? t->data_ptr() : nullptr;
    }
    const void* opt(int i, std::initializer_list<int64_t> shape, at::ScalarType st) { return given(i) ? ptr(i, shape, st) : nullptr; }
    const float* bias(int i, int64_t n) { return (const float*)opt(i, {n}, at::kFloat); }
    int num(int i, int otherwise = 0, bool optional = false) {
        if (!a[i] && optional) return otherwise;
        if (!a[i] || !PyLong_Check(a[i])) { ok = false; return 0; }              // bool is an int
        const long v = PyLong_AsLong(a[i]);
        if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        ok = ok && v >= INT_MIN && v <= INT_MAX;
        return (int)v;
    }
    float real(int i) {
        if (!a[i] || !(PyFloat_Check(a[i]) || PyLong_Check(a[i]))) { ok = false; return 0; }
        const double v = PyFloat_AsDouble(a[i]);
        if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return (float)v;
    }
    int truth(int i, int otherwise = -1) {           // -1: required
        if (!a[i] && otherwise >= 0) return otherwise;
        if (!a[i] || !PyLong_Check(a[i])) { ok = false; return 0; }
        return PyObject_IsTrue(a[i]) ? 1 : 0;
    }
    void workspace(int i, Launch& l) {
        l.ws = nullptr;
        l.ws_bytes = 0;
        if (!given(i)) return;
        if (T t = any(i)) { l.ws = t->data_ptr(); l.ws_bytes = (size_t)t->numel() * t->element_size(); }
    }
};
ago_dtype dtype_of(T t) { return t->scalar_type() == at::kBFloat16 ? AGO_BF16 : AGO_F32; }

typedef bool (*Parse)(Args&, Launch&);
#define F(i) ((const float*)l.p[i])
#define Y(i) (const_cast<void*>(l.p[i]))
#define RUN(call) l.run = [](const Launch& l) -> int { return (int)(call); }
#define SIZES(t) const auto sz = (t)->sizes(); const auto st = (t)->scalar_type(); l.dt = dtype_of(t)

// x, w1, b1, wd, bd, w2, b2, y, stride, residual [, workspace]
bool invres(Args& a, Launch& l, int ks) {
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int64_t ce = a.size(5, 2, 0), co = a.size(5, 2, 1);
    const int stride = a.num(8);
    if (ks == 0) ks = (int)a.size(3, 3, 0);
    if (!a.ok || stride < 1) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {sz[3], ce}, st);
    l.p[2] = a.bias(2, ce);
    l.p[3] = a.ptr(3, {ks, ks, ce}, st);
    l.p[4] = a.bias(4, ce);
    l.p[5] = a.ptr(5, {ce, co}, st);
    l.p[6] = a.bias(6, co);
    l.p[7] = a.ptr(7, {sz[0], (sz[1] - 1) / stride + 1, (sz[2] - 1) / stride + 1, co}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.d[4] = (int)ce; l.d[5] = (int)co;
    l.k[0] = stride; l.k[1] = ks; l.k[2] = a.truth(9);
    return a.ok;
}
bool p_invres(Args& a, Launch& l) {
    RUN(ago_fused_invres(l.p[0], l.p[1], F(2), l.p[3], F(4), l.p[5], F(6), Y(7), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], l.d[5], l.k[0], l.k[2],
                         l.dt, l.ws, l.ws_bytes, l.stream));
    a.workspace(10, l);
    return invres(a, l, 3);
}
bool p_invres_k(Args& a, Launch& l) {
    RUN(ago_fused_invres_k(l.p[0], l.p[1], F(2), l.p[3], F(4), l.p[5], F(6), Y(7), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], l.d[5], l.k[0], l.k[1],
                           l.k[2], l.dt, l.ws, l.ws_bytes, l.stream));
    a.workspace(10, l);
    return invres(a, l, 0);
}
bool p_invres_noalloc(Args& a, Launch& l) {
    RUN(ago_fused_invres_noalloc(l.p[0], l.p[1], F(2), l.p[3], F(4), l.p[5], F(6), Y(7), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], l.d[5], l.k[0],
                                 l.k[1], l.k[2], l.dt, l.stream));
    return invres(a, l, 0);
}
// x, w1, b1, wd, bd, y, stride [, workspace]
bool pw_dw(Args& a, Launch& l, int ks) {
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int64_t ce = a.size(1, 2, 1);
    const int stride = a.num(6);
    if (ks == 0) ks = (int)a.size(3, 3, 0);
    if (!a.ok || stride < 1) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {sz[3], ce}, st);
    l.p[2] = a.bias(2, ce);
    l.p[3] = a.ptr(3, {ks, ks, ce}, st);
    l.p[4] = a.bias(4, ce);
    l.p[5] = a.ptr(5, {sz[0], (sz[1] - 1) / stride + 1, (sz[2] - 1) / stride + 1, ce}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.d[4] = (int)ce; l.k[0] = stride; l.k[1] = ks;
    a.workspace(7, l);
    RUN(ago_fused_pw_dw_k(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], l.k[0], l.k[1], l.dt, l.ws, l.ws_bytes,
                          l.stream));
    return a.ok;
}
bool p_pw_dw(Args& a, Launch& l) { return pw_dw(a, l, 3); }
bool p_pw_dw_k(Args& a, Launch& l) { return pw_dw(a, l, 0); }
// x, wd, bd, w2, b2, y, stride [, workspace]
bool dw_pw(Args& a, Launch& l, int ks) {
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int64_t co = a.size(3, 2, 1);
    const int stride = a.num(6);
    if (ks == 0) ks = (int)a.size(1, 3, 0);
    if (!a.ok || stride < 1) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {ks, ks, sz[3]}, st);
    l.p[2] = a.bias(2, sz[3]);
    l.p[3] = a.ptr(3, {sz[3], co}, st);
    l.p[4] = a.bias(4, co);
    l.p[5] = a.ptr(5, {sz[0], (sz[1] - 1) / stride + 1, (sz[2] - 1) / stride + 1, co}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.d[4] = (int)co; l.k[0] = stride; l.k[1] = ks;
    a.workspace(7, l);
    RUN(ago_fused_dw_pw_k(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], l.k[0], l.k[1], l.dt, l.ws, l.ws_bytes,
                          l.stream));
    return a.ok;
}
bool p_dw_pw(Args& a, Launch& l) { return dw_pw(a, l, 3); }
bool p_dw_pw_k(Args& a, Launch& l) { return dw_pw(a, l, 0); }
// x, wa, ba, wb, bb, y, stride [, workspace]
bool p_dw_dw(Args& a, Launch& l) {
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int stride = a.num(6);
    if (!a.ok || stride < 1) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {3, 3, sz[3]}, st);
    l.p[2] = a.bias(2, sz[3]);
    l.p[3] = a.ptr(3, {3, 3, sz[3]}, st);
    l.p[4] = a.bias(4, sz[3]);
    l.p[5] = a.ptr(5, {sz[0], (sz[1] - 1) / stride + 1, (sz[2] - 1) / stride + 1, sz[3]}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.k[0] = stride;
    a.workspace(7, l);
    RUN(ago_fused_dw_dw(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], l.k[0], l.dt, l.ws, l.ws_bytes, l.stream));
    return a.ok;
}
// x, w1, b1, w2, b2, y [, act, workspace] on NHWC
bool p_pw_pw(Args& a, Launch& l) {
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int64_t f = a.size(3, 2, 0), k2 = a.size(3, 2, 1);
    if (!a.ok) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {sz[3], f}, st);
    l.p[2] = a.bias(2, f);
    l.p[3] = a.ptr(3, {f, k2}, st);
    l.p[4] = a.bias(4, k2);
    l.p[5] = a.ptr(5, {sz[0], sz[1], sz[2], k2}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.d[4] = (int)f; l.d[5] = (int)k2;
    l.k[0] = a.num(6, AGO_ACT_RELU, true);
    a.workspace(7, l);
    RUN(ago_fused_pw_pw(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], l.d[5], (ago_act)l.k[0], l.dt, l.ws,
                        l.ws_bytes, l.stream));
    return a.ok;
}
// x, wa, ba, wb, bb, y, residual [, workspace]
bool p_conv_chain(Args& a, Launch& l) {
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {3, 3, sz[3], sz[3]}, st);
    l.p[2] = a.bias(2, sz[3]);
    l.p[3] = a.ptr(3, {3, 3, sz[3], sz[3]}, st);
    l.p[4] = a.bias(4, sz[3]);
    l.p[5] = a.ptr(5, {sz[0], sz[1], sz[2], sz[3]}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.k[0] = a.truth(6);
    a.workspace(7, l);
    RUN(ago_fused_conv_chain(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], l.k[0], l.dt, l.ws, l.ws_bytes, l.stream));
    return a.ok;
}
// x, w1, b1, w2, b2, y: the weights row-major, or packed ([k / 32][n / 16][64][8])
bool chain2(Args& a, Launch& l, bool packed) {
    T x = a.first(0, 2);
    if (!x) return false;
    SIZES(x);
    const int64_t f = packed ? a.size(1, 4, 1) * 16 : a.size(3, 2, 0), k2 = packed ? a.size(3, 4, 1) * 16 : a.size(3, 2, 1);
    if (!a.ok || (packed && (sz[1] % 32 || f % 32))) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = packed ? a.ptr(1, {sz[1] / 32, f / 16, 64, 8}, st) : a.ptr(1, {sz[1], f}, st);
    l.p[2] = a.bias(2, f);
    l.p[3] = packed ? a.ptr(3, {f / 32, k2 / 16, 64, 8}, st) : a.ptr(3, {f, k2}, st);
    l.p[4] = a.bias(4, k2);
    l.p[5] = a.ptr(5, {sz[0], k2}, st);
    l.d[0] = (int)sz[0]; l.d[1] = (int)sz[1]; l.d[2] = (int)f; l.d[3] = (int)k2;
    return a.ok;
}
bool p_ffn(Args& a, Launch& l) {
    l.k[0] = a.num(6, AGO_ACT_GELU_TANH, true);
    a.workspace(7, l);
    RUN(ago_fused_ffn(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], (ago_act)l.k[0], l.dt, l.ws, l.ws_bytes, l.stream));
    return chain2(a, l, false);
}
bool p_ffn_packed(Args& a, Launch& l) {
    l.k[0] = a.num(6, AGO_ACT_GELU_TANH, true);
    a.workspace(7, l);
    RUN(ago_fused_ffn_packed(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], (ago_act)l.k[0], l.dt, l.ws, l.ws_bytes,
                             l.stream));
    return chain2(a, l, true);
}
bool p_unfused_ffn_packed(Args& a, Launch& l) {
    l.k[0] = a.num(6, AGO_ACT_GELU_TANH, true);
    a.workspace(7, l);
    RUN(ago_unfused_ffn_packed(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], (ago_act)l.k[0], l.dt, l.ws, l.ws_bytes,
                               l.stream));
    return chain2(a, l, true);
}
bool p_unfused_ffn(Args& a, Launch& l) {      // ..., act, epilogue_fused, workspace
    l.k[0] = a.num(6);
    if (!a.a[8]) return false;
    l.k[1] = a.truth(7);
    a.workspace(8, l);
    RUN(ago_unfused_ffn(l.p[0], l.p[1], F(2), l.p[3], F(4), Y(5), l.d[0], l.d[1], l.d[2], l.d[3], (ago_act)l.k[0], l.dt, l.k[1], l.ws, l.ws_bytes,
                        l.stream));
    return chain2(a, l, false);
}
bool p_pack_weight(Args& a, Launch& l) {      // w, wp
    T w = a.first(0, 2);
    if (!w) return false;
    SIZES(w);
    if (sz[0] % 32 || sz[1] % 16) return false;
    l.p[0] = w->data_ptr();
    l.p[1] = a.ptr(1, {sz[0] / 32, sz[1] / 16, 64, 8}, st);
    l.d[0] = (int)sz[0]; l.d[1] = (int)sz[1];
    RUN(ago_pack_weight(l.p[0], Y(1), l.d[0], l.d[1], l.dt, l.stream));
    return a.ok;
}
bool p_gemm(Args& a, Launch& l) {             // a, b, bias, res, c [, act]
    T x = a.first(0, 2);
    if (!x) return false;
    SIZES(x);
    const int64_t n = a.size(1, 2, 1);
    if (!a.ok) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {sz[1], n}, st);
    l.p[2] = a.bias(2, n);
    l.p[3] = a.opt(3, {sz[0], n}, st);
    l.p[4] = a.ptr(4, {sz[0], n}, st);
    l.d[0] = (int)sz[0]; l.d[1] = (int)sz[1]; l.d[2] = (int)n;
    l.k[0] = a.num(5, AGO_ACT_NONE, true);
    RUN(ago_gemm(l.p[0], l.p[1], F(2), l.p[3], Y(4), l.d[0], l.d[1], l.d[2], (ago_act)l.k[0], l.dt, l.stream));
    return a.ok;
}
bool p_gemm_packed(Args& a, Launch& l) {      // a, wp, bias, c [, act]
    T x = a.first(0, 2);
    if (!x) return false;
    SIZES(x);
    const int64_t n = a.size(1, 4, 1) * 16;
    if (!a.ok || sz[1] % 32) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {sz[1] / 32, n / 16, 64, 8}, st);
    l.p[2] = a.bias(2, n);
    l.p[3] = a.ptr(3, {sz[0], n}, st);
    l.d[0] = (int)sz[0]; l.d[1] = (int)sz[1]; l.d[2] = (int)n;
    l.k[0] = a.num(4, AGO_ACT_NONE, true);
    RUN(ago_gemm_packed(l.p[0], l.p[1], F(2), Y(3), l.d[0], l.d[1], l.d[2], (ago_act)l.k[0], l.dt, l.stream));
    return a.ok;
}
bool p_conv1x1(Args& a, Launch& l) {          // x, w, bias, res, y [, act]
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int64_t n = a.size(1, 2, 1);
    if (!a.ok) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {sz[3], n}, st);
    l.p[2] = a.bias(2, n);
    l.p[3] = a.opt(3, {sz[0], sz[1], sz[2], n}, st);
    l.p[4] = a.ptr(4, {sz[0], sz[1], sz[2], n}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.d[4] = (int)n;
    l.k[0] = a.num(5, AGO_ACT_NONE, true);
    RUN(ago_conv1x1(l.p[0], l.p[1], F(2), l.p[3], Y(4), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], (ago_act)l.k[0], l.dt, l.stream));
    return a.ok;
}
bool p_dwconv3x3(Args& a, Launch& l) {        // x, w, bias, y, stride [, act]
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int stride = a.num(4);
    if (!a.ok || stride < 1) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {3, 3, sz[3]}, st);
    l.p[2] = a.bias(2, sz[3]);
    l.p[3] = a.ptr(3, {sz[0], (sz[1] - 1) / stride + 1, (sz[2] - 1) / stride + 1, sz[3]}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.k[0] = stride;
    l.k[1] = a.num(5, AGO_ACT_NONE, true);
    RUN(ago_dwconv3x3(l.p[0], l.p[1], F(2), Y(3), l.d[0], l.d[1], l.d[2], l.d[3], l.k[0], (ago_act)l.k[1], l.dt, l.stream));
    return a.ok;
}
bool p_conv3x3(Args& a, Launch& l) {          // x, w, bias, res, y [, act]
    T x = a.first(0, 4);
    if (!x) return false;
    SIZES(x);
    const int64_t n = a.size(1, 4, 3);
    if (!a.ok) return false;
    l.p[0] = x->data_ptr();
    l.p[1] = a.ptr(1, {3, 3, sz[3], n}, st);
    l.p[2] = a.bias(2, n);
    l.p[3] = a.opt(3, {sz[0], sz[1], sz[2], n}, st);
    l.p[4] = a.ptr(4, {sz[0], sz[1], sz[2], n}, st);
    for (int q = 0; q < 4; ++q) l.d[q] = (int)sz[q];
    l.d[4] = (int)n;
    l.k[0] = a.num(5, AGO_ACT_NONE, true);
    RUN(ago_conv3x3(l.p[0], l.p[1], F(2), l.p[3], Y(4), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], (ago_act)l.k[0], l.dt, l.stream));
    return a.ok;
}
bool same_shape(Args& a, T x, int i) {
    T t = a.any(i);
    a.ok = a.ok && t && t->is_cuda() && t->is_contiguous() && t->scalar_type() == x->scalar_type() && t->sizes() == x->sizes();
    return a.ok;
}
T elementwise(Args& a) {
    T x = a.any(0);
    if (!x || !x->is_cuda() || !x->is_contiguous() || x->dim() < 1 || (x->scalar_type() != at::kBFloat16 && x->scalar_type() != at::kFloat)) return nullptr;
    return x;
}
bool p_bias_act(Args& a, Launch& l) {         // x, bias, y [, act]
    T x = elementwise(a);
    if (!x || x->sizes().back() < 1 || x->sizes().back() >= (1LL << 31)) return false;
    l.dt = dtype_of(x);
    const int64_t c = x->sizes().back();
    l.p[0] = x->data_ptr();
    l.p[1] = a.bias(1, c);
    if (!a.ok || !a.given(2) || !same_shape(a, x, 2)) return false;
    l.p[2] = a.any(2)->data_ptr();
    l.s[0] = x->numel() / c; l.d[0] = (int)c;
    l.k[0] = a.num(3, AGO_ACT_NONE, true);
    RUN(ago_bias_act(l.p[0], F(1), Y(2), (long)l.s[0], l.d[0], (ago_act)l.k[0], l.dt, l.stream));
    return a.ok;
}
bool p_add_act(Args& a, Launch& l) {          // a, b, y [, act]
    T x = elementwise(a);
    if (!x || !a.given(1) || !a.given(2) || !THPVariable_Check(a.a[1]) || !THPVariable_Check(a.a[2])) return false;
    l.dt = dtype_of(x);
    if (!same_shape(a, x, 1) || !same_shape(a, x, 2)) return false;
    l.p[0] = x->data_ptr(); l.p[1] = a.any(1)->data_ptr(); l.p[2] = a.any(2)->data_ptr();
    l.s[0] = x->numel();
    l.k[0] = a.num(3, AGO_ACT_NONE, true);
    RUN(ago_add_act(l.p[0], l.p[1], Y(2), (long)l.s[0], (ago_act)l.k[0], l.dt, l.stream));
    return a.ok;
}
bool heads(Args& a, Launch& l, int out) {     // q, k, v, (out) of one 4-d shape
    T q = a.first(0, 4);
    if (!q) return false;
    SIZES(q);
    const int at_[4] = {0, 1, 2, out};
    for (int i = 0; i < 4; ++i) l.p[i] = a.ptr(at_[i], {sz[0], sz[1], sz[2], sz[3]}, st);
    for (int i = 0; i < 4; ++i) l.d[i] = (int)sz[i];
    return a.ok;
}
bool p_attn(Args& a, Launch& l) {             // q, k, v, o, scale [, workspace]
    l.f = a.real(4);
    a.workspace(5, l);
    RUN(ago_fused_attn(l.p[0], l.p[1], l.p[2], Y(3), l.d[0], l.d[1], l.d[2], l.d[3], l.f, l.dt, l.ws, l.ws_bytes, l.stream));
    return heads(a, l, 3);
}
bool p_attn_bshd(Args& a, Launch& l) {        // the same on [B, S, Hh, D]
    l.f = a.real(4);
    a.workspace(5, l);
    if (!heads(a, l, 3)) return false;
    const long long hd = (long long)l.d[2] * l.d[3];
    l.s[0] = l.d[1] * hd; l.s[1] = l.d[3]; l.s[2] = hd;
    RUN(ago_fused_attn_strided(l.p[0], l.p[1], l.p[2], Y(3), l.d[0], l.d[2], l.d[1], l.d[3], l.s[0], l.s[1], l.s[2], l.f, l.dt, l.ws, l.ws_bytes,
                               l.stream));
    return true;
}
bool p_attn_bias(Args& a, Launch& l) {        // q, k, v, bias, o, scale [, workspace]
    l.f = a.real(5);
    a.workspace(6, l);
    if (!heads(a, l, 4)) return false;
    T b = a.any(3);
    if (!b || b->dim() != 4) return false;
    const int64_t s = l.d[2], bb = b->sizes()[0], hb = b->sizes()[1];
    if ((bb != 1 && bb != l.d[0]) || (hb != 1 && hb != l.d[1])) return false;
    l.p[4] = a.ptr(3, {bb, hb, s, s}, a.any(0)->scalar_type());
    l.s[0] = bb > 1 ? hb * s * s : 0;
    l.s[1] = hb > 1 ? s * s : 0;
    RUN(ago_fused_attn_bias(l.p[0], l.p[1], l.p[2], l.p[4], Y(3), l.d[0], l.d[1], l.d[2], l.d[3], l.s[0], l.s[1], l.f, l.dt, l.ws, l.ws_bytes,
                            l.stream));
    return a.ok;
}
bool p_qkv(Args& a, Launch& l) {              // x, wq, wk, wv, bq, bk, bv, q, k, v [, head_major, workspace]
    T x = a.first(0, 2), q = a.first(7, 4);
    if (!x || !q) return false;
    SIZES(x);
    const auto o = q->sizes();
    const int hm = a.truth(10, 1);
    const int64_t S = hm ? o[2] : o[1], Hh = hm ? o[1] : o[2], n = Hh * o[3];
    if (!a.ok || o[0] * S != sz[0] || n >= (1LL << 31)) return false;
    l.p[0] = x->data_ptr();
    for (int i = 0; i < 3; ++i) {
        l.p[1 + i] = a.ptr(1 + i, {sz[1], n}, st);
        l.p[4 + i] = a.bias(4 + i, n);
        l.p[7 + i] = a.ptr(7 + i, {o[0], o[1], o[2], o[3]}, st);
    }
    l.d[0] = (int)o[0]; l.d[1] = (int)S; l.d[2] = (int)sz[1]; l.d[3] = (int)Hh; l.d[4] = (int)o[3];
    l.k[0] = hm;
    a.workspace(11, l);
    RUN(ago_fused_qkv(l.p[0], l.p[1], l.p[2], l.p[3], F(4), F(5), F(6), Y(7), Y(8), Y(9), l.d[0], l.d[1], l.d[2], l.d[3], l.d[4], l.k[0], l.dt, l.ws,
                      l.ws_bytes, l.stream));
    return a.ok;
}

const struct { const char* name; Parse parse; } kEntries[] = {
    {"ago_fused_invres", p_invres}, {"ago_fused_invres_k", p_invres_k}, {"ago_fused_invres_noalloc", p_invres_noalloc},
    {"ago_fused_pw_dw", p_pw_dw}, {"ago_fused_pw_dw_k", p_pw_dw_k}, {"ago_fused_dw_pw", p_dw_pw}, {"ago_fused_dw_pw_k", p_dw_pw_k},
    {"ago_fused_dw_dw", p_dw_dw}, {"ago_fused_pw_pw", p_pw_pw}, {"ago_fused_conv_chain", p_conv_chain}, {"ago_fused_ffn", p_ffn},
    {"ago_fused_ffn_packed", p_ffn_packed}, {"ago_unfused_ffn", p_unfused_ffn}, {"ago_unfused_ffn_packed", p_unfused_ffn_packed},
    {"ago_pack_weight", p_pack_weight}, {"ago_gemm", p_gemm}, {"ago_gemm_packed", p_gemm_packed}, {"ago_conv1x1", p_conv1x1},
    {"ago_dwconv3x3", p_dwconv3x3}, {"ago_conv3x3", p_conv3x3}, {"ago_bias_act", p_bias_act}, {"ago_add_act", p_add_act},
    {"ago_fused_attn", p_attn}, {"ago_fused_attn_bshd", p_attn_bshd}, {"ago_fused_attn_bias", p_attn_bias}, {"ago_fused_qkv", p_qkv},
};

constexpr int kMaxArgs = 12;

// ---- Entry: the native form of one entry point ------------------------------------------------------------------
struct Entry {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    Parse parse;
    PyObject* names;              // tuple of argument names, in order
};
// ---- Launcher: a call marshalled once ----------------------------------------------------------------------------
struct Launcher {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    Launch launch;
};

int run_released(const Launch& l) {
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = l.run(l);
    Py_END_ALLOW_THREADS
    return st;
}

bool parse_call(Entry* e, PyObject* const* args, Py_ssize_t n, PyObject* kwnames, Launch& l) {
    PyObject* slots[kMaxArgs] = {};
    const Py_ssize_t total = PyTuple_GET_SIZE(e->names);
    if (n > total) return false;
    for (Py_ssize_t i = 0; i < n; ++i) slots[i] = args[i];
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t q = 0; q < nkw; ++q) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, q);
        Py_ssize_t at = -1;
        for (Py_ssize_t i = 0; i < total && at < 0; ++i)
            if (PyTuple_GET_ITEM(e->names, i) == name || PyUnicode_Compare(PyTuple_GET_ITEM(e->names, i), name) == 0) at = i;
        if (at < 0 || slots[at]) return false;
        slots[at] = args[n + q];
    }
    Args a{slots};
    l.ws = nullptr;
    l.ws_bytes = 0;
    try {
        if (!e->parse(a, l) || !a.ok) return false;
        l.stream = (void*)c10::hip::getCurrentHIPStream().stream();
    } catch (const std::exception&) {             // a tensor without storage and the like: the Python checks say what it is
        return false;
    }
    return true;
}

// ---- Sequence: several launchers issued in one go on the current stream ----------------------------------------------
struct Sequence {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    PyObject *launchers, *held;
};

PyObject* raise_status(int st) {
    PyObject* mod = PyImport_ImportModule("paper_2212_01005_amd.binding");
    PyObject* exc = mod ? PyObject_GetAttrString(mod, "AgoError") : nullptr;
    PyObject* arg = exc ? PyLong_FromLong(st) : nullptr;
    if (arg) PyErr_SetObject(exc, arg);
    Py_XDECREF(arg); Py_XDECREF(exc); Py_XDECREF(mod);
    return nullptr;
}

PyObject* entry_call(PyObject* self, PyObject* const* args, size_t nf, PyObject* kwnames) {
    Launch l;
    if (!parse_call((Entry*)self, args, PyVectorcall_NARGS(nf), kwnames, l)) Py_RETURN_NONE;
    return PyLong_FromLong(run_released(l));
}

PyObject* launcher_call(PyObject* self, PyObject* const*, size_t nf, PyObject* kwnames) {
    if (PyVectorcall_NARGS(nf) || (kwnames && PyTuple_GET_SIZE(kwnames))) {
        PyErr_SetString(PyExc_TypeError, "a launcher takes no arguments");
        return nullptr;
    }
    const int st = run_released(((Launcher*)self)->launch);
    if (st == 0) Py_RETURN_NONE;
    return raise_status(st);
}

PyObject* sequence_call(PyObject* self, PyObject* const*, size_t nf, PyObject* kwnames) {
    if (PyVectorcall_NARGS(nf) || (kwnames && PyTuple_GET_SIZE(kwnames))) {
        PyErr_SetString(PyExc_TypeError, "a launch sequence takes no arguments");
        return nullptr;
    }
    PyObject* ls = ((Sequence*)self)->launchers;
    const Py_ssize_t n = PyTuple_GET_SIZE(ls);
    void* stream = (void*)c10::hip::getCurrentHIPStream().stream();
    int st = 0;
    Py_INCREF(ls);
    Py_BEGIN_ALLOW_THREADS
    for (Py_ssize_t i = 0; i < n && st == 0; ++i) {
        Launch l = ((Launcher*)PyTuple_GET_ITEM(ls, i))->launch;      // a copy: another thread may issue the same list elsewhere
        l.stream = stream;
        st = l.run(l);
    }
    Py_END_ALLOW_THREADS
    Py_DECREF(ls);
    if (st == 0) Py_RETURN_NONE;
    return raise_status(st);
}

void entry_dealloc(PyObject* self) {
    Py_XDECREF(((Entry*)self)->names);
    PyTypeObject* tp = Py_TYPE(self);
    tp->tp_free(self);
    Py_DECREF(tp);
}
void launcher_dealloc(PyObject* self) {
    PyTypeObject* tp = Py_TYPE(self);
    tp->tp_free(self);
    Py_DECREF(tp);
}

void sequence_dealloc(PyObject* self) {
    Py_XDECREF(((Sequence*)self)->launchers);
    Py_XDECREF(((Sequence*)self)->held);
    PyTypeObject* tp = Py_TYPE(self);
    tp->tp_free(self);
    Py_DECREF(tp);
}

PyTypeObject *g_entry_type, *g_launcher_type, *g_sequence_type;

// entry.prepare(*args) -> Launcher, or None when the arguments do not pass
PyObject* entry_prepare(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
    Launch l;
    if (!parse_call((Entry*)self, args, n, kwnames, l)) Py_RETURN_NONE;
    Launcher* la = (Launcher*)g_launcher_type->tp_alloc(g_launcher_type, 0);
    if (!la) return nullptr;
    la->vectorcall = launcher_call;
    la->launch = l;
    return (PyObject*)la;
}

PyMethodDef kEntryMethods[] = {
    {"prepare", (PyCFunction)(void (*)(void))entry_prepare, METH_FASTCALL | METH_KEYWORDS, "marshal the arguments once; a launcher or None"},
    {nullptr, nullptr, 0, nullptr}};
PyMemberDef kEntryMembers[] = {{"__vectorcalloffset__", T_PYSSIZET, offsetof(Entry, vectorcall), READONLY, nullptr}, {nullptr, 0, 0, 0, nullptr}};
PyMemberDef kLauncherMembers[] = {{"__vectorcalloffset__", T_PYSSIZET, offsetof(Launcher, vectorcall), READONLY, nullptr},
                                  {nullptr, 0, 0, 0, nullptr}};
PyMemberDef kSequenceMembers[] = {{"__vectorcalloffset__", T_PYSSIZET, offsetof(Sequence, vectorcall), READONLY, nullptr},
                                  {nullptr, 0, 0, 0, nullptr}};
PyType_Slot kSequenceSlots[] = {{Py_tp_dealloc, (void*)sequence_dealloc}, {Py_tp_call, (void*)PyVectorcall_Call},
                                {Py_tp_members, kSequenceMembers}, {0, nullptr}};
PyType_Slot kEntrySlots[] = {{Py_tp_dealloc, (void*)entry_dealloc}, {Py_tp_call, (void*)PyVectorcall_Call}, {Py_tp_methods, kEntryMethods},
                             {Py_tp_members, kEntryMembers}, {0, nullptr}};
PyType_Slot kLauncherSlots[] = {{Py_tp_dealloc, (void*)launcher_dealloc}, {Py_tp_call, (void*)PyVectorcall_Call},
                                {Py_tp_members, kLauncherMembers}, {0, nullptr}};
PyType_Spec kEntrySpec = {"_agocall.Entry", sizeof(Entry), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL, kEntrySlots};
PyType_Spec kSequenceSpec = {"_agocall.Sequence", sizeof(Sequence), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL, kSequenceSlots};
PyType_Spec kLauncherSpec = {"_agocall.Launcher", sizeof(Launcher), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL, kLauncherSlots};

// entry(name, argument names) -> Entry, or None for an entry point that is marshalled in Python only
PyObject* make_entry(PyObject*, PyObject* args) {
    const char* name;
    PyObject* names;
    if (!PyArg_ParseTuple(args, "sO!", &name, &PyTuple_Type, &names)) return nullptr;
    for (const auto& k : kEntries) {
        if (strcmp(k.name, name) != 0 || PyTuple_GET_SIZE(names) > kMaxArgs) continue;
        Entry* e = (Entry*)g_entry_type->tp_alloc(g_entry_type, 0);
        if (!e) return nullptr;
        e->vectorcall = entry_call;
        e->parse = k.parse;
        Py_INCREF(names);
        e->names = names;
        return (PyObject*)e;
    }
    Py_RETURN_NONE;
}

// sequence(tuple of launchers, held) -> Sequence
PyObject* make_sequence(PyObject*, PyObject* args) {
    PyObject *ls, *held;
    if (!PyArg_ParseTuple(args, "O!O", &PyTuple_Type, &ls, &held)) return nullptr;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(ls); ++i)
        if (Py_TYPE(PyTuple_GET_ITEM(ls, i)) != g_launcher_type) {
            PyErr_SetString(PyExc_TypeError, "a launch sequence is made of launchers");
            return nullptr;
        }
    Sequence* q = (Sequence*)g_sequence_type->tp_alloc(g_sequence_type, 0);
    if (!q) return nullptr;
    q->vectorcall = sequence_call;
    Py_INCREF(ls);
    Py_INCREF(held);
    q->launchers = ls;
    q->held = held;
    return (PyObject*)q;
}

PyMethodDef kMethods[] = {{"sequence", make_sequence, METH_VARARGS, "launchers issued in one go"},
                          {"entry", make_entry, METH_VARARGS, "the native form of an entry point, or None"}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_agocall", "native marshalling of the binding", -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__agocall(void) {
    PyObject* m = PyModule_Create(&kModule);
    if (!m) return nullptr;
    g_entry_type = (PyTypeObject*)PyType_FromSpec(&kEntrySpec);
    g_launcher_type = (PyTypeObject*)PyType_FromSpec(&kLauncherSpec);
    g_sequence_type = (PyTypeObject*)PyType_FromSpec(&kSequenceSpec);
    if (!g_entry_type || !g_launcher_type || !g_sequence_type) { Py_DECREF(m); return nullptr; }
    return m;
}
