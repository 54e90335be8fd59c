// The per-layer entry points of libpsw called without ctypes: a CPython module
// that takes the arguments of psw.py's functions, checks the tensors as
// psw._ptr does and calls the C function.
//
// Marshalling with ctypes cost 6 us a call (max-pool) to 14 us (batch norm),
// more than the small layers' kernels take: batch norm forward and backward of
// 40x32x16x16 took 31 us and takes 15 with these calls, a 64 to 10 classifier
// of 128 samples with its loss, three calls, 24.6 and 20.4 (its kernels' time).  A function
// returns the C status, or None when an argument is anything but what the
// common case has (device tensors, contiguous, float32 / int32 / uint8; plain
// numbers), and psw.py then takes its own path, which also raises the errors.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <exception>

#include "../../include/psw.h"

namespace {

struct Entry {
    const char* name;
    void* fn;
};
Entry g_fns[] = {
    {"psw_conv_fwd", nullptr},        {"psw_conv_bwd_data", nullptr}, {"psw_conv_bwd_weight", nullptr},
    {"psw_bn_relu_fwd", nullptr},     {"psw_bn_relu_bwd", nullptr},   {"psw_pool_fwd", nullptr},
    {"psw_pool_bwd", nullptr},        {"psw_fc_fwd", nullptr},        {"psw_fc_bwd", nullptr},
    {"psw_relu_mask", nullptr},       {"psw_softmax_xent", nullptr},  {"psw_sgd_momentum_step", nullptr},
};
enum { CONV_FWD, CONV_DX, CONV_DW, BN_FWD, BN_BWD, POOL_FWD, POOL_BWD, FC_FWD, FC_BWD, RELU_MASK, XENT, SGD };

// The arguments of one call; `ok` turns false at the first that is not of the
// common case.
struct Args {
    PyObject* const* a;
    bool ok = true;

    const at::Tensor* tensor(int i)
    {
        // exact: a subclass may give its own data_ptr()
        if (!ok || !THPVariable_CheckExact(a[i])) {
            ok = false;
            return nullptr;
        }
        const at::Tensor& t = THPVariable_Unpack(a[i]);
        const auto ty = t.defined() ? t.scalar_type() : at::kDouble;
        if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided ||
            (ty != at::kFloat && ty != at::kInt && ty != at::kByte) || !t.is_contiguous() || t.numel() == 0)
            ok = false;
        return &t;
    }
    void* ptr(int i) { return ptr_of(tensor(i)); }
    void* opt(int i) { return a[i] == Py_None ? nullptr : ptr(i); }
    void* ptr_of(const at::Tensor* t) { return ok ? t->data_ptr() : nullptr; }
    int64_t num(int i)
    {
        if (!ok || !PyLong_Check(a[i])) {  // bools are ints
            ok = false;
            return 0;
        }
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(a[i], &over);
        if (over) ok = false;
        return v;
    }
    int i32(int i)
    {
        const int64_t v = num(i);
        if (v < INT32_MIN || v > INT32_MAX) ok = false;
        return (int)v;
    }
    float real(int i)
    {
        if (!ok || !PyFloat_Check(a[i])) {
            ok = false;
            return 0.f;
        }
        return (float)PyFloat_AS_DOUBLE(a[i]);
    }
    // None: the current stream
    void* stream(int i)
    {
        if (a[i] != Py_None) return (void*)num(i);
        return ok ? (void*)c10::hip::getCurrentHIPStream().stream() : nullptr;
    }
    // the n sizes of a tensor of n dimensions
    size_t numel(const at::Tensor* t) { return ok ? (size_t)t->numel() : 0; }
    template <int N>
    struct Dims {
        int d[N];
    };
    template <int N>
    Dims<N> dims(const at::Tensor* t)
    {
        Dims<N> r{};
        if (!ok || t->dim() != N) {
            ok = false;
            return r;
        }
        for (int k = 0; k < N; ++k) {
            const int64_t v = t->size(k);
            if (v > INT32_MAX) ok = false;
            r.d[k] = (int)v;
        }
        return r;
    }
    // a shape given as a tuple of four ints
    Dims<4> shape(int i)
    {
        Dims<4> r{};
        if (!ok || !PyTuple_Check(a[i]) || PyTuple_GET_SIZE(a[i]) != 4) {
            ok = false;
            return r;
        }
        for (int k = 0; k < 4; ++k) {
            PyObject* o = PyTuple_GET_ITEM(a[i], k);
            const long v = PyLong_Check(o) ? PyLong_AsLong(o) : -1;
            if (v < 0 || v > INT32_MAX) ok = false;
            r.d[k] = (int)v;
        }
        if (PyErr_Occurred()) PyErr_Clear();
        return r;
    }
};

template <typename F>
F fn(int which)
{
    return (F)g_fns[which].fn;
}

// calls `call()` when every argument was of the common case
template <typename C>
PyObject* finish(const Args& g, int which, C call)
{
    if (!g.ok || !g_fns[which].fn) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = call();
    Py_END_ALLOW_THREADS return PyLong_FromLong(rc);
}

// x, w, y, stride, pad, bias, relu, bf16, stream
PyObject* conv_fwd(Args g)
{
    const at::Tensor *x = g.tensor(0), *w = g.tensor(1);
    const auto X = g.dims<4>(x);
    const auto W = g.dims<4>(w);
    void *px = g.ptr_of(x), *pw = g.ptr_of(w), *py = g.ptr(2), *pb = g.opt(5);
    const int st = g.i32(3), pad = g.i32(4), relu = g.i32(6), prec = g.i32(7) ? PSW_BF16 : PSW_FP32;
    void* s = g.stream(8);
    return finish(g, CONV_FWD, [&] {
        return fn<decltype(&psw_conv_fwd)>(CONV_FWD)(X.d[0], X.d[1], X.d[2], X.d[3], W.d[0], W.d[2], W.d[3], st, pad,
                                                     (float*)px, (float*)pw, (float*)pb, relu, (float*)py, prec, s);
    });
}

// x_shape, w, dy, dx, stride, pad, accumulate, bf16, stream
PyObject* conv_bwd_data(Args g)
{
    const auto X = g.shape(0);
    const at::Tensor* w = g.tensor(1);
    const auto W = g.dims<4>(w);
    void *pw = g.ptr_of(w), *pdy = g.ptr(2), *pdx = g.ptr(3);
    const int st = g.i32(4), pad = g.i32(5), acc = g.i32(6), prec = g.i32(7) ? PSW_BF16 : PSW_FP32;
    void* s = g.stream(8);
    return finish(g, CONV_DX, [&] {
        return fn<decltype(&psw_conv_bwd_data)>(CONV_DX)(X.d[0], X.d[1], X.d[2], X.d[3], W.d[0], W.d[2], W.d[3], st, pad,
                                                         (float*)pw, (float*)pdy, (float*)pdx, acc, prec, s);
    });
}

// x, dy, dw, stride, pad, dbias, bf16, ws, stream
PyObject* conv_bwd_weight(Args g)
{
    const at::Tensor *x = g.tensor(0), *dw = g.tensor(2), *ws = g.tensor(7);
    const auto X = g.dims<4>(x);
    const auto W = g.dims<4>(dw);
    void *px = g.ptr_of(x), *pdy = g.ptr(1), *pdw = g.ptr_of(dw), *pdb = g.opt(5), *pws = g.ptr_of(ws);
    const int st = g.i32(3), pad = g.i32(4), prec = g.i32(6) ? PSW_BF16 : PSW_FP32;
    const size_t ws_bytes = g.ok ? (size_t)ws->nbytes() : 0;
    void* s = g.stream(8);
    return finish(g, CONV_DW, [&] {
        return fn<decltype(&psw_conv_bwd_weight)>(CONV_DW)(X.d[0], X.d[1], X.d[2], X.d[3], W.d[0], W.d[2], W.d[3], st, pad,
                                                           (float*)px, (float*)pdy, (float*)pdw, (float*)pdb, prec, pws,
                                                           ws_bytes, s);
    });
}

// y, gamma, beta, z, save_mean, save_invstd, res, relu, eps, momentum, run_mean, run_var, ws, stream
PyObject* bn_relu_fwd(Args g)
{
    const at::Tensor *y = g.tensor(0), *ws = g.tensor(12);
    const auto Y = g.dims<4>(y);
    void *py = g.ptr_of(y), *pg = g.ptr(1), *pb = g.ptr(2), *pz = g.ptr(3), *pm = g.ptr(4), *pi = g.ptr(5);
    Args::Dims<4> R{};
    void* pr = nullptr;
    if (g.a[6] != Py_None) {
        const at::Tensor* r = g.tensor(6);
        R = g.dims<4>(r);
        pr = g.ptr_of(r);
    }
    const int relu = g.i32(7);
    const float eps = g.real(8), mom = g.real(9);
    void *rm = g.opt(10), *rv = g.opt(11), *pws = g.ptr_of(ws);
    const size_t ws_bytes = g.numel(ws);
    void* s = g.stream(13);
    return finish(g, BN_FWD, [&] {
        return fn<decltype(&psw_bn_relu_fwd)>(BN_FWD)(Y.d[0], Y.d[1], Y.d[2], Y.d[3], (float*)py, (float*)pg, (float*)pb,
                                                      (float*)pr, R.d[1], R.d[2], R.d[3], relu, eps, mom, (float*)pz,
                                                      (float*)pm, (float*)pi, (float*)rm, (float*)rv, pws,
                                                      ws_bytes, s);
    });
}

// dz, z, y, gamma, save_mean, save_invstd, dy, dgamma, dbeta, dres, relu, res_accumulate, ws, stream
PyObject* bn_relu_bwd(Args g)
{
    const at::Tensor *y = g.tensor(2), *ws = g.tensor(12);
    const auto Y = g.dims<4>(y);
    void *pdz = g.ptr(0), *pz = g.ptr(1), *py = g.ptr_of(y), *pg = g.ptr(3), *pm = g.ptr(4), *pi = g.ptr(5);
    void *pdy = g.ptr(6), *pdg = g.ptr(7), *pdb = g.ptr(8);
    Args::Dims<4> R{};
    void* pr = nullptr;
    if (g.a[9] != Py_None) {
        const at::Tensor* r = g.tensor(9);
        R = g.dims<4>(r);
        pr = g.ptr_of(r);
    }
    const int relu = g.i32(10), acc = g.i32(11);
    void* pws = g.ptr_of(ws);
    const size_t ws_bytes = g.numel(ws);
    void* s = g.stream(13);
    return finish(g, BN_BWD, [&] {
        return fn<decltype(&psw_bn_relu_bwd)>(BN_BWD)(Y.d[0], Y.d[1], Y.d[2], Y.d[3], (float*)pdz, (float*)pz, (float*)py,
                                                      (float*)pg, (float*)pm, (float*)pi, relu, (float*)pdy, (float*)pdg,
                                                      (float*)pdb, (float*)pr, R.d[1], R.d[2], R.d[3], acc, pws,
                                                      ws_bytes, s);
    });
}

// kind, x, y, k, stride, argmax, stream
PyObject* pool_fwd(Args g)
{
    const int kind = g.i32(0);
    const at::Tensor* x = g.tensor(1);
    const auto X = g.dims<4>(x);
    void *px = g.ptr_of(x), *py = g.ptr(2), *pa = g.opt(5);
    const int k = g.i32(3), st = g.i32(4);
    void* s = g.stream(6);
    return finish(g, POOL_FWD, [&] {
        return fn<decltype(&psw_pool_fwd)>(POOL_FWD)(kind, X.d[0], X.d[1], X.d[2], X.d[3], k, st, (float*)px, (float*)py,
                                                     (int32_t*)pa, s);
    });
}

// kind, x_shape, dy, dx, k, stride, argmax, accumulate, stream
PyObject* pool_bwd(Args g)
{
    const int kind = g.i32(0);
    const auto X = g.shape(1);
    void *pdy = g.ptr(2), *pdx = g.ptr(3), *pa = g.opt(6);
    const int k = g.i32(4), st = g.i32(5), acc = g.i32(7);
    void* s = g.stream(8);
    return finish(g, POOL_BWD, [&] {
        return fn<decltype(&psw_pool_bwd)>(POOL_BWD)(kind, X.d[0], X.d[1], X.d[2], X.d[3], k, st, (float*)pdy,
                                                     (int32_t*)pa, (float*)pdx, acc, s);
    });
}

// x, w, y, b, relu, bf16, stream
PyObject* fc_fwd(Args g)
{
    const at::Tensor *x = g.tensor(0), *w = g.tensor(1);
    const auto X = g.dims<2>(x);
    const int out = g.ok && w->dim() >= 1 && w->size(0) <= INT32_MAX ? (int)w->size(0) : (g.ok = false, 0);
    void *px = g.ptr_of(x), *pw = g.ptr_of(w), *py = g.ptr(2), *pb = g.opt(3);
    const int relu = g.i32(4), prec = g.i32(5) ? PSW_BF16 : PSW_FP32;
    void* s = g.stream(6);
    return finish(g, FC_FWD, [&] {
        return fn<decltype(&psw_fc_fwd)>(FC_FWD)(X.d[0], X.d[1], out, (float*)px, (float*)pw, (float*)pb, relu, (float*)py,
                                                 prec, s);
    });
}

// x, w, dy, dw, dx, db, dx_accumulate, bf16, ws, stream
PyObject* fc_bwd(Args g)
{
    const at::Tensor *x = g.tensor(0), *w = g.tensor(1), *ws = g.tensor(8);
    const auto X = g.dims<2>(x);
    const int out = g.ok && w->dim() >= 1 && w->size(0) <= INT32_MAX ? (int)w->size(0) : (g.ok = false, 0);
    void *px = g.ptr_of(x), *pw = g.ptr_of(w), *pdy = g.ptr(2), *pdw = g.ptr(3), *pdx = g.opt(4), *pdb = g.opt(5);
    const int acc = g.i32(6), prec = g.i32(7) ? PSW_BF16 : PSW_FP32;
    void* pws = g.ptr_of(ws);
    const size_t ws_bytes = g.numel(ws);
    void* s = g.stream(9);
    return finish(g, FC_BWD, [&] {
        return fn<decltype(&psw_fc_bwd)>(FC_BWD)(X.d[0], X.d[1], out, (float*)px, (float*)pw, (float*)pdy, (float*)pdx, acc,
                                                 (float*)pdw, (float*)pdb, prec, pws, ws_bytes, s);
    });
}

// z, g, stream
PyObject* relu_mask(Args g)
{
    const at::Tensor* z = g.tensor(0);
    void *pz = g.ptr_of(z), *pg = g.ptr(1);
    void* s = g.stream(2);
    const int64_t numel = (int64_t)g.numel(z);
    return finish(g, RELU_MASK, [&] {
        return fn<decltype(&psw_relu_mask)>(RELU_MASK)(numel, (float*)pz, (float*)pg, s);
    });
}

// logits, labels, loss, dlogits, stream
PyObject* softmax_xent(Args g)
{
    const at::Tensor* z = g.tensor(0);
    const auto Z = g.dims<2>(z);
    void *pz = g.ptr_of(z), *pl = g.ptr(1), *po = g.ptr(2), *pd = g.ptr(3);
    void* s = g.stream(4);
    return finish(g, XENT, [&] {
        return fn<decltype(&psw_softmax_xent)>(XENT)(Z.d[0], Z.d[1], (float*)pz, (int32_t*)pl, (float*)po, (float*)pd, s);
    });
}

// w_in, w_out, v, g, lr, mom, wd, nesterov, stream
PyObject* sgd(Args g)
{
    const at::Tensor* w = g.tensor(0);
    void *pw = g.ptr_of(w), *po = g.ptr(1), *pv = g.ptr(2), *pg = g.ptr(3);
    const float lr = g.real(4), mom = g.real(5), wd = g.real(6);
    const int nest = g.i32(7);
    void* s = g.stream(8);
    const int64_t numel = (int64_t)g.numel(w);
    return finish(g, SGD, [&] {
        return fn<decltype(&psw_sgd_momentum_step)>(SGD)(numel, (float*)pw, (float*)po, (float*)pv, (float*)pg, lr, mom,
                                                         wd, nest, s);
    });
}

// The Python entry of F: a tensor without storage makes data_ptr() throw, and
// the caller's own path then raises that error.
template <PyObject* (*F)(Args), int COUNT>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t count)
{
    if (count != COUNT) Py_RETURN_NONE;
    try {
        return F(Args{a});
    } catch (const std::exception&) {
        Py_RETURN_NONE;
    }
}

// bind(name, address): the loaded library's function
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t count)
{
    if (count != 2) {
        PyErr_SetString(PyExc_TypeError, "bind(name, address)");
        return nullptr;
    }
    const char* name = PyUnicode_AsUTF8(a[0]);
    if (!name) return nullptr;
    void* p = PyLong_AsVoidPtr(a[1]);
    if (PyErr_Occurred()) return nullptr;
    for (Entry& e : g_fns)
        if (!strcmp(e.name, name)) e.fn = p;
    Py_RETURN_NONE;
}

#define PSW_DEF(F, COUNT) {#F, (PyCFunction)(void (*)(void))entry<F, COUNT>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    PSW_DEF(conv_fwd, 9),
    PSW_DEF(conv_bwd_data, 9),
    PSW_DEF(conv_bwd_weight, 9),
    PSW_DEF(bn_relu_fwd, 14),
    PSW_DEF(bn_relu_bwd, 14),
    PSW_DEF(pool_fwd, 7),
    PSW_DEF(pool_bwd, 9),
    PSW_DEF(fc_fwd, 7),
    PSW_DEF(fc_bwd, 10),
    PSW_DEF(relu_mask, 3),
    PSW_DEF(softmax_xent, 5),
    PSW_DEF(sgd, 9),
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&g_module); }
