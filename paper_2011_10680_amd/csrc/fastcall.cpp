// Argument marshalling of the per-layer entry points for CPython, in C: module `_fastcall`.
//
// A small layer's call is bound by the host: a kernel launch takes 2.5 us, and the same call through ctypes (a descriptor by
// reference, ten pointers converted one by one, the stream handle) took 2.7 us on top of it: 56x56x64 at batch 1 4.7 us a call
// where its kernel needs 3.6, a module of nine small launches 44 us where they need 26.  Through here the marshalling takes 0.5 us.
//
// Every function returns the C function's status, or None for any argument that is not of the exact usual type (a
// torch.Tensor or Parameter, an int, the descriptor class): the caller then takes the ctypes path, whose conversions and
// errors are the reference.  Nothing is kept from one call to the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <initializer_list>

#include "../../include/hawq.h"

namespace {

struct Library {
    decltype(&hawq_conv2d_int) conv2d;
    decltype(&hawq_conv2d_dual_int) dual;
    decltype(&hawq_gemm_int) gemm;
    decltype(&hawq_residual_add_dyadic) residual_add;
    decltype(&hawq_avgpool_int) avgpool;
    decltype(&hawq_maxpool_int) maxpool;
    decltype(&hawq_pool2d_sum_int) pool2d_sum;
    decltype(&hawq_concat_dyadic) concat;
} lib;

PyTypeObject *tensor_type, *parameter_type, *desc_type;   // exact types taken here
PyCFunction tensor_data_ptr, tensor_numel;                // torch.Tensor's methods
PyObject *get_device, *get_stream;                        // torch's raw queries of the current device and its current stream

// One call's arguments, taken in order.  `ok` turns false on the first one that is not of the usual type.
struct Args {
    PyObject *const *at, *const *end;
    Py_buffer views[2];
    int n_views = 0;
    bool ok = true;

    Args(PyObject *const *a, Py_ssize_t n, Py_ssize_t want) : at(a), end(a + n) { ok = n == want; }
    ~Args() { while (n_views > 0) PyBuffer_Release(&views[--n_views]); }

    static bool is_tensor(PyObject *o) { return Py_TYPE(o) == tensor_type || Py_TYPE(o) == parameter_type; }
    static bool call_int(PyObject *tensor, PyCFunction f, int64_t &v) {
        PyObject *r = f(tensor, nullptr);
        if (r == nullptr) { PyErr_Clear(); return false; }
        v = PyLong_Check(r) ? (int64_t)PyLong_AsUnsignedLongLongMask(r) : -1;
        const bool good = PyLong_Check(r) && !PyErr_Occurred();
        Py_DECREF(r);
        PyErr_Clear();
        return good;
    }
    void *tensor(PyObject *o) {
        int64_t p = 0;
        if (!is_tensor(o) || !call_int(o, tensor_data_ptr, p)) { ok = false; return nullptr; }
        return (void *)(intptr_t)p;
    }
    template <class T = void>
    T *ptr() {
        if (!ok) return nullptr;
        PyObject *o = *at++;
        return o == Py_None ? nullptr : (T *)tensor(o);
    }
    int64_t i64() {
        if (!ok) return 0;
        PyObject *o = *at++;
        int overflow = 0;
        const long long v = PyLong_Check(o) ? PyLong_AsLongLongAndOverflow(o, &overflow) : 0;
        if (!PyLong_Check(o) || overflow != 0) ok = false;
        return v;
    }
    int32_t i32() { return (int32_t)i64(); }
    const hawq_conv_desc *desc() {
        if (!ok) return nullptr;
        PyObject *o = *at++;
        if (Py_TYPE(o) != desc_type || PyObject_GetBuffer(o, &views[n_views], PyBUF_SIMPLE) != 0) { PyErr_Clear(); ok = false; return nullptr; }
        const Py_buffer &v = views[n_views++];
        if ((size_t)v.len < sizeof(hawq_conv_desc)) ok = false;
        return (const hawq_conv_desc *)v.buf;
    }
    // the stream argument: a handle, or None for the current device's current stream
    void *stream() {
        if (!ok) return nullptr;
        PyObject *o = *at++;
        if (o != Py_None) {
            if (!PyLong_Check(o)) { ok = false; return nullptr; }
            void *p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
            if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
            return p;
        }
        PyObject *dev = PyObject_CallNoArgs(get_device), *s = dev != nullptr ? PyObject_CallOneArg(get_stream, dev) : nullptr;
        void *p = nullptr;
        if (s != nullptr && PyLong_Check(s)) p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(s);
        else ok = false;
        Py_XDECREF(dev);
        Py_XDECREF(s);
        PyErr_Clear();
        return p;
    }
};

// the library's call, other threads running meanwhile (a launch waits when its queue is full)
template <class F>
PyObject *status_of(bool ok, F &&f) {
    if (!ok) Py_RETURN_NONE;
    hawq_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

PyObject *conv2d(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 11);
    const hawq_conv_desc *d = g.desc();
    const void *x = g.ptr(), *w = g.ptr();
    const int32_t *bias = g.ptr<int32_t>(), *b = g.ptr<int32_t>();
    const uint8_t *c = g.ptr<uint8_t>();
    const void *res = g.ptr();
    const int32_t *rb = g.ptr<int32_t>();
    const uint8_t *rc = g.ptr<uint8_t>();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.conv2d(d, x, w, bias, b, c, res, rb, rc, y, s); });
}

PyObject *dual(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 14);
    const hawq_conv_desc *d = g.desc();
    const void *x = g.ptr(), *w = g.ptr();
    const int32_t *bias = g.ptr<int32_t>(), *b = g.ptr<int32_t>();
    const uint8_t *c = g.ptr<uint8_t>();
    const hawq_conv_desc *ds = g.desc();
    const void *xs = g.ptr(), *ws = g.ptr();
    const int32_t *bias_s = g.ptr<int32_t>(), *b_s = g.ptr<int32_t>();
    const uint8_t *c_s = g.ptr<uint8_t>();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.dual(d, x, w, bias, b, c, ds, xs, ws, bias_s, b_s, c_s, y, s); });
}

PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 16);
    const int32_t M = g.i32(), N = g.i32(), K = g.i32(), x_dt = g.i32(), w_dt = g.i32(), y_dt = g.i32();
    const void *x = g.ptr(), *w = g.ptr();
    const int32_t *bias = g.ptr<int32_t>(), *b = g.ptr<int32_t>();
    const uint8_t *c = g.ptr<uint8_t>();
    const int32_t relu = g.i32(), lo = g.i32(), hi = g.i32();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.gemm(M, N, K, x_dt, w_dt, y_dt, x, w, bias, b, c, relu, lo, hi, y, s); });
}

PyObject *residual_add(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 16);
    const int64_t P = g.i64();
    const int32_t K = g.i32(), m_dt = g.i32(), r_dt = g.i32(), y_dt = g.i32();
    const void *m = g.ptr();
    const int32_t *mb = g.ptr<int32_t>();
    const uint8_t *mc = g.ptr<uint8_t>();
    const void *r = g.ptr();
    const int32_t *rb = g.ptr<int32_t>();
    const uint8_t *rc = g.ptr<uint8_t>();
    const int32_t relu = g.i32(), lo = g.i32(), hi = g.i32();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.residual_add(P, K, m_dt, r_dt, y_dt, m, mb, mc, r, rb, rc, relu, lo, hi, y, s); });
}

PyObject *avgpool(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 13);
    const int32_t N = g.i32(), H = g.i32(), W = g.i32(), C = g.i32(), x_dt = g.i32(), y_dt = g.i32();
    const void *x = g.ptr();
    const int32_t *b = g.ptr<int32_t>();
    const uint8_t *c = g.ptr<uint8_t>();
    const int32_t lo = g.i32(), hi = g.i32();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.avgpool(N, H, W, C, x_dt, y_dt, x, b, c, lo, hi, y, s); });
}

PyObject *maxpool(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 11);
    const int32_t N = g.i32(), H = g.i32(), W = g.i32(), C = g.i32(), x_dt = g.i32(), y_dt = g.i32();
    const void *x = g.ptr();
    const int32_t lo = g.i32(), hi = g.i32();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.maxpool(N, H, W, C, x_dt, y_dt, x, lo, hi, y, s); });
}

PyObject *pool2d_sum(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 19);
    int32_t v[12];
    for (int32_t &i : v) i = g.i32();
    const void *x = g.ptr();
    const int32_t *b = g.ptr<int32_t>();
    const uint8_t *c = g.ptr<uint8_t>();
    const int32_t lo = g.i32(), hi = g.i32();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.pool2d_sum(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11], x, b, c, lo, hi, y, s); });
}

// (n_pixels, branches, y_dt, y_lo, y_hi, y, stream); branches: a list of (q, dtype, b, c) tuples
PyObject *concat(PyObject *, PyObject *const *a, Py_ssize_t n) {
    Args g(a, n, 7);
    const int64_t P = g.i64();
    constexpr Py_ssize_t kMost = 32;                 // (longer lists take the general path)
    hawq_concat_branch br[kMost];
    Py_ssize_t count = 0;
    if (g.ok) {
        PyObject *list = *g.at++;
        g.ok = PyList_CheckExact(list) && PyList_GET_SIZE(list) <= kMost;
        if (g.ok) count = PyList_GET_SIZE(list);
        for (Py_ssize_t i = 0; g.ok && i < count; ++i) {
            PyObject *t = PyList_GET_ITEM(list, i);
            if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) != 4) { g.ok = false; break; }
            PyObject *dt = PyTuple_GET_ITEM(t, 1), *b = PyTuple_GET_ITEM(t, 2);
            int overflow = 0;
            int64_t K = 0;
            br[i].q = g.tensor(PyTuple_GET_ITEM(t, 0));
            br[i].b = (const int32_t *)g.tensor(b);
            br[i].c = (const uint8_t *)g.tensor(PyTuple_GET_ITEM(t, 3));
            br[i].dtype = PyLong_Check(dt) ? (int32_t)PyLong_AsLongLongAndOverflow(dt, &overflow) : 0;
            if (!g.ok || !PyLong_Check(dt) || overflow != 0 || !Args::call_int(b, tensor_numel, K)) { g.ok = false; break; }
            br[i].K = (int32_t)K;
        }
    }
    const int32_t y_dt = g.i32(), lo = g.i32(), hi = g.i32();
    void *y = g.ptr(), *s = g.stream();
    return status_of(g.ok, [&] { return lib.concat(P, (int32_t)count, br, y_dt, lo, hi, y, s); });
}

bool no_args_method(PyObject *o, PyCFunction &f) {
    if (Py_TYPE(o) != &PyMethodDescr_Type) return false;
    const PyMethodDef *m = ((PyMethodDescrObject *)o)->d_method;
    f = m->ml_meth;
    return m->ml_flags == METH_NOARGS;
}

// setup(addresses of the eight entry points, torch.Tensor, torch.nn.Parameter, the descriptor class, device query, stream query):
// whether the functions above may be used.
PyObject *setup(PyObject *, PyObject *args) {
    PyObject *addr, *tensor, *param, *desc, *device, *stream;
    if (!PyArg_ParseTuple(args, "O!OOOOO", &PyTuple_Type, &addr, &tensor, &param, &desc, &device, &stream)) return nullptr;
    if (PyTuple_GET_SIZE(addr) != 8 || !PyType_Check(tensor) || !PyType_Check(param) || !PyType_Check(desc)) Py_RETURN_FALSE;
    uintptr_t p[8];
    for (int i = 0; i < 8; ++i) {
        p[i] = (uintptr_t)PyLong_AsUnsignedLongLong(PyTuple_GET_ITEM(addr, i));
        if (PyErr_Occurred()) return nullptr;
    }
    PyObject *dp = PyObject_GetAttrString(tensor, "data_ptr"), *nu = PyObject_GetAttrString(tensor, "numel");
    const bool good = dp != nullptr && nu != nullptr && no_args_method(dp, tensor_data_ptr) && no_args_method(nu, tensor_numel);
    Py_XDECREF(dp);
    Py_XDECREF(nu);
    if (!good) { PyErr_Clear(); Py_RETURN_FALSE; }
    lib = {(decltype(lib.conv2d))p[0], (decltype(lib.dual))p[1], (decltype(lib.gemm))p[2], (decltype(lib.residual_add))p[3],
           (decltype(lib.avgpool))p[4], (decltype(lib.maxpool))p[5], (decltype(lib.pool2d_sum))p[6], (decltype(lib.concat))p[7]};
    for (PyObject *o : {tensor, param, desc, device, stream}) Py_INCREF(o);   // (for the life of the process)
    tensor_type = (PyTypeObject *)tensor;
    parameter_type = (PyTypeObject *)param;
    desc_type = (PyTypeObject *)desc;
    get_device = device;
    get_stream = stream;
    Py_RETURN_TRUE;
}

#define HAWQ_FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HAWQ_FAST(conv2d), HAWQ_FAST(dual), HAWQ_FAST(gemm), HAWQ_FAST(residual_add), HAWQ_FAST(avgpool), HAWQ_FAST(maxpool),
                         HAWQ_FAST(pool2d_sum), HAWQ_FAST(concat), {"setup", setup, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&module); }
