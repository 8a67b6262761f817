// The calls a serving loop makes for every Matmul -- ft_plan_cached, ft_launch, ft_launch_epilogue -- as CPython functions.
//
// Small launches take 3 to 5 us of GPU time, and a pass of shape, look-up and launch took the host 4.6 to 5.3 us: 2.3 in HIP, 0.85 in the
// look-up's ctypes call and 0.4 around the launch's, the rest in the interpreter.  Here a call reads its arguments straight from the
// objects, look-up 0.17 us (0.6 with the shape object that it takes), launch 2.65, pass 3.4 to 4.2 by the host's state: 77 x 768 x 768 goes
// from 4.7-5.3 us to 3.75-4.4, 105 x 3072 x 768 with 16-bit results from 4.65-5.05 to 4.20, which is GPU time.
// What these functions do not read themselves -- keywords, addresses that are neither int nor None, a shape of another type, a
// library not loaded yet -- they hand to the ctypes functions of the same name in binding.py, which also define the errors.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "ftuner.h"

namespace {

typedef ft_status (*cached_fn)(const ft_op *, ft_ukset *, const ft_shape *, uint32_t, const ft_plan **);
typedef ft_status (*launch_fn)(const ft_plan *, const void *, const void *, void *, void *);
typedef ft_status (*epilogue_fn)(const ft_plan *, const void *, const void *, void *, const float *, void *);

// set once by bind(), under the interpreter's lock
cached_fn g_cached;
launch_fn g_launch;
epilogue_fn g_epilogue;
PyObject *g_check, *g_shape, *g_plan, *g_slow_cached, *g_slow_launch, *g_slow_epilogue;
PyObject *s_ptr, *s_owner, *g_no_args;

// an address as ctypes' c_void_p takes it from an int or None
bool address(PyObject *o, void **out) {
    if (o == Py_None) { *out = nullptr; return true; }
    if (!PyLong_CheckExact(o)) return false;
    *out = reinterpret_cast<void *>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(o)));
    return true;
}
bool pointer_of(PyObject *handle, void **out) {
    PyObject *p = PyObject_GetAttr(handle, s_ptr);
    if (!p) { PyErr_Clear(); return false; }                          // (the ctypes function raises it again)
    const bool ok = address(p, out);
    Py_DECREF(p);
    return ok;
}
PyObject *checked(ft_status st, const char *what) {
    if (st == FT_OK) Py_RETURN_NONE;
    return PyObject_CallFunction(g_check, "is", (int)st, what);
}

PyObject *launch(PyObject *, PyObject *const *a, Py_ssize_t n, PyObject *kw) {
    void *p[5] = {};
    bool plain = g_launch && !kw && (n == 4 || n == 5) && pointer_of(a[0], &p[0]);
    for (Py_ssize_t i = 1; plain && i < n; ++i) plain = address(a[i], &p[i]);
    if (!plain) return PyObject_Vectorcall(g_slow_launch, a, n, kw);
    ft_status st;
    Py_BEGIN_ALLOW_THREADS
    st = g_launch(static_cast<const ft_plan *>(p[0]), p[1], p[2], p[3], p[4]);
    Py_END_ALLOW_THREADS
    return checked(st, "ft_launch");
}

PyObject *launch_epilogue(PyObject *, PyObject *const *a, Py_ssize_t n, PyObject *kw) {
    void *p[6] = {};
    bool plain = g_epilogue && !kw && (n == 5 || n == 6) && pointer_of(a[0], &p[0]);
    for (Py_ssize_t i = 1; plain && i < n; ++i) plain = address(a[i], &p[i]);
    if (!plain) return PyObject_Vectorcall(g_slow_epilogue, a, n, kw);
    ft_status st;
    Py_BEGIN_ALLOW_THREADS
    st = g_epilogue(static_cast<const ft_plan *>(p[0]), p[1], p[2], p[3], static_cast<const float *>(p[4]), p[5]);
    Py_END_ALLOW_THREADS
    return checked(st, "ft_launch_epilogue");
}

PyObject *plan_cached(PyObject *, PyObject *const *a, Py_ssize_t n, PyObject *kw) {
    void *op, *set;
    Py_buffer shape;
    if (!g_cached || kw || n != 3 || (PyObject *)Py_TYPE(a[2]) != g_shape || !pointer_of(a[0], &op) || !pointer_of(a[1], &set))
        return PyObject_Vectorcall(g_slow_cached, a, n, kw);
    if (PyObject_GetBuffer(a[2], &shape, PyBUF_SIMPLE) != 0) return nullptr;
    const ft_plan *plan = nullptr;
    ft_status st;
    Py_BEGIN_ALLOW_THREADS
    st = g_cached(static_cast<const ft_op *>(op), static_cast<ft_ukset *>(set), static_cast<const ft_shape *>(shape.buf), 0u, &plan);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&shape);
    if (st != FT_OK) return checked(st, "ft_plan_cached");
    // CachedPlan(plan, a[1]) without its __init__
    PyTypeObject *type = reinterpret_cast<PyTypeObject *>(g_plan);
    PyObject *out = type->tp_new(type, g_no_args, nullptr), *ptr = out ? PyLong_FromVoidPtr(const_cast<ft_plan *>(plan)) : nullptr;
    if (!ptr || PyObject_SetAttr(out, s_ptr, ptr) != 0 || PyObject_SetAttr(out, s_owner, a[1]) != 0) Py_CLEAR(out);
    Py_XDECREF(ptr);
    return out;
}

void keep(PyObject *&to, PyObject *from) {
    Py_INCREF(from);
    Py_XSETREF(to, from);
}

// slow(check, shape type, plan type, the three ctypes functions): once, before the first call
PyObject *slow(PyObject *, PyObject *args) {
    PyObject *o[6];
    if (!PyArg_ParseTuple(args, "OOOOOO", &o[0], &o[1], &o[2], &o[3], &o[4], &o[5])) return nullptr;
    keep(g_check, o[0]); keep(g_shape, o[1]); keep(g_plan, o[2]);
    keep(g_slow_cached, o[3]); keep(g_slow_launch, o[4]); keep(g_slow_epilogue, o[5]);
    Py_RETURN_NONE;
}
// bind(addresses of ft_plan_cached, ft_launch, ft_launch_epilogue in the loaded library)
PyObject *bind(PyObject *, PyObject *args) {
    unsigned long long c, l, e;
    if (!PyArg_ParseTuple(args, "KKK", &c, &l, &e)) return nullptr;
    g_cached = reinterpret_cast<cached_fn>(c); g_launch = reinterpret_cast<launch_fn>(l); g_epilogue = reinterpret_cast<epilogue_fn>(e);
    Py_RETURN_NONE;
}

template <typename F> PyCFunction fn(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }
PyMethodDef methods[] = {
    {"slow", slow, METH_VARARGS, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {"ft_plan_cached", fn(plan_cached), METH_FASTCALL | METH_KEYWORDS,
     "ft_plan_cached(op, s, shape, flags=FT_PLAN_PATCHWORK)\n\nThe set's plan for the shape, made on the first call."},
    {"ft_launch", fn(launch), METH_FASTCALL | METH_KEYWORDS,
     "ft_launch(p, A, B, Cptr, stream=0)\n\nA, B, Cptr: device addresses (e.g. torch.Tensor.data_ptr()); stream: hipStream_t value."},
    {"ft_launch_epilogue", fn(launch_epilogue), METH_FASTCALL | METH_KEYWORDS,
     "ft_launch_epilogue(p, A, B, Cptr, bias, stream=0)\n\nAs ft_launch, with bias = device address of N fp32 values (0 / None for none)."},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycalls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycalls(void) {
    s_ptr = PyUnicode_InternFromString("ptr");
    s_owner = PyUnicode_InternFromString("_owner");
    g_no_args = PyTuple_New(0);
    if (!s_ptr || !s_owner || !g_no_args) return nullptr;
    return PyModule_Create(&module);
}
