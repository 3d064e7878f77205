// CPython entry points of the run calls a serving loop makes once per layer or stack: argument marshalling only, like the
// rest of the binding.  A call through ctypes costs about a microsecond more than this (a conversion object per argument,
// a Python frame per tensor), a fifth of what a small layer takes from call to call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/npas.h"

namespace {

PyObject *error_class; // NpasError(code, message), set by init()
PyObject *c_void_p;    // ctypes.c_void_p, set by init()
PyObject *s_handle, *s_value, *s_is_contiguous, *s_data_ptr;

// The arguments of one call, converted in their order.  Once one does not convert, the later conversions do nothing.
struct Args {
    PyObject *const *a;
    enum { PLAIN, FAILED, OTHER } state = PLAIN; // all plain so far; a Python error is set; one is of a kind that is left to ctypes

    // Device pointer: None, an address, or a contiguous tensor.
    void *pointer(int i)
    {
        PyObject *o = a[i];
        if (state != PLAIN || o == Py_None) return nullptr;
        if (PyLong_Check(o)) return number(PyLong_AsUnsignedLongLongMask(o));
        PyObject *c = PyObject_CallMethodNoArgs(o, s_is_contiguous);
        const int yes = c ? PyObject_IsTrue(c) : -1;
        Py_XDECREF(c);
        if (yes == 0) PyErr_SetString(PyExc_AssertionError, "tensor is not contiguous");
        PyObject *p = yes == 1 ? PyObject_CallMethodNoArgs(o, s_data_ptr) : nullptr;
        if (!p) return fail();
        void *v = PyLong_Check(p) ? number(PyLong_AsUnsignedLongLongMask(p)) : other();
        Py_DECREF(p);
        return v;
    }

    // Address that is not a tensor's, such as a stream: None or an integer; ctypes knows the rest (c_void_p, _as_parameter_).
    void *address(int i)
    {
        PyObject *o = a[i];
        if (state != PLAIN || o == Py_None) return nullptr;
        return PyLong_Check(o) ? number(PyLong_AsUnsignedLongLongMask(o)) : other();
    }

    // Library handle of a Packed / Stack object: its `handle` is a ctypes c_void_p, or None once released.
    void *handle(int i)
    {
        if (state != PLAIN) return nullptr;
        PyObject *h = PyObject_GetAttr(a[i], s_handle);
        if (!h) return fail();
        void *v = nullptr;
        if (PyLong_Check(h)) v = number(PyLong_AsUnsignedLongLongMask(h));
        else if (h != Py_None) {
            PyObject *p = PyObject_IsInstance(h, c_void_p) == 1 ? PyObject_GetAttr(h, s_value) : nullptr;
            if (p && PyLong_Check(p)) v = number(PyLong_AsUnsignedLongLongMask(p));
            else if (p != Py_None) v = PyErr_Occurred() ? fail() : other();
            Py_XDECREF(p);
        }
        Py_DECREF(h);
        return v;
    }

    // As ctypes: anything with __index__, an int reduced to 32 bits; no floats.
    int integer(int i) { return (int)(unsigned int)size(i); }
    size_t size(int i)
    {
        if (state != PLAIN) return 0;
        if (PyFloat_Check(a[i])) {
            PyErr_SetString(PyExc_TypeError, "int expected instead of float");
            fail();
            return 0;
        }
        if (!PyIndex_Check(a[i])) return (size_t)(uintptr_t)other();
        return (size_t)(uintptr_t)number(PyLong_AsUnsignedLongLongMask(a[i]));
    }

private:
    void *fail()
    {
        state = FAILED;
        return nullptr;
    }
    void *other()
    {
        state = OTHER;
        return nullptr;
    }
    void *number(unsigned long long v) { return v == (unsigned long long)-1 && PyErr_Occurred() ? fail() : (void *)(uintptr_t)v; }
};

PyObject *result(int rc)
{
    if (rc == NPAS_OK) Py_RETURN_NONE;
    PyObject *e = PyObject_CallFunction(error_class, "is", rc, npas_last_error());
    if (e) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// What follows the conversions: the library call without the interpreter lock, or, where an argument is of another kind, the
// same call through ctypes (which accepts or refuses it).
enum Call { CONV2D, FC, DEPTHWISE, STACK, CALLS };
PyObject *by_ctypes[CALLS]; // set by init()

template <typename F> PyObject *finish(const Args &g, Call which, Py_ssize_t n, F call)
{
    if (g.state == Args::FAILED) return nullptr;
    if (g.state == Args::OTHER) return PyObject_Vectorcall(by_ctypes[which], g.a, (size_t)n, nullptr);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return result(rc);
}

bool argc(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
    return false;
}

// conv2d_sparse(packed, x, y, N, H, W, stride, pad, bias, residual, act, stream)
PyObject *conv2d_sparse(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!argc(n, 12)) return nullptr;
    Args g{a};
    npas_packed *p = (npas_packed *)g.handle(0);
    void *x = g.pointer(1), *y = g.pointer(2);
    const int N = g.integer(3), H = g.integer(4), W = g.integer(5), stride = g.integer(6), pad = g.integer(7);
    void *b = g.pointer(8), *r = g.pointer(9);
    const int act = g.integer(10);
    void *st = g.address(11);
    return finish(g, CONV2D, n, [&] { return npas_conv2d_sparse(p, x, y, N, H, W, stride, pad, b, r, (npas_act)act, st); });
}

// fc_sparse(packed, x, y, B, bias, act, stream)
PyObject *fc_sparse(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!argc(n, 7)) return nullptr;
    Args g{a};
    npas_packed *p = (npas_packed *)g.handle(0);
    void *x = g.pointer(1), *y = g.pointer(2);
    const int B = g.integer(3);
    void *b = g.pointer(4);
    const int act = g.integer(5);
    void *st = g.address(6);
    return finish(g, FC, n, [&] { return npas_fc_sparse(p, x, y, B, b, (npas_act)act, st); });
}

// depthwise3x3(packed, x, y, N, H, W, stride, bias, residual, act, stream)
PyObject *depthwise3x3(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!argc(n, 11)) return nullptr;
    Args g{a};
    npas_packed *p = (npas_packed *)g.handle(0);
    void *x = g.pointer(1), *y = g.pointer(2);
    const int N = g.integer(3), H = g.integer(4), W = g.integer(5), stride = g.integer(6);
    void *b = g.pointer(7), *r = g.pointer(8);
    const int act = g.integer(9);
    void *st = g.address(10);
    return finish(g, DEPTHWISE, n, [&] { return npas_depthwise3x3(p, x, y, N, H, W, stride, b, r, (npas_act)act, st); });
}

// run_stack(stack, x, y, N, workspace, workspace_bytes, stream)
PyObject *run_stack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!argc(n, 7)) return nullptr;
    Args g{a};
    npas_stack *s = (npas_stack *)g.handle(0);
    void *x = g.pointer(1), *y = g.pointer(2);
    const int N = g.integer(3);
    void *w = g.pointer(4);
    const size_t bytes = g.size(5);
    void *st = g.address(6);
    return finish(g, STACK, n, [&] { return npas_run_stack(s, x, y, N, w, bytes, st); });
}

// init(NpasError, c_void_p, conv2d_sparse, fc_sparse, depthwise3x3, run_stack): the last four are the calls through ctypes
PyObject *init(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (!argc(n, 2 + CALLS)) return nullptr;
    auto keep = [](PyObject *&slot, PyObject *o) {
        Py_INCREF(o);
        Py_XSETREF(slot, o);
    };
    keep(error_class, a[0]);
    keep(c_void_p, a[1]);
    for (int i = 0; i < CALLS; ++i) keep(by_ctypes[i], a[2 + i]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", (PyCFunction)(void (*)(void))init, METH_FASTCALL, nullptr},
    {"conv2d_sparse", (PyCFunction)(void (*)(void))conv2d_sparse, METH_FASTCALL, nullptr},
    {"fc_sparse", (PyCFunction)(void (*)(void))fc_sparse, METH_FASTCALL, nullptr},
    {"depthwise3x3", (PyCFunction)(void (*)(void))depthwise3x3, METH_FASTCALL, nullptr},
    {"run_stack", (PyCFunction)(void (*)(void))run_stack, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycalls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__pycalls()
{
    s_handle = PyUnicode_InternFromString("handle");
    s_value = PyUnicode_InternFromString("value");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!s_handle || !s_value || !s_is_contiguous || !s_data_ptr) return nullptr;
    return PyModule_Create(&module);
}
