// CPython entry points of the run calls a serving loop makes once per layer or stack: argument marshalling only, like the
// rest of the binding.  A call through ctypes costs about a microsecond more than this (a conversion object per argument,
// a Python frame per tensor), a fifth of what a small layer takes from call to call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/npas.h"

namespace {

PyObject *error_class; // NpasError(code, message), set by init()
PyObject *s_handle, *s_value, *s_is_contiguous, *s_data_ptr;

// Device pointer of an argument: None, an address, or a contiguous tensor.
bool device_pointer(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    if (PyLong_Check(o)) {
        *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
        return !PyErr_Occurred();
    }
    PyObject *c = PyObject_CallMethodNoArgs(o, s_is_contiguous);
    if (!c) return false;
    const int yes = PyObject_IsTrue(c);
    Py_DECREF(c);
    if (yes < 0) return false;
    if (!yes) {
        PyErr_SetString(PyExc_AssertionError, "tensor is not contiguous");
        return false;
    }
    PyObject *p = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!p) return false;
    *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    return !PyErr_Occurred();
}

// Library handle of a Packed / Stack object: its `handle` is a ctypes c_void_p, or None once released.
bool library_handle(PyObject *o, void **out)
{
    PyObject *h = PyObject_GetAttr(o, s_handle);
    if (!h) return false;
    *out = nullptr;
    bool ok = true;
    if (h != Py_None) {
        PyObject *v = PyLong_Check(h) ? (Py_INCREF(h), h) : PyObject_GetAttr(h, s_value);
        ok = v != nullptr;
        if (ok && v != Py_None) {
            *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(v);
            ok = !PyErr_Occurred();
        }
        Py_XDECREF(v);
    }
    Py_DECREF(h);
    return ok;
}

bool c_int(PyObject *o, int *out) // (as ctypes: integers, reduced to 32 bits; no floats)
{
    if (PyFloat_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "int expected instead of float");
        return false;
    }
    *out = (int)(unsigned int)PyLong_AsUnsignedLongMask(o);
    return !PyErr_Occurred();
}

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

bool argc(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
    return false;
}

// conv2d_sparse(packed, x, y, N, H, W, stride, pad, bias, residual, act, stream)
PyObject *conv2d_sparse(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p, *x, *y, *b, *r, *st;
    int v[5], act, rc;
    if (!argc(n, 12) || !library_handle(a[0], &p) || !device_pointer(a[1], &x) || !device_pointer(a[2], &y)) return nullptr;
    for (int i = 0; i < 5; ++i)
        if (!c_int(a[3 + i], &v[i])) return nullptr;
    if (!device_pointer(a[8], &b) || !device_pointer(a[9], &r) || !c_int(a[10], &act) || !device_pointer(a[11], &st)) return nullptr;
    Py_BEGIN_ALLOW_THREADS
    rc = npas_conv2d_sparse((npas_packed *)p, x, y, v[0], v[1], v[2], v[3], v[4], b, r, (npas_act)act, st);
    Py_END_ALLOW_THREADS
    return result(rc);
}

// fc_sparse(packed, x, y, B, bias, act, stream)
PyObject *fc_sparse(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p, *x, *y, *b, *st;
    int B, act, rc;
    if (!argc(n, 7) || !library_handle(a[0], &p) || !device_pointer(a[1], &x) || !device_pointer(a[2], &y) || !c_int(a[3], &B) ||
        !device_pointer(a[4], &b) || !c_int(a[5], &act) || !device_pointer(a[6], &st))
        return nullptr;
    Py_BEGIN_ALLOW_THREADS
    rc = npas_fc_sparse((npas_packed *)p, x, y, B, b, (npas_act)act, st);
    Py_END_ALLOW_THREADS
    return result(rc);
}

// depthwise3x3(packed, x, y, N, H, W, stride, bias, residual, act, stream)
PyObject *depthwise3x3(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p, *x, *y, *b, *r, *st;
    int v[4], act, rc;
    if (!argc(n, 11) || !library_handle(a[0], &p) || !device_pointer(a[1], &x) || !device_pointer(a[2], &y)) return nullptr;
    for (int i = 0; i < 4; ++i)
        if (!c_int(a[3 + i], &v[i])) return nullptr;
    if (!device_pointer(a[7], &b) || !device_pointer(a[8], &r) || !c_int(a[9], &act) || !device_pointer(a[10], &st)) return nullptr;
    Py_BEGIN_ALLOW_THREADS
    rc = npas_depthwise3x3((npas_packed *)p, x, y, v[0], v[1], v[2], v[3], b, r, (npas_act)act, st);
    Py_END_ALLOW_THREADS
    return result(rc);
}

// run_stack(stack, x, y, N, workspace, workspace_bytes, stream)
PyObject *run_stack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *s, *x, *y, *w, *st;
    int N, rc;
    if (!argc(n, 7) || !library_handle(a[0], &s) || !device_pointer(a[1], &x) || !device_pointer(a[2], &y) || !c_int(a[3], &N) ||
        !device_pointer(a[4], &w))
        return nullptr;
    if (PyFloat_Check(a[5])) {
        PyErr_SetString(PyExc_TypeError, "int expected instead of float");
        return nullptr;
    }
    const size_t bytes = (size_t)PyLong_AsUnsignedLongLongMask(a[5]);
    if (PyErr_Occurred() || !device_pointer(a[6], &st)) return nullptr;
    Py_BEGIN_ALLOW_THREADS
    rc = npas_run_stack((npas_stack *)s, x, y, N, w, bytes, st);
    Py_END_ALLOW_THREADS
    return result(rc);
}

PyObject *init(PyObject *, PyObject *cls)
{
    Py_INCREF(cls);
    Py_XDECREF(error_class);
    error_class = cls;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", init, METH_O, nullptr},
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
