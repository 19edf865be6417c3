// The binding's call of fbq_linear for one layer whose result and workspace the caller keeps: collects the pointers of the tensors and calls the
// library, without the argument objects that ctypes builds (one token through 4096 x 4096: the call took longer than its kernel, 6.1 us; 5.0 this way).
// It knows nothing of torch: it asks the objects what the binding's Python code asks (is_cuda, is_contiguous(), data_ptr(), numel(),
// element_size()).  Whatever is not as it should be makes it return None, and the Python code does the call, or raises;
// exceptions that are no `Exception` pass through.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "fbq.h"

typedef fbq_status (*linear_fn)(const fbq_desc *, int, const void *, const void *, const void *, const void *, const void *, const void *, void *, void *,
                                size_t, fbq_stream);

static PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_numel, *s_element_size, *s_desc, *s_N, *s_K, *s_r, *s_bits, *s_group, *s_shape;
static PyObject *s_tensor[5];                           // qweight, scales, zeros, At, Bt

// An attribute or a method's result as a whole number; 0 where it is none.
static int number(PyObject *v, unsigned long long *out)
{
    const int ok = v && PyLong_CheckExact(v);
    if (ok) *out = PyLong_AsUnsignedLongLongMask(v);
    Py_XDECREF(v);
    return ok;
}

static int is_true(PyObject *v)
{
    const int yes = v == Py_True;
    Py_XDECREF(v);
    return yes;
}

static int pointer(PyObject *t, unsigned long long *out)
{
    *out = 0;
    if (t == Py_None) return 1;
    return is_true(PyObject_GetAttr(t, s_is_cuda)) && is_true(PyObject_CallMethodNoArgs(t, s_is_contiguous)) && number(PyObject_CallMethodNoArgs(t, s_data_ptr), out);
}

// linear(address of fbq_linear, layer, x, y, workspace, stream) -> status, or None
static PyObject *linear(PyObject *self, PyObject *const *arg, Py_ssize_t n)
{
    (void)self;
    if (n != 6) {
        PyErr_SetString(PyExc_TypeError, "six arguments");
        return NULL;
    }
    unsigned long long fn, p[8] = {0}, field[5], M = 0, count = 0, each = 0, stream;
    PyObject *const names[5] = {s_N, s_K, s_r, s_bits, s_group};
    PyObject *desc = NULL, *shape = NULL, *first = NULL;
    int ok = PyLong_CheckExact(arg[0]) && PyLong_CheckExact(arg[5]);
    fn = ok ? PyLong_AsUnsignedLongLongMask(arg[0]) : 0;
    stream = ok ? PyLong_AsUnsignedLongLongMask(arg[5]) : 0;
    ok = ok && fn && (desc = PyObject_GetAttr(arg[1], s_desc));
    for (int i = 0; ok && i < 5; ++i) ok = number(PyObject_GetAttr(desc, names[i]), &field[i]) && field[i] <= INT32_MAX;
    Py_XDECREF(desc);
    ok = ok && (shape = PyObject_GetAttr(arg[2], s_shape)) && (first = PySequence_GetItem(shape, 0)) && PyLong_CheckExact(first);
    if (ok) M = PyLong_AsUnsignedLongLongMask(first);
    Py_XDECREF(first);
    Py_XDECREF(shape);
    ok = ok && M <= INT32_MAX && pointer(arg[2], &p[0]);
    for (int i = 0; ok && i < 5; ++i) {
        PyObject *t = PyObject_GetAttr(arg[1], s_tensor[i]);
        ok = t && pointer(t, &p[1 + i]);
        Py_XDECREF(t);
    }
    ok = ok && pointer(arg[3], &p[6]) && pointer(arg[4], &p[7]);
    if (ok && arg[4] != Py_None) ok = number(PyObject_CallMethodNoArgs(arg[4], s_numel), &count) && number(PyObject_CallMethodNoArgs(arg[4], s_element_size), &each);
    if (!ok) {
        if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) return NULL;   // (an interrupt, say: not this call's to drop)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const fbq_desc d = {(int32_t)field[0], (int32_t)field[1], (int32_t)field[2], (int32_t)field[3], (int32_t)field[4]};
    fbq_status st;
    Py_BEGIN_ALLOW_THREADS                              // (as ctypes does)
    st = ((linear_fn)(uintptr_t)fn)(&d, (int)M, (const void *)(uintptr_t)p[0], (const void *)(uintptr_t)p[1], (const void *)(uintptr_t)p[2],
                                    (const void *)(uintptr_t)p[3], (const void *)(uintptr_t)p[4], (const void *)(uintptr_t)p[5],
                                    (void *)(uintptr_t)p[6], (void *)(uintptr_t)p[7], (size_t)(count * each), (fbq_stream)(uintptr_t)stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

static PyMethodDef methods[] = {{"linear", (PyCFunction)(void (*)(void))linear, METH_FASTCALL, "fbq_linear of one layer; None: not as expected, nothing done"},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fbq_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fbq_call(void)
{
    static const char *const tensors[5] = {"qweight", "scales", "zeros", "At", "Bt"};
    struct { PyObject **to; const char *name; } all[] = {
        {&s_is_cuda, "is_cuda"}, {&s_is_contiguous, "is_contiguous"}, {&s_data_ptr, "data_ptr"}, {&s_numel, "numel"}, {&s_element_size, "element_size"},
        {&s_desc, "desc"}, {&s_N, "N"}, {&s_K, "K"}, {&s_r, "r"}, {&s_bits, "bits"}, {&s_group, "group"}, {&s_shape, "shape"}};
    for (size_t i = 0; i < sizeof(all) / sizeof(all[0]); ++i)
        if (!(*all[i].to = PyUnicode_InternFromString(all[i].name))) return NULL;
    for (int i = 0; i < 5; ++i)
        if (!(s_tensor[i] = PyUnicode_InternFromString(tensors[i]))) return NULL;
    return PyModule_Create(&module);
}
