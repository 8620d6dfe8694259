/* CPython extension behind binding.py: turns the arguments of the hot entry points into C values and calls the library.
 * The library's symbols are not linked: binding.py loads libngconv.so and hands each function's address over once.
 *
 * A call of a small node is bound by the host.  ctypes took 1.1 us of the 4.9 us of such a call (a c_void_p object per
 * pointer, a conversion per argument); here an argument costs a type test and, for a tensor, one data_ptr() call. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/ngconv.h"

static PyObject *s_data_ptr, *s_numel, *s_element_size;
static PyObject *t_desc[2];      /* the descriptor classes: two spatial axes, three */

/* None -> NULL, int -> that address, anything else -> its data_ptr().  -1 with an exception set on failure. */
static int as_ptr(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = NULL;
        return 0;
    }
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
    } else {
        PyObject *r = PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (!r) return -1;
        *out = PyLong_AsVoidPtr(r);
        Py_DECREF(r);
    }
    return PyErr_Occurred() ? -1 : 0;
}

/* bytes of a workspace tensor; 0 for None and for a raw address */
static int as_bytes(PyObject *o, size_t *out)
{
    *out = 0;
    if (o == Py_None || PyLong_Check(o)) return 0;
    PyObject *n = PyObject_CallMethodNoArgs(o, s_numel), *e = n ? PyObject_CallMethodNoArgs(o, s_element_size) : NULL;
    if (e) *out = PyLong_AsSize_t(n) * PyLong_AsSize_t(e);
    Py_XDECREF(n);
    Py_XDECREF(e);
    return PyErr_Occurred() ? -1 : 0;
}

/* a stream: None or an address; a false value is the default stream.  What is no address (a stream object) is refused. */
static int as_stream(PyObject *o, void **out)
{
    const int set = o == Py_None ? 0 : PyObject_IsTrue(o);
    *out = NULL;
    if (set <= 0) return set;
    if (!PyLong_Check(o)) {
        PyErr_Format(PyExc_TypeError, "stream: None or its address expected, not %.100s", Py_TYPE(o)->tp_name);
        return -1;
    }
    *out = PyLong_AsVoidPtr(o);
    return PyErr_Occurred() ? -1 : 0;
}

/* the descriptor: an instance of the ctypes structure, whose first `size` bytes are copied */
static int as_desc(PyObject *o, PyObject *type, void *out, Py_ssize_t size)
{
    Py_buffer b;
    const int is = type ? PyObject_IsInstance(o, type) : 0;
    if (is < 0) return -1;
    if (!is) {
        PyErr_Format(PyExc_TypeError, "descriptor of another type expected, not %.100s", Py_TYPE(o)->tp_name);
        return -1;
    }
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return -1;
    const int ok = b.len >= size;
    if (ok) memcpy(out, b.buf, (size_t)size);
    else PyErr_SetString(PyExc_TypeError, "descriptor of another size expected");
    PyBuffer_Release(&b);
    return ok ? 0 : -1;
}

static int as_int(PyObject *o, long long *out)
{
    *out = PyLong_AsLongLong(o);
    return *out == -1 && PyErr_Occurred() ? -1 : 0;
}

#define MAX_PTR 7
typedef struct {
    ngc_conv_desc d;
    ngc_conv3d_desc d3;
    void *p[MAX_PTR];
    size_t ws_bytes;
} Args;

/* args: descriptor, np pointers of which the last but one is the workspace (ws) and the last the stream */
static int parse(PyObject *const *a, Py_ssize_t n, int rank3, int np, int ws, Args *out)
{
    if (n != np + 1) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return -1;
    }
    if (rank3 ? as_desc(a[0], t_desc[1], &out->d3, sizeof(out->d3)) : as_desc(a[0], t_desc[0], &out->d, sizeof(out->d))) return -1;
    for (int i = 0; i < np; ++i)
        if (i == np - 1 ? as_stream(a[1 + i], &out->p[i]) : as_ptr(a[1 + i], &out->p[i])) return -1;
    return ws ? as_bytes(a[np - 1], &out->ws_bytes) : 0;
}

/* one wrapper per entry point: NAME is the C function, NP its pointer arguments (workspace and stream among them) */
#define ENTRY(NAME, RANK3, NP, WS, CALL)                                                    \
    static __typeof__(NAME) *f_##NAME;                                                      \
    static PyObject *w_##NAME(PyObject *self, PyObject *const *a, Py_ssize_t n)             \
    {                                                                                       \
        Args x;                                                                             \
        (void)self;                                                                         \
        if (parse(a, n, RANK3, NP, WS, &x)) return NULL;                                    \
        int rc;                                                                             \
        Py_BEGIN_ALLOW_THREADS                                                              \
        rc = f_##NAME CALL;                                                                 \
        Py_END_ALLOW_THREADS                                                                \
        return PyLong_FromLong(rc);                                                         \
    }

ENTRY(ngc_conv_fwd, 0, 6, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.ws_bytes, x.p[5]))
ENTRY(ngc_conv_bwd_data, 0, 5, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3], x.ws_bytes, x.p[4]))
ENTRY(ngc_conv_bwd_data_relu, 0, 6, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.ws_bytes, x.p[5]))
ENTRY(ngc_conv_bwd_data_relu_db, 0, 7, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.p[5], x.ws_bytes, x.p[6]))
ENTRY(ngc_bias_grad, 0, 4, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.ws_bytes, x.p[3]))
ENTRY(ngc_conv_bwd_filters, 0, 5, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3], x.ws_bytes, x.p[4]))
ENTRY(ngc_conv_bwd_filters_noalloc, 0, 4, 0, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3]))
ENTRY(ngc_conv_bwd_data_filters, 0, 7, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.p[5], x.ws_bytes, x.p[6]))
ENTRY(ngc_conv_bwd_data_filters_relu, 0, 7, 1, (&x.d, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.p[5], x.ws_bytes, x.p[6]))
ENTRY(ngc_conv3d_fwd, 1, 6, 1, (&x.d3, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.ws_bytes, x.p[5]))
ENTRY(ngc_conv3d_bwd_data, 1, 5, 1, (&x.d3, x.p[0], x.p[1], x.p[2], x.p[3], x.ws_bytes, x.p[4]))
ENTRY(ngc_conv3d_bwd_data_relu, 1, 6, 1, (&x.d3, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.ws_bytes, x.p[5]))
ENTRY(ngc_conv3d_bwd_data_relu_db, 1, 7, 1, (&x.d3, x.p[0], x.p[1], x.p[2], x.p[3], x.p[4], x.p[5], x.ws_bytes, x.p[6]))
ENTRY(ngc_conv3d_bias_grad, 1, 4, 1, (&x.d3, x.p[0], x.p[1], x.p[2], x.ws_bytes, x.p[3]))
ENTRY(ngc_conv3d_bwd_filters, 1, 5, 1, (&x.d3, x.p[0], x.p[1], x.p[2], x.p[3], x.ws_bytes, x.p[4]))

/* entry points whose leading arguments are integers: KINDS holds 'i' (integer), 'p' (pointer) or 's' (stream) per argument */
static int parse_kinds(PyObject *const *a, Py_ssize_t n, const char *kinds, long long *i, void **p)
{
    if (n != (Py_ssize_t)strlen(kinds)) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return -1;
    }
    for (Py_ssize_t k = 0; k < n; ++k)
        if (kinds[k] == 'i' ? as_int(a[k], i++) : kinds[k] == 's' ? as_stream(a[k], p++) : as_ptr(a[k], p++)) return -1;
    return 0;
}

#define ENTRY_KINDS(NAME, KINDS, CALL)                                                      \
    static __typeof__(NAME) *f_##NAME;                                                      \
    static PyObject *w_##NAME(PyObject *self, PyObject *const *a, Py_ssize_t n)             \
    {                                                                                       \
        long long i[8];                                                                     \
        void *p[8];                                                                         \
        (void)self;                                                                         \
        if (parse_kinds(a, n, KINDS, i, p)) return NULL;                                    \
        int rc;                                                                             \
        Py_BEGIN_ALLOW_THREADS                                                              \
        rc = f_##NAME CALL;                                                                 \
        Py_END_ALLOW_THREADS                                                                \
        return PyLong_FromLong(rc);                                                         \
    }

ENTRY_KINDS(ngc_softmax, "iiipps", ((int32_t)i[0], i[1], (int32_t)i[2], p[0], p[1], p[2]))
ENTRY_KINDS(ngc_softmax_bwd, "iiippps", ((int32_t)i[0], i[1], (int32_t)i[2], p[0], p[1], p[2], p[3]))
ENTRY_KINDS(ngc_layout_convert, "iiiiipipis",
            ((int32_t)i[0], (int32_t)i[1], (int32_t)i[2], (int32_t)i[3], (int32_t)i[4], p[0], (int32_t)i[5], p[1], (int32_t)i[6], p[2]))

static const struct {
    const char *name;
    void **slot;
} slots[] = {
#define SLOT(NAME) {#NAME, (void **)&f_##NAME}
    SLOT(ngc_conv_fwd), SLOT(ngc_conv_bwd_data), SLOT(ngc_conv_bwd_data_relu), SLOT(ngc_conv_bwd_data_relu_db), SLOT(ngc_bias_grad),
    SLOT(ngc_conv_bwd_filters), SLOT(ngc_conv_bwd_filters_noalloc), SLOT(ngc_conv_bwd_data_filters), SLOT(ngc_conv_bwd_data_filters_relu),
    SLOT(ngc_conv3d_fwd), SLOT(ngc_conv3d_bwd_data), SLOT(ngc_conv3d_bwd_data_relu), SLOT(ngc_conv3d_bwd_data_relu_db),
    SLOT(ngc_conv3d_bias_grad), SLOT(ngc_conv3d_bwd_filters), SLOT(ngc_softmax), SLOT(ngc_softmax_bwd), SLOT(ngc_layout_convert),
#undef SLOT
};

static PyObject *names(PyObject *self, PyObject *arg)
{
    (void)self; (void)arg;
    const Py_ssize_t n = (Py_ssize_t)(sizeof(slots) / sizeof(slots[0]));
    PyObject *t = PyTuple_New(n);
    for (Py_ssize_t i = 0; t && i < n; ++i) PyTuple_SET_ITEM(t, i, PyUnicode_FromString(slots[i].name));
    return t;
}

/* bind(name, address): where the library's function of that name is */
static PyObject *bind(PyObject *self, PyObject *args)
{
    const char *name;
    PyObject *addr;
    (void)self;
    if (!PyArg_ParseTuple(args, "sO", &name, &addr)) return NULL;
    for (size_t i = 0; i < sizeof(slots) / sizeof(slots[0]); ++i)
        if (strcmp(slots[i].name, name) == 0) {
            *slots[i].slot = PyLong_AsVoidPtr(addr);
            if (PyErr_Occurred()) return NULL;
            Py_RETURN_NONE;
        }
    PyErr_SetString(PyExc_KeyError, name);
    return NULL;
}

/* descs(class, class3): the descriptor classes the entry points take */
static PyObject *descs(PyObject *self, PyObject *args)
{
    PyObject *d, *d3;
    (void)self;
    if (!PyArg_ParseTuple(args, "O!O!", &PyType_Type, &d, &PyType_Type, &d3)) return NULL;
    Py_INCREF(d);
    Py_INCREF(d3);
    Py_XSETREF(t_desc[0], d);
    Py_XSETREF(t_desc[1], d3);
    Py_RETURN_NONE;
}

#define METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))w_##NAME, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {
    {"names", names, METH_NOARGS, NULL},
    {"bind", bind, METH_VARARGS, NULL},
    {"descs", descs, METH_VARARGS, NULL},
    METHOD(ngc_conv_fwd), METHOD(ngc_conv_bwd_data), METHOD(ngc_conv_bwd_data_relu), METHOD(ngc_conv_bwd_data_relu_db), METHOD(ngc_bias_grad),
    METHOD(ngc_conv_bwd_filters), METHOD(ngc_conv_bwd_filters_noalloc), METHOD(ngc_conv_bwd_data_filters), METHOD(ngc_conv_bwd_data_filters_relu),
    METHOD(ngc_conv3d_fwd), METHOD(ngc_conv3d_bwd_data), METHOD(ngc_conv3d_bwd_data_relu), METHOD(ngc_conv3d_bwd_data_relu_db),
    METHOD(ngc_conv3d_bias_grad), METHOD(ngc_conv3d_bwd_filters), METHOD(ngc_softmax), METHOD(ngc_softmax_bwd), METHOD(ngc_layout_convert),
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__pycall(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    return PyModule_Create(&module);
}
