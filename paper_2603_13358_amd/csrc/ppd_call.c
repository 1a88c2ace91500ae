// Argument marshalling of the calls a serving loop makes for every layer (CPython extension module ppd_call): the same
// conversions that the ctypes binding does, for a fifth of its time.  Each function takes the address of a libppd entry
// point first, so this module links to nothing; the GIL is released around the call.
// A small step is bound by the host: ctypes cost 1.1 us of the 4.0 us of an append call and 2.2 of the 5.6 of an
// attention call whose plan is on the device.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

static PyObject *s_data_ptr, *s_value, *s_shape;
static PyObject *t_void_p, *f_cast;  // ctypes.c_void_p and ctypes.cast

// What a ctypes parameter of type c_void_p takes: None, an int and a c_void_p (a context's handle) here, anything else --
// objects with _as_parameter_ (torch.cuda.Stream is one), pointers, arrays -- by ctypes itself, which also refuses the rest
static int to_handle(PyObject* o, void** out) {
    *out = NULL;
    if (o == Py_None) return 1;
    if (PyLong_Check(o)) {
        *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
        return !PyErr_Occurred();
    }
    PyObject* p = (PyObject*)Py_TYPE(o) == t_void_p ? Py_NewRef(o) : PyObject_CallFunctionObjArgs(f_cast, o, t_void_p, NULL);
    if (!p) return 0;
    PyObject* v = PyObject_GetAttr(p, s_value);
    Py_DECREF(p);
    if (!v) return 0;
    if (v != Py_None) *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    return !PyErr_Occurred();
}
// a tensor's data_ptr(), or None or an int that already is an address
static int to_address(PyObject* o, void** out) {
    if (o == Py_None || PyLong_Check(o)) return to_handle(o, out);
    PyObject* v = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!v) return 0;
    const int ok = to_handle(v, out);
    Py_DECREF(v);
    return ok;
}
static int to_int(PyObject* o, int64_t* out) {
    PyObject* v = PyNumber_Long(o);
    if (!v) return 0;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    return !PyErr_Occurred();
}
// `o` as an int, or x.shape[dim] if it is None
static int to_int_or_shape(PyObject* o, PyObject* x, Py_ssize_t dim, int64_t* out) {
    if (o != Py_None) return to_int(o, out);
    PyObject* shape = PyObject_GetAttr(x, s_shape);
    if (!shape) return 0;
    PyObject* v = PySequence_GetItem(shape, dim);
    Py_DECREF(shape);
    if (!v) return 0;
    const int ok = to_int(v, out);
    Py_DECREF(v);
    return ok;
}
static int expect(Py_ssize_t have, Py_ssize_t want) {
    if (have == want) return 1;
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return 0;
}

typedef int32_t (*append_fn)(void*, const void*, const void*, void*, const int64_t*, int64_t, void*);
typedef int32_t (*land_fn)(void*, const void*, const void*, void*, int64_t, int32_t, const int64_t*, int64_t, void*);
typedef int32_t (*mixed_fn)(void*, const void*, const void*, const int32_t*, int32_t, const int32_t*, const int32_t*, int32_t, float, void*, void*);

// kv_append(fn, ctx, k, v, kv_pages, slot_mapping, T, stream) -> status
static PyObject* call_append(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    void *fn, *ctx, *k, *v, *pages, *slots, *stream;
    int64_t T;
    (void)self;
    if (!expect(n, 8) || !to_handle(a[0], &fn) || !to_handle(a[1], &ctx) || !to_int_or_shape(a[6], a[5], 0, &T) ||
        !to_address(a[2], &k) || !to_address(a[3], &v) || !to_address(a[4], &pages) ||
        !to_address(a[5], &slots) || !to_handle(a[7], &stream))
        return NULL;
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = ((append_fn)fn)(ctx, k, v, pages, (const int64_t*)slots, T, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// kv_land(fn, ctx, k, v, kv_pages, layer_stride_elems, num_layers, slot_mapping, T, stream) -> status
static PyObject* call_land(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    void *fn, *ctx, *k, *v, *pages, *slots, *stream;
    int64_t stride, layers, T;
    (void)self;
    if (!expect(n, 10) || !to_handle(a[0], &fn) || !to_handle(a[1], &ctx) || !to_int_or_shape(a[8], a[7], 0, &T) ||
        !to_address(a[2], &k) || !to_address(a[3], &v) || !to_address(a[4], &pages) ||
        !to_int(a[5], &stride) || !to_int(a[6], &layers) || !to_address(a[7], &slots) || !to_handle(a[9], &stream))
        return NULL;
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = ((land_fn)fn)(ctx, k, v, pages, stride, (int32_t)layers, (const int64_t*)slots, T, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// A one-dimensional contiguous array of native 32-bit integers: 1 and a filled buffer; anything else: 0, no error
static int int32_array(PyObject* o, Py_buffer* b) {
    if (!PyObject_CheckBuffer(o)) return 0;
    if (PyObject_GetBuffer(o, b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
        PyErr_Clear();
        return 0;
    }
    if (b->ndim == 1 && b->itemsize == 4 && b->format && b->format[0] == 'i' && b->format[1] == 0) return 1;
    PyBuffer_Release(b);
    return 0;
}

// mixed_attention(fn, ctx, q, kv_pages, page_tables, max_pages, L, n, scale, out, stream) -> status, or None if L and n are not
// plain int32 arrays yet
static PyObject* call_mixed(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    void *fn, *ctx, *q, *pages, *tables, *out, *stream;
    int64_t max_pages;
    Py_buffer L, nn;
    (void)self;
    if (!expect(n, 11)) return NULL;
    if (!int32_array(a[6], &L)) Py_RETURN_NONE;
    if (!int32_array(a[7], &nn)) {
        PyBuffer_Release(&L);
        Py_RETURN_NONE;
    }
    PyObject* result = NULL;
    PyObject* scale = NULL;
    if (to_handle(a[0], &fn) && to_handle(a[1], &ctx) && to_int_or_shape(a[5], a[4], 1, &max_pages) &&
        to_address(a[2], &q) && to_address(a[3], &pages) && to_address(a[4], &tables) &&
        (scale = PyNumber_Float(a[8])) && to_address(a[9], &out) && to_handle(a[10], &stream)) {
        const float s = (float)PyFloat_AS_DOUBLE(scale);
        int32_t status;
        Py_BEGIN_ALLOW_THREADS
        status = ((mixed_fn)fn)(ctx, q, pages, (const int32_t*)tables, (int32_t)max_pages, (const int32_t*)L.buf, (const int32_t*)nn.buf,
                                (int32_t)L.shape[0], s, out, stream);
        Py_END_ALLOW_THREADS
        result = PyLong_FromLong(status);
    }
    Py_XDECREF(scale);
    PyBuffer_Release(&nn);
    PyBuffer_Release(&L);
    return result;
}

static PyMethodDef kMethods[] = {
    {"kv_append", (PyCFunction)(void (*)(void))call_append, METH_FASTCALL, NULL},
    {"kv_land", (PyCFunction)(void (*)(void))call_land, METH_FASTCALL, NULL},
    {"mixed_attention", (PyCFunction)(void (*)(void))call_mixed, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "ppd_call", "Calls of libppd's per-layer entry points.", -1, kMethods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit_ppd_call(void) {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_value = PyUnicode_InternFromString("value");
    s_shape = PyUnicode_InternFromString("shape");
    PyObject* ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes) return NULL;
    t_void_p = PyObject_GetAttrString(ctypes, "c_void_p");
    f_cast = PyObject_GetAttrString(ctypes, "cast");
    Py_DECREF(ctypes);
    if (!s_data_ptr || !s_value || !s_shape || !t_void_p || !f_cast) return NULL;
    return PyModule_Create(&kModule);
}
