// The hot calls of the binding without ctypes: a small call's launch takes the host 2.6 us, and what ctypes and the Python
// around it took to bring its arguments there nearly as long again.
// Each function takes the arguments in the forms that a hot loop passes -- Python ints, a float, ctypes arrays of addresses, tensors, no
// stream -- and returns the library's status; for anything else it returns None and has done nothing, and the caller takes the ctypes route, which
// converts or refuses as it always did.
// (A pass of four calls on 135 000 elements each, 22.3 us with ctypes, 19.6 so; of two calls over eight groups, 22.1 and 19.0; 161 single calls
// 1610 and 1536.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

namespace {

typedef int (*compress_fn)(void *, int32_t, uint32_t, uint64_t, const void *, void *, void *, void *);
typedef int (*decompress_fn)(void *, int32_t, const void *, int32_t, float, const void *, void *);
typedef int (*compress_all_fn)(void *, uint32_t, uint64_t, const void *, const void *, const void *, void *);
typedef int (*decompress_all_fn)(void *, const void *, int32_t, float, const void *, void *);

PyObject *g_data_ptr;                 // the name

// The entry points of one loaded library.
struct Calls {
    PyObject_HEAD
    PyTypeObject *array;              // ctypes.Array
    compress_fn compress, compress_static;
    decompress_fn decompress;
    compress_all_fn compress_all;
    decompress_all_fn decompress_all;
};
// torch's current stream on the current device, as a callable without arguments
struct RawStream {
    PyObject_HEAD
    PyObject *get, *device;
};
extern PyTypeObject RawStreamType;

// An argument that is not in the form expected ends in `other`: None, with no error left behind.
PyObject *other()
{
    PyErr_Clear();
    Py_RETURN_NONE;
}
bool whole(PyObject *o, uint64_t *v)          // as ctypes takes integers: any value, its low bits
{
    if (!PyLong_Check(o)) return false;
    *v = PyLong_AsUnsignedLongLongMask(o);
    return !(*v == (uint64_t)-1 && PyErr_Occurred());
}
bool address(PyObject *o, void **p)
{
    if (!PyLong_Check(o)) return false;
    *p = reinterpret_cast<void *>((uintptr_t)PyLong_AsUnsignedLongLongMask(o));
    return !PyErr_Occurred();
}
// where a ctypes array's elements lie, and how many there are
bool array(const Calls *c, PyObject *o, void **p, Py_ssize_t *n)
{
    if (!PyObject_TypeCheck(o, c->array)) return false;
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) < 0) return false;
    *p = b.buf;
    PyBuffer_Release(&b);                     // (the array lives as long as the caller's argument)
    if (n && (*n = PyObject_Size(o)) < 0) return false;
    return true;
}
bool tensor(PyObject *o, void **p)
{
    PyObject *a = PyObject_CallMethodNoArgs(o, g_data_ptr);
    if (!a) return false;
    const bool ok = address(a, p);
    Py_DECREF(a);
    return ok;
}
PyObject *raw_stream_call(PyObject *self, PyObject *, PyObject *)
{
    RawStream *r = reinterpret_cast<RawStream *>(self);
    PyObject *d = PyObject_CallNoArgs(r->device);
    if (!d) return nullptr;
    PyObject *s = PyObject_CallOneArg(r->get, d);
    Py_DECREF(d);
    return s;
}
// what the callable says, if there is one
bool stream_of(PyObject *callable, void **p)
{
    if (callable == Py_None) return false;
    PyObject *s = Py_TYPE(callable) == &RawStreamType ? raw_stream_call(callable, nullptr, nullptr) : PyObject_CallNoArgs(callable);
    if (!s) return false;
    const bool ok = address(s, p);
    Py_DECREF(s);
    return ok;
}

// (context, group, worker, iteration, gradients, state or None, payload, the stream's callable)
PyObject *compress_by(const Calls *c, compress_fn fn, PyObject *const *a, Py_ssize_t n)
{
    void *ctx, *grads, *state = nullptr, *payload, *stream;
    uint64_t group, worker, iter;
    if (n != 8 || !address(a[0], &ctx) || !whole(a[1], &group) || !whole(a[2], &worker) || !whole(a[3], &iter) || !array(c, a[4], &grads, nullptr) ||
        (a[5] != Py_None && !tensor(a[5], &state)) || !tensor(a[6], &payload) || !stream_of(a[7], &stream)) return other();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(ctx, (int32_t)group, (uint32_t)worker, iter, grads, state, payload, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}
const Calls *of(PyObject *self) { return reinterpret_cast<const Calls *>(self); }
PyObject *compress(PyObject *self, PyObject *const *a, Py_ssize_t n) { return compress_by(of(self), of(self)->compress, a, n); }
PyObject *compress_static(PyObject *self, PyObject *const *a, Py_ssize_t n) { return compress_by(of(self), of(self)->compress_static, a, n); }

// (context, group, payloads, alpha, outputs, the stream's callable)
PyObject *decompress(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const Calls *c = of(self);
    void *ctx, *payloads, *outs, *stream;
    uint64_t group;
    Py_ssize_t W;
    if (n != 6 || !address(a[0], &ctx) || !whole(a[1], &group) || !array(c, a[2], &payloads, &W) || !PyFloat_CheckExact(a[3]) ||
        !array(c, a[4], &outs, nullptr) || !stream_of(a[5], &stream)) return other();
    const float alpha = (float)PyFloat_AS_DOUBLE(a[3]);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = c->decompress(ctx, (int32_t)group, payloads, (int32_t)W, alpha, outs, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// (context, worker, iteration, gradients, states or None, payloads, the stream's callable)
PyObject *compress_groups(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const Calls *c = of(self);
    void *ctx, *grads, *states = nullptr, *payloads, *stream;
    uint64_t worker, iter;
    if (n != 7 || !address(a[0], &ctx) || !whole(a[1], &worker) || !whole(a[2], &iter) || !array(c, a[3], &grads, nullptr) ||
        (a[4] != Py_None && !array(c, a[4], &states, nullptr)) || !array(c, a[5], &payloads, nullptr) || !stream_of(a[6], &stream)) return other();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = c->compress_all(ctx, (uint32_t)worker, iter, grads, states, payloads, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// (context, payloads, workers, alpha, outputs, the stream's callable)
PyObject *decompress_groups(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    const Calls *c = of(self);
    void *ctx, *payloads, *outs, *stream;
    uint64_t W;
    if (n != 6 || !address(a[0], &ctx) || !array(c, a[1], &payloads, nullptr) || !whole(a[2], &W) || !PyFloat_CheckExact(a[3]) ||
        !array(c, a[4], &outs, nullptr) || !stream_of(a[5], &stream)) return other();
    const float alpha = (float)PyFloat_AS_DOUBLE(a[3]);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = c->decompress_all(ctx, payloads, (int32_t)W, alpha, outs, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// Calls(ctypes.Array, addresses of mc_compress, mc_compress_static, mc_decompress_sum, mc_compress_groups, mc_decompress_sum_groups)
PyObject *calls_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    PyObject *array = nullptr;
    unsigned long long at[5] = {};
    if (!PyArg_ParseTuple(args, "O!KKKKK", &PyType_Type, &array, &at[0], &at[1], &at[2], &at[3], &at[4])) return nullptr;
    Calls *c = reinterpret_cast<Calls *>(type->tp_alloc(type, 0));
    if (!c) return nullptr;
    Py_INCREF(array);
    c->array = reinterpret_cast<PyTypeObject *>(array);
    c->compress = (compress_fn)(uintptr_t)at[0];
    c->compress_static = (compress_fn)(uintptr_t)at[1];
    c->decompress = (decompress_fn)(uintptr_t)at[2];
    c->compress_all = (compress_all_fn)(uintptr_t)at[3];
    c->decompress_all = (decompress_all_fn)(uintptr_t)at[4];
    return reinterpret_cast<PyObject *>(c);
}
void calls_gone(PyObject *self)
{
    Py_XDECREF(reinterpret_cast<PyObject *>(reinterpret_cast<Calls *>(self)->array));
    Py_TYPE(self)->tp_free(self);
}
// RawStream(stream of a device, current device): both callable
PyObject *raw_stream_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    PyObject *get, *device;
    if (!PyArg_ParseTuple(args, "OO", &get, &device)) return nullptr;
    RawStream *r = reinterpret_cast<RawStream *>(type->tp_alloc(type, 0));
    if (!r) return nullptr;
    Py_INCREF(get);
    Py_INCREF(device);
    r->get = get;
    r->device = device;
    return reinterpret_cast<PyObject *>(r);
}
void raw_stream_gone(PyObject *self)
{
    RawStream *r = reinterpret_cast<RawStream *>(self);
    Py_XDECREF(r->get);
    Py_XDECREF(r->device);
    Py_TYPE(self)->tp_free(self);
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef calls_methods[] = {FAST(compress), FAST(compress_static), FAST(decompress), FAST(compress_groups), FAST(decompress_groups), {nullptr, nullptr, 0, nullptr}};
PyTypeObject CallsType = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyTypeObject RawStreamType = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", "The hot calls of the binding without ctypes.", -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void)
{
    if (!g_data_ptr && !(g_data_ptr = PyUnicode_InternFromString("data_ptr"))) return nullptr;
    CallsType.tp_name = "_fastcall.Calls";
    CallsType.tp_basicsize = sizeof(Calls);
    CallsType.tp_flags = Py_TPFLAGS_DEFAULT;
    CallsType.tp_new = calls_new;
    CallsType.tp_dealloc = calls_gone;
    CallsType.tp_methods = calls_methods;
    RawStreamType.tp_name = "_fastcall.RawStream";
    RawStreamType.tp_basicsize = sizeof(RawStream);
    RawStreamType.tp_flags = Py_TPFLAGS_DEFAULT;
    RawStreamType.tp_new = raw_stream_new;
    RawStreamType.tp_dealloc = raw_stream_gone;
    RawStreamType.tp_call = raw_stream_call;
    if (PyType_Ready(&CallsType) < 0 || PyType_Ready(&RawStreamType) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    if (PyModule_AddObjectRef(m, "Calls", reinterpret_cast<PyObject *>(&CallsType)) < 0 ||
        PyModule_AddObjectRef(m, "RawStream", reinterpret_cast<PyObject *>(&RawStreamType)) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
