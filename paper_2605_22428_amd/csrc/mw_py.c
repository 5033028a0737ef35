// Python entry to the calls of the path.  One C function per call takes the tensors as they are: an address
// is what their data_ptr() says, None is a null pointer, a stream or a host record is an int, a context its ctypes
// pointer.  Numbers are cut to the parameter's width as ctypes cuts them.  The interpreter lock is released around the call.
// The functions are those of the library that the binding has loaded: it hands their addresses to bind().  A module linked to the
// library would get the first one of that file name in the process, another tree's for instance.
//
// What it is for: a small batch's pass is the host's time.  A call with ten tensors took 5.5 us through ctypes, 1 of them for its
// objects and conversions, 1 in Python, and 2.6 in the runtime's launch.  us, ctypes / this: mw_plan_pack and mw_unpack of 128 tokens
// 13.2 / 11.5, mw_allgather_step of a few KiB 5.4 / 4.2, mw_plan and mw_pack_quantize of 1000 tokens 11.9 / 11.3.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "mw.h"

static PyObject *s_data_ptr, *s_value;

// kind h: context, t: tensor or None, p: address, i: int32, l: int64.  Returns 0, or -1 with an exception set.
static int to_word(PyObject *o, char kind, uint64_t *out)
{
    PyObject *n;
    if (o == Py_None && (kind == 'h' || kind == 't')) {
        *out = 0;
        return 0;
    }
    if (kind == 'h') n = PyObject_GetAttr(o, s_value);
    else if (kind == 't') n = PyObject_CallMethodNoArgs(o, s_data_ptr);
    else n = PyNumber_Index(o);
    if (!n) return -1;
    *out = n == Py_None ? 0 : PyLong_AsUnsignedLongLongMask(n);          // (None: a null ctypes pointer)
    Py_DECREF(n);
    return *out == (uint64_t)-1 && PyErr_Occurred() ? -1 : 0;
}

#define MAX_ARGS 16
static PyObject *run(const char *name, const char *kinds, Py_ssize_t n_kinds, PyObject *const *args, Py_ssize_t n,
                     int32_t (*go)(const uint64_t *), int bound)
{
    uint64_t v[MAX_ARGS];
    if (!bound) return PyErr_Format(PyExc_RuntimeError, "%s is not bound to a library", name);
    if (n != n_kinds) return PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, n_kinds, n);
    for (Py_ssize_t i = 0; i < n; ++i) if (to_word(args[i], kinds[i], &v[i]) != 0) return NULL;
    int32_t status;
    Py_BEGIN_ALLOW_THREADS
    status = go(v);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

#define P(i) ((void *)(uintptr_t)v[i])
#define I(i) ((int32_t)v[i])
#define L(i) ((int64_t)v[i])
#define CALL(name, kinds, ...)                                                                              \
    static __typeof__(&name) fn_##name;                                                                     \
    static int32_t name##_go(const uint64_t *v) { return fn_##name(__VA_ARGS__); }                          \
    static PyObject *py_##name(PyObject *self, PyObject *const *args, Py_ssize_t n)                         \
    {                                                                                                       \
        _Static_assert(sizeof(kinds) - 1 <= MAX_ARGS, "room for the arguments");                            \
        return run(#name, kinds, (Py_ssize_t)sizeof(kinds) - 1, args, n, name##_go, fn_##name != NULL);     \
    }

CALL(mw_plan, "htittttp", P(0), P(1), I(2), P(3), P(4), P(5), P(6), P(7))
CALL(mw_pack, "htttttitttp", P(0), P(1), P(2), P(3), P(4), P(5), I(6), P(7), P(8), P(9), P(10))
CALL(mw_pack_quantize, "httttitttp", P(0), P(1), P(2), P(3), P(4), I(5), P(6), P(7), P(8), P(9))
CALL(mw_plan_pack, "htttitttttttp", P(0), P(1), P(2), P(3), I(4), P(5), P(6), P(7), P(8), P(9), P(10), P(11), P(12))
CALL(mw_pack_packets, "httttttitp", P(0), P(1), P(2), P(3), P(4), P(5), P(6), I(7), P(8), P(9))
CALL(mw_unpack, "htittlttttp", P(0), P(1), I(2), P(3), P(4), L(5), P(6), P(7), P(8), P(9), P(10))
CALL(mw_unpack_packets, "htittlttttp", P(0), P(1), I(2), P(3), P(4), L(5), P(6), P(7), P(8), P(9), P(10))
CALL(mw_unpack_index, "htilttp", P(0), P(1), I(2), L(3), P(4), P(5), P(6))
CALL(mw_unpack_expand, "hittlttp", P(0), I(1), P(2), P(3), L(4), P(5), P(6), P(7))
CALL(mw_combine_gather, "hitltlp", P(0), I(1), P(2), L(3), P(4), L(5), P(6))
CALL(mw_stream_step, "hpppp", P(0), P(1), P(2), P(3), P(4))
CALL(mw_plan_allgather, "hlttp", P(0), L(1), P(2), P(3), P(4))
CALL(mw_pack_allgather, "htltp", P(0), P(1), L(2), P(3), P(4))
CALL(mw_unpack_allgather, "htltp", P(0), P(1), L(2), P(3), P(4))
CALL(mw_plan_allgather_split, "hllttp", P(0), L(1), L(2), P(3), P(4), P(5))
CALL(mw_unpack_allgather_split, "httlltp", P(0), P(1), P(2), L(3), L(4), P(5), P(6))
CALL(mw_allgather_step, "htltttttp", P(0), P(1), L(2), P(3), P(4), P(5), P(6), P(7), P(8))
CALL(mw_relay, "httltp", P(0), P(1), P(2), L(3), P(4), P(5))
CALL(mw_relay_index, "httltp", P(0), P(1), P(2), L(3), P(4), P(5))
CALL(mw_relay_copy, "htttp", P(0), P(1), P(2), P(3), P(4))
CALL(mw_relay_copy_index_next, "httthttltp", P(0), P(1), P(2), P(3), P(4), P(5), P(6), L(7), P(8), P(9))
CALL(mw_relay_packets, "httltp", P(0), P(1), P(2), L(3), P(4), P(5))
CALL(mw_relay_packets_index, "htltp", P(0), P(1), L(2), P(3), P(4))
CALL(mw_relay_packets_copy, "htttp", P(0), P(1), P(2), P(3), P(4))
CALL(mw_relay_packets_copy_index_next, "httthtltp", P(0), P(1), P(2), P(3), P(4), P(5), L(6), P(7), P(8))

// The calls, once for the module's functions and once for their addresses.
#define CALLS(X)                                                                                                        \
    X(mw_plan) X(mw_pack) X(mw_pack_quantize) X(mw_plan_pack) X(mw_pack_packets) X(mw_unpack)                           \
    X(mw_unpack_packets) X(mw_unpack_index) X(mw_unpack_expand) X(mw_combine_gather) X(mw_stream_step)                  \
    X(mw_plan_allgather) X(mw_pack_allgather) X(mw_unpack_allgather) X(mw_plan_allgather_split)                         \
    X(mw_unpack_allgather_split) X(mw_allgather_step) X(mw_relay) X(mw_relay_index) X(mw_relay_copy)                    \
    X(mw_relay_copy_index_next) X(mw_relay_packets) X(mw_relay_packets_index) X(mw_relay_packets_copy)                  \
    X(mw_relay_packets_copy_index_next)

#define SLOT(name) {#name, (void **)&fn_##name},
static const struct { const char *name; void **at; } slots[] = {CALLS(SLOT)};

// bind({name: address}): every call's address, of one library.
static PyObject *bind(PyObject *self, PyObject *addresses)
{
    void *to[sizeof(slots) / sizeof(slots[0])];
    if (!PyDict_Check(addresses)) return PyErr_Format(PyExc_TypeError, "bind takes a dict of addresses");
    for (size_t i = 0; i < sizeof(slots) / sizeof(slots[0]); ++i) {
        PyObject *a = PyDict_GetItemString(addresses, slots[i].name);
        if (!a) return PyErr_Format(PyExc_KeyError, "no address for %s", slots[i].name);
        to[i] = PyLong_AsVoidPtr(a);
        if (PyErr_Occurred()) return NULL;
        if (!to[i]) return PyErr_Format(PyExc_ValueError, "%s has no address", slots[i].name);
    }
    for (size_t i = 0; i < sizeof(slots) / sizeof(slots[0]); ++i) *slots[i].at = to[i];
    Py_RETURN_NONE;
}

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, NULL},
static PyMethodDef methods[] = {CALLS(ENTRY) {"bind", bind, METH_O, NULL}, {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mwcall", "The calls of libmw.so that are made per batch.", -1, methods,
                                    NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__mwcall(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_value = PyUnicode_InternFromString("value");
    return s_data_ptr && s_value ? PyModule_Create(&module) : NULL;
}
