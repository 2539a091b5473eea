// The Python side of a call, natively: takes the device addresses out of the arguments and calls
// the library's entry point.  An extension module of its own (sw_native), so that libsw_decode.so
// stays free of Python; binding.py hands it the entry points' addresses, one Library object
// per loaded library.
//
// What bounds the smallest calls is the host.  ctypes converts every argument through a Python-level
// type, and the addresses were looked up in Python before that: with an entry point that does nothing
// a decode call with append took 6.0 us through ctypes and takes 1.1 here.  Two layers of four short
// chats, 8 heads of 64: 10.2 -> 8.8 us, which is what the GPU takes.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include "sw_decode.h"

#include <cstddef>
#include <cstdint>
#include <utility>

namespace {

PyObject *s_data_ptr, *s_cuda_stream, *s_value;       // interned attribute names
PyObject *g_cast, *g_void_p;                          // ctypes.cast, ctypes.c_void_p

// Objects that hold an address until the call is over.
struct Kept {
    PyObject *object[16];
    int n = 0;
    ~Kept()
    {
        while (n > 0) Py_DECREF(object[--n]);
    }
};

// None -> NULL, an integer -> itself, anything else -> its `method`() (or attribute): None, an integer or
// what ctypes takes for a void pointer, text and bytes aside, which are no device addresses.
bool address_of(PyObject *x, PyObject *name, bool method, void **out, Kept &kept)
{
    *out = nullptr;
    if (x == Py_None) return true;
    PyObject *got = nullptr;
    if (!PyLong_CheckExact(x)) {
        got = method ? PyObject_CallMethodNoArgs(x, name) : PyObject_GetAttr(x, name);
        if (!got) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
            if (method) {                               // missing, or raised by the call itself, which stands
                PyObject *type, *what, *trace;
                PyErr_Fetch(&type, &what, &trace);
                if (PyObject_HasAttr(x, name)) {
                    PyErr_Restore(type, what, trace);
                    return false;
                }
                Py_XDECREF(type);
                Py_XDECREF(what);
                Py_XDECREF(trace);
            } else {
                PyErr_Clear();
            }
            got = PyNumber_Long(x);                     // an object without it: anything that int() takes
            if (!got) return false;
        } else if (!PyLong_Check(got)) {
            PyObject *pointer = nullptr, *value = nullptr;
            if (PyUnicode_Check(got) || PyBytes_Check(got))
                PyErr_SetString(PyExc_TypeError, "an address must be an integer");
            else if (got != Py_None && (pointer = PyObject_CallFunctionObjArgs(g_cast, got, g_void_p, nullptr)))
                value = PyObject_GetAttr(pointer, s_value);
            const bool null = got == Py_None || value == Py_None;
            Py_DECREF(got);
            if (pointer) kept.object[kept.n++] = pointer;         // (which refers to what it was made from)
            if (null) {
                Py_XDECREF(value);
                return true;
            }
            if (!value) return false;
            got = value;
        }
        x = got;
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(x);
    Py_XDECREF(got);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *out = reinterpret_cast<void *>((uintptr_t)v);
    return true;
}

// An int argument, taken modulo 2^32 (2^64 for a long long) as C takes it; ctypes integers too.  ANY:
// whatever int() takes.
template <bool ANY>
bool integer_of(PyObject *x, unsigned long long *out)
{
    PyObject *got = nullptr;
    if (!PyLong_Check(x)) {
        got = ANY ? PyNumber_Long(x) : PyNumber_Index(x);
        if (!got && !ANY && PyErr_ExceptionMatches(PyExc_TypeError)) {
            PyObject *type, *what, *trace;
            PyErr_Fetch(&type, &what, &trace);
            got = PyObject_GetAttr(x, s_value);
            if (got && !PyLong_Check(got)) Py_CLEAR(got);
            if (got) {
                Py_XDECREF(type);
                Py_XDECREF(what);
                Py_XDECREF(trace);
            } else {
                PyErr_Clear();
                PyErr_Restore(type, what, trace);
            }
        }
        if (!got) return false;
        x = got;
    }
    *out = PyLong_AsUnsignedLongLongMask(x);
    Py_XDECREF(got);
    return !(*out == (unsigned long long)-1 && PyErr_Occurred());
}

template <size_t>
using pointer_t = void *;
template <size_t>
using int_t = int;

// An entry point of P pointers, a row count if ROWS, I ints and the stream.
template <bool ROWS, class PS, class IS>
struct Caller;
template <bool ROWS, size_t... P, size_t... I>
struct Caller<ROWS, std::index_sequence<P...>, std::index_sequence<I...>> {
    static constexpr Py_ssize_t kArgs = (Py_ssize_t)(sizeof...(P) + ROWS + sizeof...(I) + 1);
    static PyObject *call(uintptr_t fn, const char *name, PyObject *const *args, Py_ssize_t n)
    {
        if (n != kArgs) {
            PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, not %zd", name, kArgs, n);
            return nullptr;
        }
        static_assert(sizeof...(P) + 1 <= sizeof(Kept::object) / sizeof(PyObject *), "an object per address");
        void *p[sizeof...(P)], *stream;
        Kept kept;
        unsigned long long rows = 0, v[sizeof...(I)];
        size_t at = 0;
        for (size_t k = 0; k < sizeof...(P); ++k)
            if (!address_of(args[at++], s_data_ptr, true, &p[k], kept)) return nullptr;
        if (ROWS && !integer_of<true>(args[at++], &rows)) return nullptr;
        for (size_t k = 0; k < sizeof...(I); ++k)
            if (!integer_of<false>(args[at++], &v[k])) return nullptr;
        if (!address_of(args[at], s_cuda_stream, false, &stream, kept)) return nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        if constexpr (ROWS)
            rc = reinterpret_cast<int (*)(pointer_t<P>..., long long, int_t<I>..., void *)>(fn)(p[P]..., (long long)rows, (int)v[I]..., stream);
        else
            rc = reinterpret_cast<int (*)(pointer_t<P>..., int_t<I>..., void *)>(fn)(p[P]..., (int)v[I]..., stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    }
};
template <size_t P, bool ROWS, size_t I>
using Call = Caller<ROWS, std::make_index_sequence<P>, std::make_index_sequence<I>>;

// name, pointers, row count, ints; the ABI's own prototypes check the shapes below
#define SW_ENTRIES(X)                     \
    X(sw_decode_attn, 5, false, 5)        \
    X(sw_decode_attn_static, 5, false, 5) \
    X(sw_decode_attn_paged, 6, false, 7)  \
    X(sw_decode_attn_append, 7, false, 5) \
    X(sw_decode_attn_paged_append, 8, false, 7) \
    X(sw_advance_lens, 1, false, 2)       \
    X(sw_prefill_attn, 6, true, 5)        \
    X(sw_prefill_attn_paged, 7, true, 7)  \
    X(sw_mixed_attn, 7, true, 6)          \
    X(sw_mixed_attn_paged, 8, true, 8)    \
    X(sw_kv_store, 7, true, 5)            \
    X(sw_kv_store_paged, 8, true, 7)      \
    X(sw_kv_pack, 6, false, 7)            \
    X(sw_kv_unpack, 6, false, 7)          \
    X(sw_kv_span_plan, 5, false, 4)

template <class F>
struct Arity;
template <class... A>
struct Arity<int (*)(A...)> {
    static constexpr size_t n = sizeof...(A);
    static constexpr size_t bytes = (0 + ... + sizeof(A));
};
#define SW_CHECK(name, P, ROWS, I)                                                                        \
    static_assert(Arity<decltype(&name)>::n == (P) + (ROWS) + (I) + 1 &&                                  \
                      Arity<decltype(&name)>::bytes == 8 * ((P) + (ROWS) + 1) + 4 * (I), #name);
SW_ENTRIES(SW_CHECK)
#undef SW_CHECK

enum Entry {
#define SW_INDEX(name, P, ROWS, I) k_##name,
    SW_ENTRIES(SW_INDEX)
#undef SW_INDEX
    kEntries
};

const char *const kNames[kEntries] = {
#define SW_NAME(name, P, ROWS, I) #name,
    SW_ENTRIES(SW_NAME)
#undef SW_NAME
};

struct Library {
    PyObject_HEAD
    uintptr_t fn[kEntries];
};

#define SW_METHOD(name, P, ROWS, I)                                                        \
    PyObject *call_##name(PyObject *self, PyObject *const *args, Py_ssize_t n)             \
    {                                                                                      \
        return Call<P, ROWS, I>::call(reinterpret_cast<Library *>(self)->fn[k_##name], #name, args, n); \
    }
SW_ENTRIES(SW_METHOD)
#undef SW_METHOD

PyMethodDef kMethods[] = {
#define SW_DEF(name, P, ROWS, I) {#name, (PyCFunction)(void (*)(void))call_##name, METH_FASTCALL, nullptr},
    SW_ENTRIES(SW_DEF)
#undef SW_DEF
    {nullptr, nullptr, 0, nullptr}};

// Library(addresses): addresses[name] of every entry point
PyObject *library_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    PyObject *addresses;
    if (!PyArg_ParseTuple(args, "O!", &PyDict_Type, &addresses)) return nullptr;
    Library *self = reinterpret_cast<Library *>(type->tp_alloc(type, 0));
    if (!self) return nullptr;
    for (int k = 0; k < kEntries; ++k) {
        PyObject *x = PyDict_GetItemString(addresses, kNames[k]);        // borrowed
        unsigned long long v = 0;
        if (!x) PyErr_SetString(PyExc_KeyError, kNames[k]);
        if (!x || !integer_of<false>(x, &v) || v == 0) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, kNames[k]);
            Py_DECREF(self);
            return nullptr;
        }
        self->fn[k] = (uintptr_t)v;
    }
    return reinterpret_cast<PyObject *>(self);
}

PyTypeObject kLibraryType = [] {
    PyTypeObject t = {PyVarObject_HEAD_INIT(nullptr, 0)};
    t.tp_name = "sw_native.Library";
    t.tp_basicsize = sizeof(Library);
    t.tp_flags = Py_TPFLAGS_DEFAULT;
    t.tp_methods = kMethods;
    t.tp_new = library_new;
    return t;
}();

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "sw_native", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_sw_native(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_value = PyUnicode_InternFromString("value");
    PyObject *ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes) return nullptr;
    g_cast = PyObject_GetAttrString(ctypes, "cast");
    g_void_p = PyObject_GetAttrString(ctypes, "c_void_p");
    Py_DECREF(ctypes);
    if (!s_data_ptr || !s_cuda_stream || !s_value || !g_cast || !g_void_p || PyType_Ready(&kLibraryType) < 0) return nullptr;
    PyObject *m = PyModule_Create(&kModule);
    if (!m) return nullptr;
    PyObject *names = PyTuple_New(kEntries);
    for (int k = 0; names && k < kEntries; ++k) {
        PyObject *s = PyUnicode_FromString(kNames[k]);
        if (!s) Py_CLEAR(names);
        else PyTuple_SET_ITEM(names, k, s);
    }
    Py_INCREF(&kLibraryType);
    if (!names || PyModule_AddObject(m, "NAMES", names) < 0 ||
        PyModule_AddObject(m, "Library", reinterpret_cast<PyObject *>(&kLibraryType)) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
