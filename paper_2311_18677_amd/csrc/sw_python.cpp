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

PyObject *s_data_ptr, *s_cuda_stream, *s_value, *s_as_parameter;       // interned attribute names
PyObject *g_cast, *g_void_p, *g_int;                  // ctypes.cast, ctypes.c_void_p, ctypes.c_int
PyObject *g_ctypes_error, *g_argument_error;          // ctypes.ArgumentError; and it as a TypeError too

// Objects that hold an address until the call is over.
struct Kept {
    PyObject *object[16];
    int n = 0;
    ~Kept()
    {
        while (n > 0) Py_DECREF(object[--n]);
    }
};

// What a ctypes prototype refuses: ctypes.ArgumentError, which callers of it catch, and a TypeError.
bool refuse(size_t at, const char *want, PyObject *x)
{
    PyErr_Format(g_argument_error, "argument %zu: %s, not %s", at + 1, want, Py_TYPE(x)->tp_name);
    return false;
}

// None -> NULL, an integer -> itself, anything else -> its `method`() (or attribute): None, an integer or
// what ctypes takes for a void pointer, text and bytes aside, which are no device addresses.
bool address_of(PyObject *x, size_t at, PyObject *name, bool method, void **out, Kept &kept)
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
            if (PyUnicode_Check(got) || PyBytes_Check(got)) {
                refuse(at, "an address is required", got);
            } else if (got != Py_None) {
                pointer = PyObject_CallFunctionObjArgs(g_cast, got, g_void_p, nullptr);
                if (pointer) {
                    value = PyObject_GetAttr(pointer, s_value);
                } else if (PyErr_ExceptionMatches(g_ctypes_error)) {
                    PyErr_Clear();
                    refuse(at, "an address is required", got);
                }
            }
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

// The int argument number `at`, taken modulo 2^32 as C takes it, from what a c_int prototype takes: an
// integer, a c_int, or an object whose _as_parameter_ is one.
bool integer_of(PyObject *x, size_t at, unsigned long long *out)
{
    PyObject *got = nullptr;
    if (!PyLong_Check(x)) {
        const int is_int = PyObject_IsInstance(x, g_int);
        if (is_int < 0) return false;
        got = is_int ? PyObject_GetAttr(x, s_value) : PyNumber_Index(x);
        if (!got) {
            PyErr_Clear();
            PyObject *inner = PyObject_GetAttr(x, s_as_parameter);
            if (!inner) {
                PyErr_Clear();
                return refuse(at, "an integer is required", x);
            }
            bool ok = false;
            if (Py_EnterRecursiveCall(" while processing _as_parameter_") == 0) {
                ok = integer_of(inner, at, out);
                Py_LeaveRecursiveCall();
            }
            Py_DECREF(inner);
            return ok;
        }
        x = got;
    }
    *out = PyLong_AsUnsignedLongLongMask(x);
    Py_XDECREF(got);
    return !(*out == (unsigned long long)-1 && PyErr_Occurred());
}

// A row count, modulo 2^64: whatever int() takes.
bool rows_of(PyObject *x, unsigned long long *out)
{
    PyObject *got = PyLong_Check(x) ? nullptr : PyNumber_Long(x);
    if (!got && !PyLong_Check(x)) return false;
    *out = PyLong_AsUnsignedLongLongMask(got ? got : x);
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
        for (size_t k = 0; k < sizeof...(P); ++k, ++at)
            if (!address_of(args[at], at, s_data_ptr, true, &p[k], kept)) return nullptr;
        if (ROWS && !rows_of(args[at++], &rows)) return nullptr;
        for (size_t k = 0; k < sizeof...(I); ++k, ++at)
            if (!integer_of(args[at], at, &v[k])) return nullptr;
        if (!address_of(args[at], at, s_cuda_stream, false, &stream, kept)) return nullptr;
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
        if (!x || !rows_of(x, &v) || v == 0) {
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
    s_as_parameter = PyUnicode_InternFromString("_as_parameter_");
    PyObject *ctypes = PyImport_ImportModule("ctypes");
    if (!ctypes) return nullptr;
    g_cast = PyObject_GetAttrString(ctypes, "cast");
    g_void_p = PyObject_GetAttrString(ctypes, "c_void_p");
    g_int = PyObject_GetAttrString(ctypes, "c_int");
    g_ctypes_error = PyObject_GetAttrString(ctypes, "ArgumentError");
    Py_DECREF(ctypes);
    if (!s_data_ptr || !s_cuda_stream || !s_value || !s_as_parameter || !g_cast || !g_void_p || !g_int || !g_ctypes_error) return nullptr;
    PyObject *bases = PyTuple_Pack(2, g_ctypes_error, PyExc_TypeError);
    if (bases) g_argument_error = PyErr_NewException("sw_native.ArgumentError", bases, nullptr);
    Py_XDECREF(bases);
    if (!g_argument_error || PyType_Ready(&kLibraryType) < 0) return nullptr;
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
