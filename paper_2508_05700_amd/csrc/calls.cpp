// Native marshalling of the calls whose work on the device is a few microseconds: checks the torch tensors of a
// call, takes their addresses and calls the library, as binding.py does for the others through ctypes.  What a call
// costs the host bounds a small lookup: 6.2 us with ctypes, of which the launch is 2.9 (16 arguments, six of them
// tensors; a tensor's checks and address 0.24 us each in Python).
//
// A CPython module of one function, call(entry, *args); the entry points and the types of their arguments are those of
// emb.h.  bind(entry, address, spec, slow) names the address of an entry point in the loaded library and says per
// argument which tensors it takes: None (a number or an address) or (name, dtype or tuple of dtypes).  A tensor that
// is not plainly acceptable (another class, device, dtype or layout) goes to `slow`, binding._ptr, which raises or returns
// its address.
#include <Python.h>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "emb.h"

namespace {

constexpr int MAX_ARGS = 24;

struct ArgSpec {
    PyObject *name, *dtype;   // owned
    unsigned long long mask;  // bit t: scalar type t is accepted; 0: the argument is no tensor
};

struct Entry {
    const char *name;
    int n;
    PyObject *(*invoke)(const Entry &e, PyObject *const *args);
    void *fn;
    ArgSpec spec[MAX_ARGS];
};

PyObject *slow_pointer;   // binding._ptr

bool pointer_of(PyObject *o, const ArgSpec &s, void *&out)
{
    if (o == Py_None) {
        out = nullptr;
        return true;
    }
    if (PyLong_CheckExact(o) && s.mask == 0) {
        out = PyLong_AsVoidPtr(o);
        return !PyErr_Occurred();
    }
    if (s.mask == 0) {
        PyErr_SetString(PyExc_TypeError, "an address must be an int or None");
        return false;
    }
    if (THPVariable_CheckExact(o)) {
        try {   // (a sparse tensor refuses the question for its layout, one without storage that for its address)
            const at::Tensor &t = THPVariable_Unpack(o);
            if (t.is_cuda() && ((s.mask >> (int)t.scalar_type()) & 1ull) && t.is_contiguous()) {
                out = t.data_ptr();
                return true;
            }
        } catch (...) {
            // the slow way says so
        }
    }
    PyObject *r = PyObject_CallFunctionObjArgs(slow_pointer, o, s.dtype, s.name, nullptr);
    if (!r) return false;
    out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

template <typename A>
bool convert(PyObject *o, const ArgSpec &s, A &out)
{
    if constexpr (std::is_pointer_v<A>) {
        void *p;
        if (!pointer_of(o, s, p)) return false;
        out = (A)p;
        return true;
    } else if constexpr (std::is_floating_point_v<A>) {
        out = (A)PyFloat_AsDouble(o);
        return !PyErr_Occurred();
    } else if constexpr (std::is_unsigned_v<A>) {
        static_assert(sizeof(A) == 8);
        out = (A)PyLong_AsUnsignedLongLong(o);
        return !PyErr_Occurred();
    } else {
        const long long v = PyLong_AsLongLong(o);
        out = (A)v;
        if (!PyErr_Occurred() && (long long)out != v) PyErr_SetString(PyExc_OverflowError, "number out of range");
        return !PyErr_Occurred();
    }
}

template <typename... A, size_t... I>
PyObject *invoke_with(const Entry &e, PyObject *const *args, int (*fn)(A...), std::index_sequence<I...>)
{
    std::tuple<A...> a;
    if (!(convert<A>(args[I], e.spec[I], std::get<I>(a)) && ...)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS   // as ctypes does
    rc = fn(std::get<I>(a)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

template <typename F>
struct Invoker;
template <typename... A>
struct Invoker<int (*)(A...)> {
    static constexpr int n = sizeof...(A);
    static PyObject *invoke(const Entry &e, PyObject *const *args)
    {
        return invoke_with(e, args, reinterpret_cast<int (*)(A...)>(e.fn), std::index_sequence_for<A...>());
    }
};

#define EMB_ENTRY(F) {#F, Invoker<decltype(&F)>::n, &Invoker<decltype(&F)>::invoke, nullptr, {}}
Entry entries[] = {
    EMB_ENTRY(emb_bag_forward_lengths),
    EMB_ENTRY(emb_bag_forward_hashed_lengths),
    EMB_ENTRY(emb_bag_forward_train_lengths_after),
    EMB_ENTRY(emb_bag_backward_sort_prepared),
    EMB_ENTRY(emb_bag_backward_update),
    EMB_ENTRY(emb_bag_backward_rowwise_adagrad),
    EMB_ENTRY(emb_lengths_to_offsets),
    EMB_ENTRY(emb_hash_ids_tables),
    EMB_ENTRY(emb_bag_forward_mixed),
    EMB_ENTRY(emb_bag_forward_cached_hashed_lengths),
    EMB_ENTRY(emb_bag_forward_cached_tables_hashed_lengths),
    EMB_ENTRY(emb_cache_observe_hashed),
    EMB_ENTRY(emb_cache_refresh),
};
constexpr long N_ENTRIES = sizeof(entries) / sizeof(entries[0]);

PyObject *names(PyObject *, PyObject *)
{
    PyObject *l = PyList_New(0);
    if (!l) return nullptr;
    for (const Entry &e : entries) {
        PyObject *s = Py_BuildValue("(si)", e.name, e.n);
        if (!s || PyList_Append(l, s) != 0) {
            Py_XDECREF(s);
            Py_DECREF(l);
            return nullptr;
        }
        Py_DECREF(s);
    }
    return l;
}

bool mask_of(PyObject *dtype, unsigned long long &mask)
{
    if (PyTuple_Check(dtype)) {
        for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(dtype); ++i)
            if (!mask_of(PyTuple_GET_ITEM(dtype, i), mask)) return false;
        return true;
    }
    if (!THPDtype_Check(dtype)) {
        PyErr_SetString(PyExc_TypeError, "a torch.dtype is wanted");
        return false;
    }
    mask |= 1ull << (int)reinterpret_cast<THPDtype *>(dtype)->scalar_type;
    return true;
}

// bind(entry, address, spec, slow): spec has one item per argument, None or (name, dtype)
PyObject *bind(PyObject *, PyObject *args)
{
    long k;
    unsigned long long address;
    PyObject *spec, *slow;
    if (!PyArg_ParseTuple(args, "lKO!O", &k, &address, &PyTuple_Type, &spec, &slow)) return nullptr;
    if (k < 0 || k >= N_ENTRIES || entries[k].n > MAX_ARGS || PyTuple_GET_SIZE(spec) != entries[k].n) {
        PyErr_SetString(PyExc_ValueError, "no such entry, or not its number of arguments");
        return nullptr;
    }
    Entry &e = entries[k];
    for (int i = 0; i < e.n; ++i) {
        PyObject *it = PyTuple_GET_ITEM(spec, i);
        ArgSpec s{nullptr, nullptr, 0};
        if (it != Py_None && (!PyArg_ParseTuple(it, "OO", &s.name, &s.dtype) || !mask_of(s.dtype, s.mask))) return nullptr;
        Py_XINCREF(s.name);
        Py_XINCREF(s.dtype);
        Py_XDECREF(e.spec[i].name);
        Py_XDECREF(e.spec[i].dtype);
        e.spec[i] = s;
    }
    e.fn = (void *)(uintptr_t)address;
    Py_INCREF(slow);
    Py_XDECREF(slow_pointer);
    slow_pointer = slow;
    Py_RETURN_NONE;
}

// call(entry, *args) -> status
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    const long k = nargs > 0 ? PyLong_AsLong(args[0]) : -1;
    if (k == -1 && PyErr_Occurred()) return nullptr;
    if (k < 0 || k >= N_ENTRIES || !entries[k].fn || nargs != entries[k].n + 1) {
        PyErr_SetString(PyExc_TypeError, "no such entry, or not its number of arguments");
        return nullptr;
    }
    return entries[k].invoke(entries[k], args + 1);
}

PyMethodDef methods[] = {
    {"names", names, METH_NOARGS, "the entry points, (name, number of arguments) each"},
    {"bind", bind, METH_VARARGS, "address and argument kinds of an entry point"},
    {"call", (PyCFunction)(void (*)())call, METH_FASTCALL, "calls an entry point"},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
