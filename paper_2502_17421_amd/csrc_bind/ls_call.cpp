// Calls into the C ABI of include/ls_attn.h from Python: Caller(address, name, addresses) is a callable whose arguments are
// those of the entry point, a tensor or None (or, if `addresses`, an integer address) where it takes a pointer, the stream's
// handle, the ls_desc structure where it takes one.
// It returns the status.  A call with 13 arguments that is refused at once takes 0.14 us of the host, through ctypes 1.2; a program
// that accepts a path and commits its rows, two calls bound by the host, takes 9.1 us a round instead of 10.75.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <cstring>
#include <tuple>
#include <type_traits>
#include <utility>

#include <torch/csrc/autograd/python_variable.h>

#include "ls_attn.h"

namespace {

// An argument as the C function takes it; false: a Python error is set.
bool convert(PyObject *obj, const ls_desc *&value, bool)
{
    Py_buffer view;
    if (PyObject_GetBuffer(obj, &view, PyBUF_SIMPLE) != 0) return false;
    const bool fits = view.len == (Py_ssize_t)sizeof(ls_desc);
    value = (const ls_desc *)view.buf;  // lives as long as the structure, which the caller holds
    PyBuffer_Release(&view);
    if (!fits) PyErr_SetString(PyExc_TypeError, "expected an ls_desc");
    return fits;
}

bool integer(PyObject *obj, unsigned long long &value)  // wraps around like a C conversion
{
    value = PyLong_AsUnsignedLongLongMask(obj);
    return !(value == (unsigned long long)-1 && PyErr_Occurred());
}

template <typename T> std::enable_if_t<std::is_integral_v<T>, bool> convert(PyObject *obj, T &value, bool)
{
    unsigned long long wide = 0;
    if (!integer(obj, wide)) return false;
    value = (T)wide;
    return true;
}

template <typename T> bool convert(PyObject *obj, T *&value, bool address_taken)
{
    unsigned long long address = 0;
    if (obj == Py_None) {
        value = nullptr;
        return true;
    }
    if (address_taken && PyLong_Check(obj)) {
        if (!integer(obj, address)) return false;
    } else if (THPVariable_CheckExact(obj)) {
        try {
            address = (unsigned long long)(uintptr_t)THPVariable_Unpack(obj).data_ptr();
        } catch (const std::exception &e) {  // a tensor without storage
            PyErr_SetString(PyExc_RuntimeError, e.what());
            return false;
        }
    } else {  // a subclass, which may say something else, or another object with a data_ptr()
        PyObject *ptr = PyObject_CallMethod(obj, "data_ptr", nullptr);
        if (!ptr) return false;
        const bool ok = integer(ptr, address);
        Py_DECREF(ptr);
        if (!ok) return false;
    }
    value = (T *)(uintptr_t)address;
    return true;
}

template <typename... A, size_t... I>
PyObject *call_typed(int (*fn)(A...), PyObject *const *args, bool addresses, std::index_sequence<I...>)
{
    std::tuple<A...> values;
    // (the last argument is the stream)
    if (!(convert(args[I], std::get<I>(values), addresses || I + 1 == sizeof...(I)) && ...)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(std::get<I>(values)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

typedef PyObject *(*Invoke)(void *, PyObject *const *, bool);

template <typename F> struct Typed;
template <typename... A> struct Typed<int (*)(A...)> {
    static constexpr int count = sizeof...(A);
    static PyObject *invoke(void *fn, PyObject *const *args, bool addresses)
    {
        return call_typed((int (*)(A...))fn, args, addresses, std::index_sequence_for<A...>{});
    }
};

struct Entry {
    const char *name;
    Invoke invoke;
    int count;
};
#define LS_ENTRY(NAME) {#NAME, &Typed<decltype(&NAME)>::invoke, Typed<decltype(&NAME)>::count}
const Entry kEntries[] = {
    LS_ENTRY(ls_hybrid_tree_attn), LS_ENTRY(ls_hybrid_tree_attn_single), LS_ENTRY(ls_hybrid_tree_attn_static),
    LS_ENTRY(ls_hybrid_tree_attn_fused), LS_ENTRY(ls_hybrid_tree_attn_paged), LS_ENTRY(ls_workspace_init),
    LS_ENTRY(ls_cache_attn), LS_ENTRY(ls_cache_attn_paged), LS_ENTRY(ls_build_tree_mask), LS_ENTRY(ls_prefix_attn_splitkv),
    LS_ENTRY(ls_tree_attn_masked), LS_ENTRY(ls_lse_merge), LS_ENTRY(ls_tree_accept_greedy), LS_ENTRY(ls_kv_commit),
    LS_ENTRY(ls_kv_commit_paged),
};

struct Caller {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    void *fn;
    const Entry *entry;
    bool addresses;
};

PyObject *caller_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    const Caller *c = (const Caller *)self;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
    if (n != c->entry->count || (kwnames && PyTuple_GET_SIZE(kwnames) != 0)) {
        PyErr_Format(PyExc_TypeError, "%s takes %d positional arguments", c->entry->name, c->entry->count);
        return nullptr;
    }
    return c->entry->invoke(c->fn, args, c->addresses);
}

PyObject *caller_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    unsigned long long address = 0;
    const char *name = nullptr;
    int addresses = 0;
    if (!PyArg_ParseTuple(args, "Ksp", &address, &name, &addresses)) return nullptr;
    for (const Entry &entry : kEntries) {
        if (std::strcmp(entry.name, name) != 0) continue;
        Caller *c = (Caller *)type->tp_alloc(type, 0);
        if (!c) return nullptr;
        c->vectorcall = caller_call;
        c->fn = (void *)(uintptr_t)address;
        c->entry = &entry;
        c->addresses = addresses != 0;
        return (PyObject *)c;
    }
    PyErr_Format(PyExc_ValueError, "no entry point %s", name);
    return nullptr;
}

PyTypeObject CallerType = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_ls_call", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ls_call(void)
{
    CallerType.tp_name = "_ls_call.Caller";
    CallerType.tp_basicsize = sizeof(Caller);
    CallerType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
    CallerType.tp_vectorcall_offset = offsetof(Caller, vectorcall);
    CallerType.tp_call = PyVectorcall_Call;
    CallerType.tp_new = caller_new;
    if (PyType_Ready(&CallerType) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    // what the signatures above, and the tensor type, come from: the loader compares it with what it has
    if (PyModule_AddStringConstant(m, "interface_id", LS_INTERFACE_ID) < 0 ||
        PyModule_AddStringConstant(m, "torch_version", LS_TORCH_VERSION) < 0 ||
        PyModule_AddStringConstant(m, "python_version", PY_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    Py_INCREF(&CallerType);
    if (PyModule_AddObject(m, "Caller", (PyObject *)&CallerType) < 0) {
        Py_DECREF(&CallerType);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
