// CPython entry points of the calls that a decoding step makes: arguments straight to the C ABI.
//
// A step of a small model is bound by what the host spends per call beside the 2 - 3 us of a kernel launch. A call of
// vs_tree_verify_attention that is refused at once takes, with nine tensors / nine plain addresses, 6.3 / 3.6 us through ctypes (ten
// attribute tests and data_ptr() calls in Python, then ctypes' own conversions) and 1.3 / 0.3 us here. Accepted arguments,
// their conversions and defaults are those of the ctypes functions (tests/test_pycall.py compares the two): for a pointer None, an
// integer, anything with data_ptr(), or what binding._ptr makes an address of; for a scalar a number, a ctypes scalar of the
// parameter's own type or an object with _as_parameter_ that leads to one, integers of any size cut to the
// parameter's width; ctypes.ArgumentError for what converts to neither. The
// interpreter lock is released around the call. The library is not linked: binding.lib() loads it at the first call
// and hands its addresses over, so that the same module serves any build of it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <string>
#include <tuple>
#include <utility>

#include "vispec_verify.h"

namespace {

PyObject *s_data_ptr, *g_load, *g_ptr, *g_scalar, *g_struct, *g_error, *g_attn_desc, *g_kv_desc; // setup()

constexpr int kMaxArgs = 20;
struct Entry {
    const char* name;
    const char* args;  // names, separated by spaces
    int required;      // the others default to 0 / NULL
    void* fn;
    int count;
    PyObject* names[kMaxArgs];
};

// whatever was raised becomes an ArgumentError that names the argument
bool argument_error(int i) {
    if (!PyErr_ExceptionMatches(PyExc_Exception)) return false;
    PyObject *type, *value, *trace;
    PyErr_Fetch(&type, &value, &trace);
    PyErr_NormalizeException(&type, &value, &trace);
    PyErr_Format(g_error, "argument %d: %S: %S", i + 1, type, value);
    Py_XDECREF(type);
    Py_XDECREF(value);
    Py_XDECREF(trace);
    return false;
}
bool to_integer(PyObject* o, int i, char code, uint64_t& x) {
    if (PyLong_Check(o)) {
        x = PyLong_AsUnsignedLongLongMask(o);
        return true;
    }
    PyObject* n = PyNumber_Index(o);
    if (!n) { // a ctypes scalar, an object that stands for one, or an error
        PyErr_Clear();
        n = PyObject_CallFunction(g_scalar, "CO", (int)code, o);
        if (!n) return argument_error(i);
    }
    x = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return true;
}
bool to_address(PyObject* o, int i, uint64_t& x) {
    x = 0;
    if (o == Py_None) return true;
    PyObject* a = nullptr;
    if (PyLong_Check(o)) {
        a = o;
        Py_INCREF(a);
    } else if (!(a = PyObject_CallMethodNoArgs(o, s_data_ptr))) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
        PyErr_Clear();
        a = PyObject_CallOneArg(g_ptr, o);
        if (!a) return false;
    }
    bool ok = a == Py_None;
    if (!ok && PyLong_Check(a)) {
        x = PyLong_AsUnsignedLongLongMask(a);
        ok = true;
    } else if (!ok) { // data_ptr() gave something else
        PyObject* n = PyObject_CallFunction(g_scalar, "CO", 'P', a);
        if (n && n != Py_None) x = PyLong_AsUnsignedLongLongMask(n);
        ok = n || argument_error(i);
        Py_XDECREF(n);
    }
    Py_DECREF(a);
    return ok;
}
bool to_struct(PyObject* o, int i, PyObject* type, size_t bytes, uint64_t& x) {
    Py_buffer b;
    if (!PyObject_TypeCheck(o, (PyTypeObject*)type)) {
        PyObject* n = PyObject_CallOneArg(g_struct, o); // TypeError if it is no ctypes object at all
        if (!n) return false;
        Py_DECREF(n);
        PyErr_Format(g_error, "argument %d: expected %s instance instead of %s", i + 1, ((PyTypeObject*)type)->tp_name, Py_TYPE(o)->tp_name);
        return false;
    }
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) < 0) return false;
    const bool ok = (size_t)b.len >= bytes;
    x = (uint64_t)(uintptr_t)b.buf; // the caller holds the object for the whole call
    PyBuffer_Release(&b);
    if (!ok) PyErr_Format(g_error, "argument %d: a descriptor of %zu bytes is required", i + 1, bytes);
    return ok;
}

bool convert(PyObject* o, int i, int32_t& x) {
    uint64_t v;
    if (!to_integer(o, i, 'i', v)) return false;
    x = (int32_t)v;
    return true;
}
bool convert(PyObject* o, int i, int64_t& x) {
    uint64_t v;
    if (!to_integer(o, i, 'q', v)) return false;
    x = (int64_t)v;
    return true;
}
bool convert(PyObject* o, int i, size_t& x) {
    uint64_t v;
    if (!to_integer(o, i, 'N', v)) return false;
    x = (size_t)v;
    return true;
}
bool convert(PyObject* o, int i, float& x) {
    double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        PyObject* n = PyObject_CallFunction(g_scalar, "CO", 'f', o);
        if (!n) return argument_error(i);
        v = PyFloat_AsDouble(n);
        Py_DECREF(n);
    }
    x = (float)v;
    return true;
}
bool convert(PyObject* o, int i, const vs_attn_desc*& x) {
    uint64_t v;
    if (!to_struct(o, i, g_attn_desc, sizeof(vs_attn_desc), v)) return false;
    x = (const vs_attn_desc*)v;
    return true;
}
bool convert(PyObject* o, int i, const vs_kv_desc*& x) {
    uint64_t v;
    if (!to_struct(o, i, g_kv_desc, sizeof(vs_kv_desc), v)) return false;
    x = (const vs_kv_desc*)v;
    return true;
}
template <typename T>
bool convert(PyObject* o, int i, T*& x) {
    uint64_t v;
    if (!to_address(o, i, v)) return false;
    x = (T*)v;
    return true;
}

// positional and keyword arguments in the order of the parameters; absent ones stay null
bool gather(const Entry& e, PyObject* const* args, Py_ssize_t n, PyObject* kwnames, PyObject** to) {
    if (n > e.count) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", e.name, e.count, n);
        return false;
    }
    for (Py_ssize_t i = 0; i < n; ++i) to[i] = args[i];
    const Py_ssize_t kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < kw; ++k) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, k);
        int at = 0;
        while (at < e.count && e.names[at] != name && PyUnicode_Compare(e.names[at], name) != 0) ++at;
        if (at == e.count || to[at]) {
            PyErr_Format(PyExc_TypeError, at == e.count ? "%s() got an unexpected keyword argument '%U'" : "%s() got multiple values for argument '%U'",
                         e.name, name);
            return false;
        }
        to[at] = args[n + k];
    }
    for (int i = 0; i < e.required; ++i)
        if (!to[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%U'", e.name, e.names[i]);
            return false;
        }
    return true;
}

template <typename... A, size_t... I>
PyObject* invoke(Entry& e, PyObject** given, std::index_sequence<I...>) {
    std::tuple<A...> a{};
    if (!(... && (!given[I] || convert(given[I], (int)I, std::get<I>(a))))) return nullptr;
    if (!e.fn) {
        PyObject* r = g_load ? PyObject_CallNoArgs(g_load) : nullptr; // ends in bind()
        if (!r) return nullptr;
        Py_DECREF(r);
        if (!e.fn) return PyErr_Format(PyExc_RuntimeError, "%s is not bound", e.name);
    }
    int32_t rc;
    auto fn = (int32_t(*)(A...))e.fn;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(std::get<I>(a)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}
template <typename... A>
PyObject* call(Entry& e, int32_t (*)(A...), PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {
    PyObject* given[sizeof...(A)] = {};
    if (!gather(e, args, n, kwnames, given)) return nullptr;
    return invoke<A...>(e, given, std::index_sequence_for<A...>{});
}
template <typename... A>
constexpr int arity(int32_t (*)(A...)) { return (int)sizeof...(A); }

Entry entries[] = {
    {"vs_tree_mask_build", "parent B T mask depth status stream", 5},
    {"vs_tree_verify_attention", "desc q k_cache v_cache prefix_len tree_parent tree_mask out status workspace workspace_bytes stream", 8},
    {"vs_compress_attention", "desc q k v kv_len out status workspace workspace_bytes stream", 6},
    {"vs_tree_accept",
     "logits ld_logits V draft_tokens parent B T accepted_len path bonus_token row_argmax status workspace workspace_bytes stream", 10},
    {"vs_tree_accept_noalloc", "logits ld_logits V draft_tokens parent B T accepted_len path bonus_token row_argmax status stream", 10},
    {"vs_tree_accept_sample",
     "logits ld_logits V temperature draft_tokens parent u_accept u_bonus B T accepted_len path bonus_token status workspace workspace_bytes "
     "stream", 13},
    {"vs_draft_expand",
     "logits ld_logits V cum_in frontier_cand B F K cand_base cand_capacity cand_token cand_score cand_parent next_frontier_cand next_cum "
     "workspace workspace_bytes stream", 15},
    {"vs_draft_tree_build",
     "cand_token cand_score cand_parent B M cand_capacity N root_token parent draft_tokens node_cand num_nodes status stream", 12},
    {"vs_tree_kv_commit", "desc k_cache v_cache prefix_len path accepted_len new_prefix_len status stream", 7},
};

#define VS_ENTRY(INDEX, NAME)                                                                       \
    PyObject* py_##NAME(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kwnames) {        \
        static_assert(arity((decltype(&NAME))nullptr) <= kMaxArgs, "");                             \
        return call(entries[INDEX], (decltype(&NAME))nullptr, args, n, kwnames);                    \
    }
VS_ENTRY(0, vs_tree_mask_build)
VS_ENTRY(1, vs_tree_verify_attention)
VS_ENTRY(2, vs_compress_attention)
VS_ENTRY(3, vs_tree_accept)
VS_ENTRY(4, vs_tree_accept_noalloc)
VS_ENTRY(5, vs_tree_accept_sample)
VS_ENTRY(6, vs_draft_expand)
VS_ENTRY(7, vs_draft_tree_build)
VS_ENTRY(8, vs_tree_kv_commit)

// setup(load, ptr, scalar, byref, ArgumentError, AttnDesc, KVDesc)
PyObject* setup(PyObject*, PyObject* args) {
    if (!PyArg_ParseTuple(args, "OOOOOO!O!", &g_load, &g_ptr, &g_scalar, &g_struct, &g_error, &PyType_Type, &g_attn_desc, &PyType_Type, &g_kv_desc))
        return nullptr;
    for (PyObject* o : {g_load, g_ptr, g_scalar, g_struct, g_error, g_attn_desc, g_kv_desc}) Py_INCREF(o); // for good
    Py_RETURN_NONE;
}
// bind({name: address})
PyObject* bind(PyObject*, PyObject* addresses) {
    for (Entry& e : entries) {
        PyObject* a = PyMapping_GetItemString(addresses, e.name);
        if (!a) return nullptr;
        e.fn = PyLong_AsVoidPtr(a);
        Py_DECREF(a);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_RETURN_NONE;
}

#define VS_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))py_##NAME, METH_FASTCALL | METH_KEYWORDS, nullptr}
PyMethodDef methods[] = {
    VS_METHOD(vs_tree_mask_build), VS_METHOD(vs_tree_verify_attention), VS_METHOD(vs_compress_attention), VS_METHOD(vs_tree_accept),
    VS_METHOD(vs_tree_accept_noalloc), VS_METHOD(vs_tree_accept_sample), VS_METHOD(vs_draft_expand), VS_METHOD(vs_draft_tree_build),
    VS_METHOD(vs_tree_kv_commit),
    {"setup", setup, METH_VARARGS, nullptr},
    {"bind", bind, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Calls into libvispec_verify, see binding.py.", -1, methods};

} // namespace

PyMODINIT_FUNC PyInit__native() {
    static std::string docs[sizeof(entries) / sizeof(entries[0])];
    int k = 0;
    for (Entry& e : entries) {
        // parameter names, and a signature for help() and inspect
        std::string doc = std::string(e.name) + "($module, /", list = e.args, word;
        list += ' ';
        e.count = 0;
        for (char c : list) {
            if (c != ' ') {
                word += c;
                continue;
            }
            e.names[e.count] = PyUnicode_InternFromString(word.c_str());
            if (!e.names[e.count]) return nullptr;
            doc += ", " + word + (e.count < e.required ? "" : word == "workspace_bytes" ? "=0" : "=None");
            ++e.count;
            word.clear();
        }
        docs[k] = doc + ")\n--\n\nSee include/vispec_verify.h.";
        methods[k].ml_doc = docs[k].c_str();
        ++k;
    }
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    return s_data_ptr ? PyModule_Create(&module) : nullptr;
}
