// The skip calls' argument marshalling as a CPython function.
//
// One anchor's skip transitions are a 3.4 us kernel behind a call that took 8.1 us: a launch of ~3 us and 5 us of ctypes structures, array
// types and argument conversion.  Here the same conversions and checks are done on the objects themselves: 8.1 -> 6.3 us a call
// (1 x 4096 elements, four targets).  The library's function comes as an address (bind), so this module links to nothing but the interpreter.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <vector>

#include "../../include/drf.h"

namespace {

typedef drf_status (*SkipFn)(const drf_sched_config*, const float*, const float*, int, const int*, int, int, size_t, const drf_noise*, float*, void*);
SkipFn g_skip = nullptr;

PyObject *k_train_steps, *k_beta_start, *k_beta_end, *k_steps, *k_eta, *k_sampler, *k_shift, *k_get, *k_is_cuda, *k_is_contiguous, *k_dtype, *k_data_ptr, *k_shape;
PyObject *k_zero, *k_one, *k_ddim;                   // eta, shift and sampler of a schedule that has none

// New reference to d[key], or to d.get(key, fallback) where there is one.
PyObject* item(PyObject* d, PyObject* key, PyObject* fallback)
{
    if (PyDict_CheckExact(d)) {
        PyObject* v = PyDict_GetItemWithError(d, key);
        if (!v && !PyErr_Occurred()) {
            v = fallback;
            if (!v) PyErr_SetObject(PyExc_KeyError, key);
        }
        Py_XINCREF(v);
        return v;
    }
    return fallback ? PyObject_CallMethodObjArgs(d, k_get, key, fallback, nullptr) : PyObject_GetItem(d, key);
}

// A C int as ctypes converts one: integers and what has __index__, the low bits of larger ones.
bool to_int(PyObject* v, int* out)
{
    const unsigned long u = PyLong_AsUnsignedLongMask(v);
    if (u == (unsigned long)-1 && PyErr_Occurred()) return false;
    *out = (int)u;
    return true;
}

// An integer; one with a fallback goes through int() first, a double with one through float() (which also take text).
bool int_item(PyObject* d, PyObject* key, int* out, PyObject* fallback = nullptr)
{
    PyObject* v = item(d, key, fallback);
    if (v && fallback) { PyObject* n = PyNumber_Long(v); Py_DECREF(v); v = n; }
    if (!v) return false;
    const bool ok = to_int(v, out);
    Py_DECREF(v);
    return ok;
}

bool double_item(PyObject* d, PyObject* key, double* out, PyObject* fallback = nullptr)
{
    PyObject* v = item(d, key, fallback);
    if (v && fallback) { PyObject* f = PyNumber_Float(v); Py_DECREF(v); v = f; }
    if (!v) return false;
    *out = PyFloat_AsDouble(v);
    Py_DECREF(v);
    return !(*out == -1.0 && PyErr_Occurred());
}

bool schedule(PyObject* d, drf_sched_config* sc)
{
    int which = 0;
    if (!int_item(d, k_train_steps, &sc->train_steps) || !double_item(d, k_beta_start, &sc->beta_start) ||
        !double_item(d, k_beta_end, &sc->beta_end) || !int_item(d, k_steps, &sc->steps) || !double_item(d, k_eta, &sc->eta, k_zero) ||
        !int_item(d, k_sampler, &which, k_ddim) || !double_item(d, k_shift, &sc->shift, k_one)) return false;
    sc->sampler = (decltype(sc->sampler))which;
    return true;
}

// Device pointer of a contiguous device tensor of the given dtype; None: NULL.
bool device_pointer(PyObject* t, PyObject* dtype, void** out)
{
    *out = nullptr;
    if (t == Py_None) return true;
    PyObject* v = PyObject_GetAttr(t, k_is_cuda);
    if (!v) return false;
    int ok = PyObject_IsTrue(v);
    Py_DECREF(v);
    if (ok > 0) {
        v = PyObject_CallMethodNoArgs(t, k_is_contiguous);
        if (!v) return false;
        ok = PyObject_IsTrue(v);
        Py_DECREF(v);
    }
    if (ok < 0) return false;
    if (!ok) { PyErr_SetString(PyExc_AssertionError, "need a contiguous device tensor"); return false; }
    v = PyObject_GetAttr(t, k_dtype);
    if (!v) return false;
    if (v != dtype) {                               // (dtypes are singletons)
        PyErr_Format(PyExc_AssertionError, "expected %S, got %S", dtype, v);
        Py_DECREF(v);
        return false;
    }
    Py_DECREF(v);
    v = PyObject_CallMethodNoArgs(t, k_data_ptr);
    if (!v) return false;
    *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !(!*out && PyErr_Occurred());
}

// skip(sched, x_from, net_from, s_from, s_to, noise_address, out, float32, stream) -> status.  stream: a handle, or what gives the current one,
// which is asked last (it initialises the device, which a call that is refused has no need of).
PyObject* skip(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 9 || !g_skip) { PyErr_SetString(PyExc_TypeError, "skip() takes 9 arguments, after bind()"); return nullptr; }
    drf_sched_config sc{};
    if (!schedule(a[0], &sc)) return nullptr;
    PyObject* shape = PyObject_GetAttr(a[1], k_shape);
    if (!shape) return nullptr;
    PyObject* dims = PySequence_Tuple(shape);
    Py_DECREF(shape);
    if (!dims) return nullptr;
    size_t batch = 1, elems = 1;                    // a tensor without dimensions: one sample of one element
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(dims); ++i) {
        const size_t v = PyLong_AsSize_t(PyTuple_GET_ITEM(dims, i));
        if (v == (size_t)-1 && PyErr_Occurred()) { Py_DECREF(dims); return nullptr; }
        (i == 0 ? batch : elems) *= v;
    }
    Py_DECREF(dims);
    if (!batch) elems = 0;
    const Py_ssize_t m = PyObject_Length(a[4]);
    if (m < 0) return nullptr;
    // a tuple of our own: an element's __index__ is anybody's code (a device tensor's gives up the interpreter lock) and may change the caller's list
    PyObject* seq = PySequence_Tuple(a[4]);
    if (!seq) return nullptr;
    int few[16];
    std::vector<int> many;
    int* to = few;
    bool ok = PyTuple_GET_SIZE(seq) == m;
    if (!ok) PyErr_SetString(PyExc_IndexError, "invalid index");
    if (ok && m > 16) {
        try { many.resize((size_t)m); to = many.data(); } catch (...) { PyErr_NoMemory(); ok = false; }
    }
    for (Py_ssize_t i = 0; ok && i < m; ++i) ok = to_int(PyTuple_GET_ITEM(seq, i), &to[i]);
    Py_DECREF(seq);
    int s_from = 0;
    void *x = nullptr, *net = nullptr, *out = nullptr, *noise = nullptr, *stream = nullptr;
    ok = ok && device_pointer(a[1], a[7], &x) && device_pointer(a[2], a[7], &net) && to_int(a[3], &s_from) && device_pointer(a[6], a[7], &out);
    if (!ok) return nullptr;
    if (a[5] != Py_None && !(noise = PyLong_AsVoidPtr(a[5])) && PyErr_Occurred()) return nullptr;
    PyObject* handle = PyLong_Check(a[8]) ? Py_NewRef(a[8]) : PyObject_CallNoArgs(a[8]);
    if (!handle) return nullptr;
    stream = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (!stream && PyErr_Occurred()) return nullptr;
    drf_status rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_skip(&sc, (const float*)x, (const float*)net, s_from, to, (int)m, (int)batch, elems, (const drf_noise*)noise, (float*)out, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)rc);
}

// bind(address of drf_skip_transition_noise)
PyObject* bind(PyObject*, PyObject* address)
{
    void* p = PyLong_AsVoidPtr(address);
    if (!p) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "NULL address");
        return nullptr;
    }
    g_skip = reinterpret_cast<SkipFn>(p);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    { "skip", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(skip)), METH_FASTCALL, "status of drf_skip_transition_noise on these arguments" },
    { "bind", bind, METH_O, "address of drf_skip_transition_noise" },
    { nullptr, nullptr, 0, nullptr },
};
PyModuleDef kModule = { PyModuleDef_HEAD_INIT, "_native", "Argument marshalling of the skip calls", -1, kMethods, nullptr, nullptr, nullptr, nullptr };

}  // namespace

PyMODINIT_FUNC PyInit__native()
{
    struct { PyObject** at; const char* text; } names[] = {
        { &k_train_steps, "train_steps" }, { &k_beta_start, "beta_start" }, { &k_beta_end, "beta_end" }, { &k_steps, "steps" }, { &k_eta, "eta" },
        { &k_sampler, "sampler" }, { &k_shift, "shift" }, { &k_get, "get" }, { &k_is_cuda, "is_cuda" }, { &k_is_contiguous, "is_contiguous" },
        { &k_dtype, "dtype" }, { &k_data_ptr, "data_ptr" }, { &k_shape, "shape" } };
    for (auto& n : names)
        if (!(*n.at = PyUnicode_InternFromString(n.text))) return nullptr;
    if (!(k_zero = PyFloat_FromDouble(0.0)) || !(k_one = PyFloat_FromDouble(1.0)) || !(k_ddim = PyLong_FromLong(DRF_DDIM))) return nullptr;
    return PyModule_Create(&kModule);
}
