// The calls of a decode step from Python: arguments from Python objects straight into the C ABI of include/iflow.h.
//
// These kernels take a few microseconds each, as long as it takes to call them: through ctypes a product costs 1.5 us of marshalling and the
// three-matrix call of a decoder layer 4, next to the 2.3 or more of the launch itself.  Here an address is one method call (data_ptr) and an array lives
// on the stack.  Measured, us to enqueue, ctypes -> here: a product with one vector 5.2 -> 4.6, a decoder layer's six calls 43 -> 32.
// The functions are the library's own, bound by address (bind), so the library is loaded once and in one place.  An address is an integer, None
// (null) or an object with data_ptr(), a number what has __index__ or __float__, matrices and outputs are lists or tuples; a call returns the library's
// status and runs without the interpreter's lock, as a ctypes call does.  A call with anything else among its arguments (ctypes' own numbers, an iterator,
// a text) is handed on as it is to the function that otherwise() was given, which takes or refuses it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/iflow.h"

namespace {

constexpr Py_ssize_t MAX_ARRAY = 16;                           // matrices of one call that are handed on (the library takes 8 and refuses more by their count)

decltype(&iflow_quantize) p_quantize;
decltype(&iflow_dequant) p_dequant;
decltype(&iflow_qgemv) p_qgemv;
decltype(&iflow_qgemm) p_qgemm;
decltype(&iflow_qgemv_fused) p_qgemv_fused;
decltype(&iflow_qgemv_gated) p_qgemv_gated;
decltype(&iflow_qgemm_fused) p_qgemm_fused;
decltype(&iflow_attn_decode) p_attn_decode;
decltype(&iflow_rope_append) p_rope_append;
PyObject *s_data_ptr, *general;                                // general(name, arguments ...): the call that takes every form of argument

// One call's arguments in order; the first that does not fit ends the reading (bad; perhaps a Python exception) and turns the rest into zeros.
struct Args {
    const char *name;
    PyObject *const *first, *const *at;
    Py_ssize_t count;
    bool bad = false;
    Args(const char *call, PyObject *const *args, Py_ssize_t nargs, Py_ssize_t want) : name(call), first(args), at(args), count(nargs) { bad = nargs != want; }
    PyObject *next() { return bad ? nullptr : *at++; }
    static bool address(PyObject *o, void **out)
    {
        if (o == Py_None) { *out = nullptr; return true; }
        PyObject *v = PyLong_Check(o) ? Py_NewRef(o) : PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (!v) return false;
        const bool number = PyLong_Check(v);
        if (number) *out = reinterpret_cast<void *>(PyLong_AsUnsignedLongLongMask(v));
        Py_DECREF(v);
        return number;
    }
    template <typename T> T *ptr()
    {
        PyObject *o = next();
        void *p = nullptr;
        if (o && !address(o, &p)) bad = true;
        return static_cast<T *>(p);
    }
    // a stream's handle: a number already
    void *handle()
    {
        PyObject *o = next();
        void *p = nullptr;
        if (o && !((o == Py_None || PyLong_Check(o)) && address(o, &p))) bad = true;
        return p;
    }
    // whole numbers as ctypes takes them: what has __index__, its low bits (a capacity of 2^64 - 1 is one)
    static bool whole(PyObject *o, int64_t *out)
    {
        PyObject *v = PyNumber_Index(o);
        if (!v) return false;
        *out = (int64_t)PyLong_AsUnsignedLongLongMask(v);
        Py_DECREF(v);
        return true;
    }
    int64_t num()
    {
        PyObject *o = next();
        int64_t v = 0;
        if (o && !whole(o, &v)) bad = true;
        return v;
    }
    int word() { return (int)num(); }
    float real()
    {
        PyObject *o = next();
        if (!o) return 0.f;
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) bad = true;
        return (float)v;
    }
    // a list of addresses or of whole numbers, its first MAX_ARRAY entries; its length, or -1 for None
    template <typename Put> Py_ssize_t each(Put put)
    {
        PyObject *o = next();
        if (!o || o == Py_None) return -1;
        PyObject *seq = PyList_Check(o) || PyTuple_Check(o) ? PySequence_Tuple(o) : nullptr;      // (a copy that holds its entries: data_ptr or another thread may change the list meanwhile)
        if (!seq) { bad = true; return -1; }
        const Py_ssize_t n = PyTuple_GET_SIZE(seq);
        for (Py_ssize_t i = 0; i < n && i < MAX_ARRAY && !bad; ++i)
            if (!put(i, PyTuple_GET_ITEM(seq, i))) bad = true;
        Py_DECREF(seq);
        return n;
    }
    template <typename T> Py_ssize_t addresses(T **out)
    {
        return each([&](Py_ssize_t i, PyObject *o) {
            void *p = nullptr;
            const bool ok = address(o, &p);
            out[i] = static_cast<T *>(p);
            return ok;
        });
    }
    Py_ssize_t numbers(int64_t *out)
    {
        return each([&](Py_ssize_t i, PyObject *o) {
            PyObject *v = PyNumber_Long(o);                    // int(o)
            if (!v) return false;
            const bool ok = whole(v, &out[i]);
            Py_DECREF(v);
            return ok;
        });
    }
};

// A call whose arguments do not fit here, as it came: what data_ptr, __index__ or __float__ raised is raised again there, or not.  (An interrupt goes up.)
PyObject *hand_on(const Args &a)
{
    if (PyErr_Occurred()) {
        if (!PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;
        PyErr_Clear();
    }
    if (!general) { PyErr_SetString(PyExc_RuntimeError, "not bound"); return nullptr; }
    PyObject *args = PyTuple_New(a.count + 1), *name = PyUnicode_FromString(a.name), *result = nullptr;
    if (args && name) {
        PyTuple_SET_ITEM(args, 0, Py_NewRef(name));
        for (Py_ssize_t i = 0; i < a.count; ++i) PyTuple_SET_ITEM(args, i + 1, Py_NewRef(a.first[i]));
        result = PyObject_Call(general, args, nullptr);
    }
    Py_XDECREF(args);
    Py_XDECREF(name);
    return result;
}

template <typename Call> PyObject *run(const Args &a, Call call)
{
    if (a.bad) return hand_on(a);
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = (int)call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

PyObject *quantize(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("quantize", args, nargs, 7);
    const int fmt = a.word();
    const float *w = a.ptr<const float>();
    const int64_t rows = a.num(), cols = a.num();
    void *packed = a.ptr<void>();
    const int64_t capacity = a.num();
    void *stream = a.handle();
    return run(a, [&] { return p_quantize((iflow_format_t)fmt, w, rows, cols, packed, (size_t)capacity, stream); });
}

PyObject *dequant(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("dequant", args, nargs, 6);
    const int fmt = a.word();
    const void *packed = a.ptr<const void>();
    const int64_t rows = a.num(), cols = a.num();
    uint16_t *w16 = a.ptr<uint16_t>();
    void *stream = a.handle();
    return run(a, [&] { return p_dequant((iflow_format_t)fmt, packed, rows, cols, w16, stream); });
}

PyObject *qgemv(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("qgemv", args, nargs, 7);
    const int fmt = a.word();
    const void *packed = a.ptr<const void>();
    const int64_t rows = a.num(), cols = a.num();
    const uint16_t *x = a.ptr<const uint16_t>();
    uint16_t *y = a.ptr<uint16_t>();
    void *stream = a.handle();
    return run(a, [&] { return p_qgemv((iflow_format_t)fmt, packed, rows, cols, x, y, stream); });
}

PyObject *qgemm(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("qgemm", args, nargs, 8);
    const int fmt = a.word();
    const void *packed = a.ptr<const void>();
    const int64_t rows = a.num(), cols = a.num();
    const uint16_t *x = a.ptr<const uint16_t>();
    const int64_t batch = a.num();
    uint16_t *y = a.ptr<uint16_t>();
    void *stream = a.handle();
    return run(a, [&] { return p_qgemm((iflow_format_t)fmt, packed, rows, cols, x, batch, y, stream); });
}

PyObject *qgemv_fused(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("qgemv_fused", args, nargs, 11);
    const int fmt = a.word();
    // (what a shorter list leaves out is null or zero: no residual, or refused by the library)
    const void *packed[MAX_ARRAY] = {};
    int64_t rows[MAX_ARRAY] = {};
    uint16_t *y[MAX_ARRAY] = {};
    const uint16_t *residual[MAX_ARRAY] = {};
    const Py_ssize_t n = a.addresses(packed), nr = a.numbers(rows);
    const int64_t cols = a.num();
    const uint16_t *x = a.ptr<const uint16_t>();
    const Py_ssize_t ny = a.addresses(y);
    const int x_op = a.word();
    const uint16_t *aux = a.ptr<const uint16_t>();
    const float eps = a.real();
    const Py_ssize_t nres = a.addresses(residual);
    void *stream = a.handle();
    if (n < 0 || nr < 0 || ny < 0 || nr > n || ny > n || nres > n) a.bad = true;
    return run(a, [&] {
        return p_qgemv_fused((iflow_format_t)fmt, (int)n, packed, rows, cols, x, (iflow_x_op_t)x_op, aux, eps, nres < 0 ? nullptr : residual, y, stream);
    });
}

PyObject *qgemv_gated(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("qgemv_gated", args, nargs, 11);
    const int fmt = a.word();
    const void *gate = a.ptr<const void>(), *up = a.ptr<const void>();
    const int64_t rows = a.num(), cols = a.num();
    const uint16_t *x = a.ptr<const uint16_t>();
    uint16_t *y = a.ptr<uint16_t>();
    const int x_op = a.word();
    const uint16_t *aux = a.ptr<const uint16_t>();
    const float eps = a.real();
    void *stream = a.handle();
    return run(a, [&] { return p_qgemv_gated((iflow_format_t)fmt, gate, up, rows, cols, x, (iflow_x_op_t)x_op, aux, eps, y, stream); });
}

PyObject *qgemm_fused(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("qgemm_fused", args, nargs, 12);
    const int fmt = a.word();
    const void *packed = a.ptr<const void>();
    const int64_t rows = a.num(), cols = a.num();
    const uint16_t *x = a.ptr<const uint16_t>();
    const int64_t batch = a.num();
    uint16_t *y = a.ptr<uint16_t>();
    const int x_op = a.word();
    const uint16_t *aux = a.ptr<const uint16_t>();
    const float eps = a.real();
    const uint16_t *residual = a.ptr<const uint16_t>();
    void *stream = a.handle();
    return run(a, [&] { return p_qgemm_fused((iflow_format_t)fmt, packed, rows, cols, x, batch, (iflow_x_op_t)x_op, aux, eps, residual, y, stream); });
}

PyObject *attn_decode(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("attn_decode", args, nargs, 13);
    const uint16_t *q = a.ptr<const uint16_t>(), *k = a.ptr<const uint16_t>(), *v = a.ptr<const uint16_t>();
    const int heads = a.word(), kv_heads = a.word(), head_dim = a.word();
    const int64_t seq_len = a.num(), max_seq = a.num();
    const float scale = a.real();
    uint16_t *out = a.ptr<uint16_t>();
    void *workspace = a.ptr<void>();
    const int64_t bytes = a.num();
    void *stream = a.handle();
    return run(a, [&] { return p_attn_decode(q, k, v, heads, kv_heads, head_dim, seq_len, max_seq, scale, out, workspace, (size_t)bytes, stream); });
}

PyObject *rope_append(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("rope_append", args, nargs, 13);
    uint16_t *q = a.ptr<uint16_t>();
    const uint16_t *k = a.ptr<const uint16_t>(), *v = a.ptr<const uint16_t>();
    const int heads = a.word(), kv_heads = a.word(), head_dim = a.word();
    const int64_t position = a.num(), max_seq = a.num();
    const float base = a.real();
    const int pairing = a.word();
    uint16_t *k_cache = a.ptr<uint16_t>(), *v_cache = a.ptr<uint16_t>();
    void *stream = a.handle();
    return run(a, [&] {
        return p_rope_append(q, k, v, heads, kv_heads, head_dim, position, max_seq, base, (iflow_rope_pairing_t)pairing, k_cache, v_cache, stream);
    });
}

// bind(addresses of the nine functions, in this order)
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a("bind", args, nargs, 9);
    void *f[9];
    for (void *&p : f) p = a.handle();
    if (a.bad) { PyErr_SetString(PyExc_TypeError, "nine addresses are wanted"); return nullptr; }
    p_quantize = reinterpret_cast<decltype(p_quantize)>(f[0]);
    p_dequant = reinterpret_cast<decltype(p_dequant)>(f[1]);
    p_qgemv = reinterpret_cast<decltype(p_qgemv)>(f[2]);
    p_qgemm = reinterpret_cast<decltype(p_qgemm)>(f[3]);
    p_qgemv_fused = reinterpret_cast<decltype(p_qgemv_fused)>(f[4]);
    p_qgemv_gated = reinterpret_cast<decltype(p_qgemv_gated)>(f[5]);
    p_qgemm_fused = reinterpret_cast<decltype(p_qgemm_fused)>(f[6]);
    p_attn_decode = reinterpret_cast<decltype(p_attn_decode)>(f[7]);
    p_rope_append = reinterpret_cast<decltype(p_rope_append)>(f[8]);
    Py_RETURN_NONE;
}

// otherwise(function): what general is
PyObject *otherwise(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 1) { PyErr_SetString(PyExc_TypeError, "a function is wanted"); return nullptr; }
    PyObject *was = general;
    general = Py_NewRef(args[0]);
    Py_XDECREF(was);
    Py_RETURN_NONE;
}

#define IFLOW_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {IFLOW_METHOD(bind), IFLOW_METHOD(otherwise), IFLOW_METHOD(quantize), IFLOW_METHOD(dequant), IFLOW_METHOD(qgemv), IFLOW_METHOD(qgemm),
                         IFLOW_METHOD(qgemv_fused), IFLOW_METHOD(qgemv_gated), IFLOW_METHOD(qgemm_fused), IFLOW_METHOD(attn_decode),
                         IFLOW_METHOD(rope_append), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    return s_data_ptr ? PyModule_Create(&module) : nullptr;
}
