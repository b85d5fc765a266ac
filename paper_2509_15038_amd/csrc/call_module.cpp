// CPython module: the argument marshalling of the entry points that a program calls over and over (binding.py).  What it does is
// what ctypes did from Python: tensors to addresses, the current stream where none is given, checks of the host arrays.
// A call of one kernel on a few tokens takes the GPU 3 us and the launch itself 3.5 us of the host's time; marshalling from
// Python added 1.9 us to that, this adds 0.8 (one token for 256 heads, a call among others: 5.4 -> 4.3 us).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>

#include "curdkv.h"

namespace {

// set by bind(): the library's entry points, and Python callables for what is not worth writing out here
struct Bound {
    decltype(&curdkv_scores) scores;
    decltype(&curdkv_scores_append) scores_append;
    decltype(&curdkv_normalise) normalise;
    decltype(&curdkv_select) select;
    decltype(&curdkv_compact) compact;
    decltype(&curdkv_compress) compress;
    decltype(&curdkv_compress_adaptive) compress_adaptive;
} lib;
PyObject *slow_address, *slow_stream, *name_data_ptr;

// A value, or an error that has been set (`ok` false): one per call, passed along.
struct Args {
    PyObject* const* v;
    bool ok = true;

    // int(x) as a 64-bit value, wrapped as ctypes wraps it
    int64_t integer(int i) {
        if (!ok) return 0;
        PyObject* x = v[i];
        if (PyLong_CheckExact(x)) return wrapped(x);
        x = PyNumber_Long(x);
        if (!x) { ok = false; return 0; }
        const int64_t r = wrapped(x);
        Py_DECREF(x);
        return r;
    }
    double real(int i) {
        if (!ok) return 0.0;
        PyObject* x = PyNumber_Float(v[i]);
        if (!x) { ok = false; return 0.0; }
        const double r = PyFloat_AS_DOUBLE(x);
        Py_DECREF(x);
        return r;
    }
    // a tensor's data_ptr(), an integer as it is, None as NULL; anything else is left to Python
    void* address(int i) {
        if (!ok || v[i] == Py_None) return nullptr;
        if (PyLong_CheckExact(v[i])) return reinterpret_cast<void*>(wrapped(v[i]));
        PyObject* x = PyObject_CallMethodNoArgs(v[i], name_data_ptr);
        if (!x && PyErr_ExceptionMatches(PyExc_AttributeError)) {
            PyErr_Clear();
            x = PyObject_CallOneArg(slow_address, v[i]);
        }
        return taken(x);
    }
    // None: torch's current stream
    void* stream(int i) {
        if (!ok) return nullptr;
        if (PyLong_CheckExact(v[i])) return reinterpret_cast<void*>(wrapped(v[i]));
        return taken(PyObject_CallOneArg(slow_stream, v[i]));
    }
    // a host array of `count` integers of `width` bytes, one after the other (at any address: a view into a file or a
    // record need not be aligned, which numpy's format says with a '=')
    const void* array(int i, Py_ssize_t count, int width) {
        if (!ok) return nullptr;
        Py_buffer b;
        if (PyObject_GetBuffer(v[i], &b, PyBUF_STRIDES | PyBUF_FORMAT) != 0) { ok = false; return nullptr; }
        const void* p = b.buf;
        const char* f = b.format ? b.format : "";
        if (*f == '=' || *f == '@') ++f;
        const bool type = width == 4 ? !std::strcmp(f, "i") : !std::strcmp(f, "l") || !std::strcmp(f, "q");
        const bool fits = type && b.itemsize == width && b.len == count * width && PyBuffer_IsContiguous(&b, 'C');
        PyBuffer_Release(&b);                      // (the caller's reference keeps it during the call)
        if (!fits) {
            PyErr_Format(PyExc_AssertionError, "expected a contiguous array of %zd int%d", count, 8 * width);
            ok = false;
        }
        return p;
    }

  private:
    int64_t wrapped(PyObject* x) {
        const unsigned long long r = PyLong_AsUnsignedLongLongMask(x);
        if (r == (unsigned long long)-1 && PyErr_Occurred()) ok = false;
        return (int64_t)r;
    }
    void* taken(PyObject* x) {
        if (!x) { ok = false; return nullptr; }
        void* r = reinterpret_cast<void*>(wrapped(x));
        Py_DECREF(x);
        return r;
    }
};

bool counted(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return false;
}

template <class F>
PyObject* run(const Args& a, F f) {
    if (!a.ok) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

curdkv_ctx* context(Args& a) { return static_cast<curdkv_ctx*>(a.address(0)); }

PyObject* scores(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 6)) return nullptr;
    Args a{v};
    curdkv_ctx* c = context(a);
    void *K = a.address(1), *V = a.address(2), *out = a.address(4), *st = a.stream(5);
    const int64_t tokens = a.integer(3);
    return run(a, [&] { return lib.scores(c, K, V, tokens, (float*)out, st); });
}

PyObject* scores_append(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 9)) return nullptr;
    Args a{v};
    curdkv_ctx* c = context(a);
    void *K = a.address(1), *V = a.address(2), *raw = a.address(6), *sums = a.address(7), *st = a.stream(8);
    const int64_t m = a.integer(3), n_old = a.integer(4), stride = a.integer(5);
    return run(a, [&] { return lib.scores_append(c, K, V, m, n_old, stride, (float*)raw, (double*)sums, st); });
}

PyObject* normalise(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 7)) return nullptr;
    Args a{v};
    curdkv_ctx* c = context(a);
    void *raw = a.address(1), *sums = a.address(2), *out = a.address(5), *st = a.stream(6);
    const int64_t stride = a.integer(3), tokens = a.integer(4);
    return run(a, [&] { return lib.normalise(c, (const float*)raw, (const double*)sums, stride, tokens, (float*)out, st); });
}

// (the last argument of the next three: the context's number of (layer, head) pairs)
PyObject* select(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 9)) return nullptr;
    Args a{v};
    curdkv_ctx* c = context(a);
    const Py_ssize_t heads = (Py_ssize_t)a.integer(8);
    const auto* budgets = (const int32_t*)a.array(3, heads, 4);
    const auto* offsets = (const int64_t*)a.array(5, heads + 1, 8);
    void *sc = a.address(1), *indices = a.address(6), *st = a.stream(7);
    const int64_t tokens = a.integer(2), sinks = a.integer(4);
    return run(a, [&] { return lib.select(c, (const float*)sc, tokens, budgets, (int32_t)sinks, offsets, (int32_t*)indices, st); });
}

PyObject* compact(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 10)) return nullptr;
    Args a{v};
    curdkv_ctx* c = context(a);
    const auto* offsets = (const int64_t*)a.array(5, (Py_ssize_t)a.integer(9) + 1, 8);
    void *K = a.address(1), *V = a.address(2), *indices = a.address(4), *Ko = a.address(6), *Vo = a.address(7), *st = a.stream(8);
    const int64_t tokens = a.integer(3);
    return run(a, [&] { return lib.compact(c, K, V, tokens, (const int32_t*)indices, offsets, Ko, Vo, st); });
}

PyObject* compress(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 13)) return nullptr;
    Args a{v};
    curdkv_ctx* c = context(a);
    const Py_ssize_t heads = (Py_ssize_t)a.integer(12);
    const auto* budgets = (const int32_t*)a.array(4, heads, 4);
    const auto* offsets = (const int64_t*)a.array(6, heads + 1, 8);
    void *K = a.address(1), *V = a.address(2), *sc = a.address(7), *indices = a.address(8), *Ko = a.address(9), *Vo = a.address(10), *st = a.stream(11);
    const int64_t tokens = a.integer(3), sinks = a.integer(5);
    return run(a, [&] { return lib.compress(c, K, V, tokens, budgets, (int32_t)sinks, offsets, (float*)sc, (int32_t*)indices, Ko, Vo, st); });
}

PyObject* compress_adaptive(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 14)) return nullptr;
    Args a{v};
    curdkv_ctx* c = context(a);
    void *K = a.address(1), *V = a.address(2), *sc = a.address(7), *budgets = a.address(8), *offsets = a.address(9), *indices = a.address(10);
    void *Ko = a.address(11), *Vo = a.address(12), *st = a.stream(13);
    const int64_t tokens = a.integer(3), budget = a.integer(4), sinks = a.integer(5);
    const double alpha = a.real(6);
    return run(a, [&] {
        return lib.compress_adaptive(c, K, V, tokens, (int32_t)budget, (int32_t)sinks, alpha, (float*)sc, (int32_t*)budgets, (int64_t*)offsets,
                                     (int32_t*)indices, Ko, Vo, st);
    });
}

// bind(addresses of the seven entry points in the order of Bound, address(object) -> int, stream(object) -> int)
PyObject* bind(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (!counted(n, 9)) return nullptr;
    Args a{v};
    void* p[7];
    for (int i = 0; i < 7; ++i) p[i] = a.address(i);
    if (!a.ok) return nullptr;
    lib.scores = reinterpret_cast<decltype(lib.scores)>(p[0]);
    lib.scores_append = reinterpret_cast<decltype(lib.scores_append)>(p[1]);
    lib.normalise = reinterpret_cast<decltype(lib.normalise)>(p[2]);
    lib.select = reinterpret_cast<decltype(lib.select)>(p[3]);
    lib.compact = reinterpret_cast<decltype(lib.compact)>(p[4]);
    lib.compress = reinterpret_cast<decltype(lib.compress)>(p[5]);
    lib.compress_adaptive = reinterpret_cast<decltype(lib.compress_adaptive)>(p[6]);
    Py_INCREF(v[7]);
    Py_XSETREF(slow_address, v[7]);
    Py_INCREF(v[8]);
    Py_XSETREF(slow_stream, v[8]);
    Py_RETURN_NONE;
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(bind), ENTRY(scores), ENTRY(scores_append), ENTRY(normalise), ENTRY(select),
                         ENTRY(compact), ENTRY(compress), ENTRY(compress_adaptive), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) {
    name_data_ptr = PyUnicode_InternFromString("data_ptr");
    return name_data_ptr ? PyModule_Create(&module) : nullptr;
}
