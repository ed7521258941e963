// The hot entry points as one native call from Python (module _native): the checks of binding.py on torch's own tensors, the
// current stream, and the C entry point, whose address binding.py hands over.
//
// A decode step is a launch of 2.7 us, and the same in Python and ctypes took 4.9 us: fifteen attribute and method calls on
// tensors, one on the stream, the conversion of nine arguments.  Here they are some dozens of loads (3.0 us with the launch).
//
// Each function returns the status of the entry point, or None for what it does not take: a stream that was named, objects
// that are not exactly what is usual (a tensor subclass, a numpy integer), and everything that is to be refused.  binding.py
// then goes its general way, which knows all cases and has the words.
//
// torch's objects are read where the headers of the build say, so the module names the torch it was built for, and binding.py
// does without it where that is another one.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using RunFn = int (*)(void*, void*, const void*, float, int64_t, int64_t, int, const void*, void*);
using SiluFn = int (*)(const void*, void*, int64_t, int64_t, int, const void*, void*);
using MergeFn = int (*)(const void*, const float*, const void*, const float*, void*, float*, int64_t, int64_t, int, const void*, void*);
using GateFn = int (*)(const void*, const void*, const void*, const void*, int64_t, int, uint32_t, void*, void*);

RunFn g_run;
SiluFn g_silu;
MergeFn g_merge;
GateFn g_gate;
PyObject* g_formats;                                         // dict: name of a storage format -> its number
PyTypeObject* g_cfg;                                         // binding.Cfg

constexpr at::ScalarType kX[] = {at::kBFloat16, at::kHalf, at::kHalf, at::kFloat};
constexpr at::ScalarType kR[] = {at::kBFloat16, at::kHalf, at::kFloat, at::kFloat};

bool whole(PyObject* o, int64_t* out)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *out = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0;
}
bool format(PyObject* o, int* out)
{
    int64_t v = -1;
    if (PyUnicode_CheckExact(o)) o = PyDict_GetItem(g_formats, o);               // borrowed; no error is raised
    if (!o || !whole(o, &v) || v < 0 || v > 3) return false;
    *out = static_cast<int>(v);
    return true;
}
// A configuration's eight integers, from where ctypes keeps them; NULL for None.
bool configuration(PyObject* o, const void** out)
{
    *out = nullptr;
    if (o == Py_None) return true;
    if (Py_TYPE(o) != g_cfg) return false;
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return false; }
    *out = b.buf;                                            // lives as long as the object, which the caller holds
    PyBuffer_Release(&b);
    return true;
}
// The tensor's data, if it has `numel` contiguous elements of `type` on the device.
bool data(PyObject* o, at::ScalarType type, int64_t numel, void** out)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || t.numel() != numel || !t.is_contiguous()) return false;
    *out = t.data_ptr();
    return true;
}
void* stream_of(PyObject* tensor)
{
    return c10::hip::getCurrentHIPStream(THPVariable_Unpack(tensor).get_device()).stream();
}
PyObject* general() { Py_RETURN_NONE; }

// Runs `call` without the interpreter's lock: a launch waits where the stream's queue is full.
template <class Call>
PyObject* status(Call call)
{
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}
// What torch throws (a tensor without storage, a symbolic size) goes the general way, too.
template <class Body>
PyObject* guarded(Body body)
{
    try {
        return body();
    } catch (...) {
        PyErr_Clear();
        return general();
    }
}

// (x, residual, weight, eps, M, N, dtype, cfg)
PyObject* addrms_run(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int dt;
        int64_t M, N, all;
        void *x, *r, *w;
        const void* cfg;
        if (n != 8 || !g_run || !PyFloat_CheckExact(a[3]) || !whole(a[4], &M) || !whole(a[5], &N) || !format(a[6], &dt) ||
            !configuration(a[7], &cfg) || __builtin_mul_overflow(M, N, &all) || !data(a[0], kX[dt], all, &x) ||
            !data(a[1], kR[dt], all, &r) || !data(a[2], kX[dt], N, &w))
            return general();
        const float eps = static_cast<float>(PyFloat_AS_DOUBLE(a[3]));
        void* s = stream_of(a[0]);
        return status([=] { return g_run(x, r, w, eps, M, N, dt, cfg, s); });
    });
}
// (x, out, M, d, dtype, cfg)
PyObject* silumul_run(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int dt;
        int64_t M, d, all, twice;
        void *x, *out;
        const void* cfg;
        if (n != 6 || !g_silu || !whole(a[2], &M) || !whole(a[3], &d) || !format(a[4], &dt) || !configuration(a[5], &cfg) ||
            __builtin_mul_overflow(M, d, &all) || __builtin_add_overflow(all, all, &twice) || !data(a[0], kX[dt], twice, &x) ||
            !data(a[1], kX[dt], all, &out))
            return general();
        void* s = stream_of(a[0]);
        return status([=] { return g_silu(x, out, M, d, dt, cfg, s); });
    });
}
// (v_a, s_a, v_b, s_b, v_out, s_out, rows, d, dtype, cfg)
PyObject* mergestates_run(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int dt;
        int64_t rows, d, all;
        void* p[6];
        const void* cfg;
        if (n != 10 || !g_merge || !whole(a[6], &rows) || !whole(a[7], &d) || !format(a[8], &dt) || !configuration(a[9], &cfg) ||
            __builtin_mul_overflow(rows, d, &all))
            return general();
        for (int i = 0; i < 6; ++i)
            if (!(i % 2 ? data(a[i], at::kFloat, rows, &p[i]) : data(a[i], kX[dt], all, &p[i]))) return general();
        void* s = stream_of(a[0]);
        return status([=] {
            return g_merge(p[0], static_cast<float*>(p[1]), p[2], static_cast<float*>(p[3]), p[4], static_cast<float*>(p[5]), rows, d,
                           dt, cfg, s);
        });
    });
}
// (y, y_ref, residual, residual_ref, dtype, tol, counts_out)
PyObject* gate_probe_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        int dt;
        int64_t tol;
        void* p[4];
        if (n != 7 || !g_gate || !format(a[4], &dt) || !whole(a[5], &tol) || tol < 0 || tol > UINT32_MAX || !THPVariable_CheckExact(a[0]) ||
            !THPVariable_CheckExact(a[6]))
            return general();
        const int64_t all = THPVariable_Unpack(a[0]).numel();
        for (int i = 0; i < 4; ++i)
            if (!data(a[i], i < 2 ? kX[dt] : kR[dt], all, &p[i])) return general();
        const at::Tensor& counts = THPVariable_Unpack(a[6]);
        if (!counts.is_cuda() || counts.numel() * static_cast<int64_t>(counts.element_size()) < 16) return general();
        void *out = counts.data_ptr(), *s = stream_of(a[0]);
        return status([=] { return g_gate(p[0], p[1], p[2], p[3], all, dt, static_cast<uint32_t>(tol), out, s); });
    });
}

// (formats, Cfg, addresses of addrms_run, silumul_run, mergestates_run and addrms_gate_probe_noalloc)
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject *formats, *cfg;
    unsigned long long run, silu, merge, gate;
    if (!PyArg_ParseTuple(args, "O!O!KKKK", &PyDict_Type, &formats, &PyType_Type, &cfg, &run, &silu, &merge, &gate)) return nullptr;
    Py_INCREF(formats);
    Py_XSETREF(g_formats, formats);
    Py_INCREF(cfg);
    PyTypeObject* old = g_cfg;
    g_cfg = reinterpret_cast<PyTypeObject*>(cfg);
    Py_XDECREF(old);
    g_run = reinterpret_cast<RunFn>(static_cast<uintptr_t>(run));
    g_silu = reinterpret_cast<SiluFn>(static_cast<uintptr_t>(silu));
    g_merge = reinterpret_cast<MergeFn>(static_cast<uintptr_t>(merge));
    g_gate = reinterpret_cast<GateFn>(static_cast<uintptr_t>(gate));
    Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef g_methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                           {"addrms_run", FAST(addrms_run), nullptr},
                           {"silumul_run", FAST(silumul_run), nullptr},
                           {"mergestates_run", FAST(mergestates_run), nullptr},
                           {"addrms_gate_probe_noalloc", FAST(gate_probe_noalloc), nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native()
{
    PyObject* m = PyModule_Create(&g_module);
    if (m && PyModule_AddStringConstant(m, "TORCH", TORCH_IDENTITY) != 0) Py_CLEAR(m);
    return m;
}
