// Argument marshalling of the calls that a program makes once or more per step, for binding.py.
//
// The same checks in Python take five attribute calls per tensor and a ctypes conversion per argument: a call with four buffers and
// one launch was issued in 5.7 us, in 3.2 with this, where the kernels of a small step take 3 to 8.  A tensor that is not of torch's own classes
// or does not pass a check, and everything that is no tensor, goes to binding.py's own function, which converts it or raises.
// Measured on an MI355X machine: the two calls of a step of 256 tokens, 4 experts 14.2 -> 9.4 us, its first pass on new buffers 33.3 ->
// 25.6; a call whose kernel takes longer than this marshalling gains it only where the GPU is waited for.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include "monta.h"

namespace {

// from binding.py: the cfg class, _ptr, _stream, _current_raw_stream, _check; kept until the process ends
PyObject *g_cfg_type, *g_ptr, *g_stream, *g_current_stream, *g_check;
decltype(&monta_ws_layout_query) g_layout;
decltype(&monta_route) g_route;
decltype(&monta_route_dispatch_regather) g_route_dispatch_regather;
decltype(&monta_route_dispatch_combine_static) g_static;
decltype(&monta_combine) g_combine;
decltype(&monta_unregather_combine) g_unregather_combine;
decltype(&monta_gate) g_gate;
decltype(&monta_expert_linear) g_expert_linear;
decltype(&monta_route_dispatch_expert) g_route_dispatch_expert;

// One call: sizes from its cfg, then its arguments in order.  The first failure leaves a Python error and ends the rest.
struct Call {
    typedef __int128 Size;          // a cfg that nothing has validated yet may hold any numbers
    monta_cfg cfg;
    monta_ws_layout L;
    const char *what;
    bool ok = false;
    Size T, E, k, bpe, row;

    Call(const char *name, PyObject *const *args, Py_ssize_t n, Py_ssize_t want, bool layout) : what(name)
    {
        if (n != want) {
            PyErr_Format(PyExc_TypeError, "%s: expected %zd arguments, got %zd", name, want, n);
            return;
        }
        if (!PyObject_TypeCheck(args[0], reinterpret_cast<PyTypeObject *>(g_cfg_type))) {
            PyErr_Format(PyExc_TypeError, "%s: cfg is not a monta_cfg", name);
            return;
        }
        Py_buffer b;
        if (PyObject_GetBuffer(args[0], &b, PyBUF_SIMPLE)) return;
        ok = b.len >= (Py_ssize_t)sizeof(cfg);
        if (ok) memcpy(&cfg, b.buf, sizeof(cfg));
        PyBuffer_Release(&b);
        if (!ok) {
            PyErr_Format(PyExc_TypeError, "%s: cfg is too short", name);
            return;
        }
        if (layout)
            if (const int rc = g_layout(&cfg, &L)) {
                check(rc, "monta_ws_layout_query");
                ok = false;
                return;
            }
        T = cfg.tokens, E = cfg.experts, k = cfg.top_k, bpe = cfg.dtype == MONTA_FP32 ? 4 : 2, row = cfg.hidden * bpe;
    }

    static PyObject *check(int rc, const char *name) { return PyObject_CallFunction(g_check, "is", rc, name); }

    static void *address(PyObject *number)      // a new reference, or null after an error
    {
        if (!number) return nullptr;
        void *p = reinterpret_cast<void *>((uintptr_t)PyLong_AsUnsignedLongLongMask(number));
        Py_DECREF(number);
        return p;
    }

    // The address of a buffer of at least `need` bytes.
    template <typename V = void>
    V *ptr(PyObject *o, Size need, const char *name)
    {
        if (!ok) return nullptr;
        if (THPVariable_CheckTypeExact(Py_TYPE(o))) {
            try {
                const at::Tensor &t = THPVariable_Unpack(o);
                if (t.is_cuda() && t.is_contiguous() && (Size)t.numel() * t.element_size() >= need) return static_cast<V *>(t.data_ptr());
            } catch (...) {         // binding.py's function meets the same and raises it as Python does
            }
        }
        const Size most = INT64_MAX, least = INT64_MIN;
        const long long clamped = (long long)(need > most ? most : need < least ? least : need);
        void *p = address(PyObject_CallFunction(g_ptr, "OLs", o, clamped, name));
        if (PyErr_Occurred()) ok = false;
        return static_cast<V *>(p);
    }

    // an argument that binding.py has turned into a number; as ctypes does, its low 32 bits
    Size number(PyObject *o)
    {
        if (!ok) return 0;
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (PyErr_Occurred()) ok = false;
        return overflow > 0 ? (Size)INT64_MAX : overflow < 0 ? (Size)INT64_MIN : (Size)v;
    }
    static int low32(PyObject *o) { return (int)(uint32_t)PyLong_AsUnsignedLongLongMask(o); }

    void *stream(PyObject *o)
    {
        if (!ok) return nullptr;
        void *p = address(o == Py_None ? PyObject_CallNoArgs(g_current_stream) : PyObject_CallOneArg(g_stream, o));
        if (PyErr_Occurred()) ok = false;
        return p;
    }

    // f() without the interpreter's lock, as ctypes calls it
    template <typename F>
    PyObject *finish(F f)
    {
        if (!ok) return nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = f();
        Py_END_ALLOW_THREADS
        if (rc) return check(rc, what);
        Py_RETURN_NONE;
    }
};

PyObject *route(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_route", a, n, 6, true);
    if (!c.ok) return nullptr;
    const float *logits = c.ptr<float>(a[1], c.T * c.E * 4, "logits");
    int32_t *idx = c.ptr<int32_t>(a[2], c.T * c.k * 4, "topk_idx");
    float *gates = c.ptr<float>(a[3], c.T * c.k * 4, "gates");
    void *ws = c.ptr(a[4], c.L.ws_bytes, "ws"), *st = c.stream(a[5]);
    return c.finish([&] { return g_route(&c.cfg, logits, idx, gates, ws, st); });
}

PyObject *route_dispatch_regather(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_route_dispatch_regather", a, n, 9, true);
    if (!c.ok) return nullptr;
    const Call::Size rows = c.L.max_rows * c.row;
    const float *logits = c.ptr<float>(a[1], c.T * c.E * 4, "logits");
    const void *x = c.ptr(a[2], c.T * c.row, "x");
    int32_t *idx = c.ptr<int32_t>(a[3], c.T * c.k * 4, "topk_idx");
    float *gates = c.ptr<float>(a[4], c.T * c.k * 4, "gates");
    void *stage = c.ptr(a[5], rows, "stage"), *fin = c.ptr(a[6], rows, "final_"), *ws = c.ptr(a[7], c.L.ws_bytes, "ws"), *st = c.stream(a[8]);
    return c.finish([&] { return g_route_dispatch_regather(&c.cfg, logits, x, idx, gates, stage, fin, ws, st); });
}

PyObject *route_dispatch_combine_static(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_route_dispatch_combine_static", a, n, 9, true);
    if (!c.ok) return nullptr;
    const Call::Size rows = c.L.max_rows * c.row;
    const float *logits = c.ptr<float>(a[1], c.T * c.E * 4, "logits");
    const void *x = c.ptr(a[2], c.T * c.row, "x");
    int32_t *idx = c.ptr<int32_t>(a[3], c.T * c.k * 4, "topk_idx");
    float *gates = c.ptr<float>(a[4], c.T * c.k * 4, "gates");
    void *stage = c.ptr(a[5], rows, "stage"), *fin = c.ptr(a[6], rows, "final_"), *out = c.ptr(a[7], c.T * c.row, "out"), *st = c.stream(a[8]);
    return c.finish([&] { return g_static(&c.cfg, logits, x, idx, gates, stage, fin, out, st); });
}

PyObject *combine(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_combine", a, n, 6, true);
    if (!c.ok) return nullptr;
    const void *y = c.ptr(a[1], c.L.max_rows * c.row, "y");
    const float *gates = c.ptr<float>(a[2], c.T * c.k * 4, "gates");
    void *out = c.ptr(a[3], c.T * c.row, "out"), *ws = c.ptr(a[4], c.L.ws_bytes, "ws"), *st = c.stream(a[5]);
    return c.finish([&] { return g_combine(&c.cfg, y, gates, out, ws, st); });
}

PyObject *unregather_combine(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_unregather_combine", a, n, 7, true);
    if (!c.ok) return nullptr;
    const void *y = c.ptr(a[1], c.L.max_rows * c.row, "y");
    void *y_stage = c.ptr(a[2], c.L.max_rows * c.row, "y_stage");
    const float *gates = c.ptr<float>(a[3], c.T * c.k * 4, "gates");
    void *out = c.ptr(a[4], c.T * c.row, "out"), *ws = c.ptr(a[5], c.L.ws_bytes, "ws"), *st = c.stream(a[6]);
    return c.finish([&] { return g_unregather_combine(&c.cfg, y, y_stage, gates, out, ws, st); });
}

PyObject *gate(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_gate", a, n, 5, false);
    if (!c.ok) return nullptr;
    const void *x = c.ptr(a[1], c.T * c.row, "x"), *w = c.ptr(a[2], c.E * c.row, "w_gate");
    float *logits = c.ptr<float>(a[3], c.T * c.E * 4, "logits");
    void *st = c.stream(a[4]);
    return c.finish([&] { return g_gate(&c.cfg, x, w, logits, st); });
}

PyObject *expert_linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_expert_linear", a, n, 8, true);
    if (!c.ok) return nullptr;
    const Call::Size N = c.number(a[3]);
    const void *x = c.ptr(a[1], c.L.max_rows * c.row, "x_final"), *w = c.ptr(a[2], c.E * N * c.row, "w_exp");
    void *y = c.ptr(a[4], c.L.max_rows * N * c.bpe, "y"), *ws = c.ptr(a[5], c.L.ws_bytes, "ws"), *st = c.stream(a[7]);
    const int out_features = Call::low32(a[3]), slice = Call::low32(a[6]);
    return c.finish([&] { return g_expert_linear(&c.cfg, x, w, out_features, y, ws, slice, st); });
}

PyObject *route_dispatch_expert(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Call c("monta_route_dispatch_expert", a, n, 13, true);
    if (!c.ok) return nullptr;
    const Call::Size N = c.number(a[8]), rows = c.L.max_rows * c.row;
    const float *logits = c.ptr<float>(a[1], c.T * c.E * 4, "logits");
    const void *x = c.ptr(a[2], c.T * c.row, "x");
    int32_t *idx = c.ptr<int32_t>(a[3], c.T * c.k * 4, "topk_idx");
    float *gates = c.ptr<float>(a[4], c.T * c.k * 4, "gates");
    void *stage = c.ptr(a[5], rows, "stage"), *fin = c.ptr(a[6], rows, "final");
    const void *w = c.ptr(a[7], c.E * N * c.row, "w_exp");
    void *y = c.ptr(a[9], c.L.max_rows * N * c.bpe, "y"), *ws = c.ptr(a[10], c.L.ws_bytes, "ws"), *st = c.stream(a[12]);
    const int out_features = Call::low32(a[8]), overlap = Call::low32(a[11]);
    return c.finish([&] {
        return g_route_dispatch_expert(&c.cfg, logits, x, idx, gates, stage, fin, w, out_features, y, ws, overlap, st);
    });
}

// setup(cfg class, _ptr, _stream, _current_raw_stream, _check, address of each entry point in the order below)
PyObject *setup(PyObject *, PyObject *args)
{
    PyObject *cfg, *ptr, *stream, *current, *check;
    unsigned long long f[9];
    if (!PyArg_ParseTuple(args, "OOOOO(KKKKKKKKK)", &cfg, &ptr, &stream, &current, &check, f, f + 1, f + 2, f + 3, f + 4, f + 5, f + 6, f + 7,
                          f + 8))
        return nullptr;
    if (!PyType_Check(cfg)) {
        PyErr_SetString(PyExc_TypeError, "setup: the first argument is not a class");
        return nullptr;
    }
    for (PyObject *o : {cfg, ptr, stream, current, check}) Py_INCREF(o);
    g_cfg_type = cfg, g_ptr = ptr, g_stream = stream, g_current_stream = current, g_check = check;
    auto set = [](auto &fn, unsigned long long at) { fn = reinterpret_cast<std::decay_t<decltype(fn)>>((uintptr_t)at); };
    set(g_layout, f[0]);
    set(g_route, f[1]);
    set(g_route_dispatch_regather, f[2]);
    set(g_static, f[3]);
    set(g_combine, f[4]);
    set(g_unregather_combine, f[5]);
    set(g_gate, f[6]);
    set(g_expert_linear, f[7]);
    set(g_route_dispatch_expert, f[8]);
    Py_RETURN_NONE;
}

#define MONTA_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    {"setup", setup, METH_VARARGS, nullptr}, MONTA_FAST(route), MONTA_FAST(route_dispatch_regather), MONTA_FAST(route_dispatch_combine_static),
    MONTA_FAST(combine), MONTA_FAST(unregather_combine), MONTA_FAST(gate), MONTA_FAST(expert_linear), MONTA_FAST(route_dispatch_expert),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&g_module); }
