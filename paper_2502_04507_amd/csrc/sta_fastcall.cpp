// CPython extension: the hot entry points called with ordinary arguments (dense device tensors of the expected types, tuples or
// lists of plain integers, the current stream) without ctypes and without a Python object per argument.
//
// Every function returns the library's status, or None where an argument is anything else; the caller then takes the general
// path, which accepts what it always accepted and raises what it always raised.  Nothing is launched before every argument has
// been looked at.
//
// What bounds a small layer is the host: five launches of 2.4 us each and, through ctypes, as much again in Python.  us per call,
// host alone, ctypes against this: sta_tile_permute 5.3, 3.05; sta_forward of 2 heads 7.5, 3.5, of 24 11.4, 3.9.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using PermuteFn = int (*)(const void *, void *, int, int, int, int, int, const int *, const int *, void *);
using ForwardFn = int (*)(const void *, const void *, const void *, void *, int, int, int, const int *, const int *, const int *,
                          float, void *, size_t, void *);
using ForwardLseFn = int (*)(const void *, const void *, const void *, void *, float *, int, int, int, const int *, const int *,
                             const int *, float, void *);
using BackwardFn = int (*)(const void *, const void *, const void *, const void *, const void *, const float *, void *, void *,
                           void *, int, int, int, const int *, const int *, const int *, float, void *, size_t, void *);

struct Entries {
    PermuteFn tile_permute, untile;
    ForwardFn forward;
    ForwardLseFn forward_lse;
    BackwardFn backward;
} entries = {};
PyObject *current_device, *current_raw_stream;      // torch's own, called for every launch

constexpr int kMaxHeads = 1024;                     // more go the general way
enum { kBf16 = 0, kF32 = 1 };                       // STA_BF16, STA_F32

// A dense device tensor as the kernels take it.
struct View {
    const at::Tensor *t;
    void *ptr;
};
bool dense(PyObject *o, View &v)
{
    if (!THPVariable_CheckExact(o)) return false;
    v.t = &THPVariable_Unpack(o);
    if (!v.t->is_cuda() || !v.t->is_contiguous() || v.t->layout() != at::kStrided) return false;
    v.ptr = v.t->data_ptr();                        // throws for tensors without storage
    return true;
}
bool same_shape4(const View *v, int n)
{
    const auto shape = v[0].t->sizes();
    if (shape.size() != 4) return false;
    for (int i = 0; i < 4; ++i)
        if (shape[i] > INT32_MAX) return false;
    for (int i = 1; i < n; ++i)
        if (v[i].t->sizes() != shape) return false;
    return true;
}
bool all_bf16(const View *v, int n)
{
    for (int i = 0; i < n; ++i)
        if (v[i].t->scalar_type() != at::kBFloat16) return false;
    return true;
}
bool dtype_code(const View &v, int &code)
{
    const auto type = v.t->scalar_type();
    code = type == at::kBFloat16 ? kBf16 : kF32;
    return type == at::kBFloat16 || type == at::kFloat;
}

// n plain integers from a tuple or a list.
bool ints(PyObject *o, Py_ssize_t n, int *out)
{
    PyObject **items;
    if (PyTuple_CheckExact(o)) {
        if (PyTuple_GET_SIZE(o) != n) return false;
        items = &PyTuple_GET_ITEM(o, 0);
    } else if (PyList_CheckExact(o)) {
        if (PyList_GET_SIZE(o) != n) return false;
        items = &PyList_GET_ITEM(o, 0);
    } else {
        return false;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        if (!PyLong_CheckExact(items[i])) return false;
        int overflow;
        const long x = PyLong_AsLongAndOverflow(items[i], &overflow);
        if (overflow != 0 || x < INT32_MIN || x > INT32_MAX) return false;
        out[i] = (int)x;
    }
    return true;
}
bool windows(PyObject *o, int64_t heads, int *out)
{
    if (heads > kMaxHeads) return false;
    PyObject **items;
    if (PyList_CheckExact(o) && PyList_GET_SIZE(o) == heads) items = &PyList_GET_ITEM(o, 0);
    else if (PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == heads) items = &PyTuple_GET_ITEM(o, 0);
    else return false;
    for (int64_t h = 0; h < heads; ++h)
        if (!ints(items[h], 3, out + 3 * h)) return false;
    return true;
}
bool number(PyObject *o, float &out)
{
    if (!PyFloat_CheckExact(o)) return false;
    out = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
bool tokens_match(int64_t n, const int *grid) { return n == (int64_t)grid[0] * grid[1] * grid[2]; }

// The current stream of the current device; false with an exception set.
bool stream_of(void *&stream)
{
    PyObject *device = PyObject_CallNoArgs(current_device);
    if (!device) return false;
    PyObject *raw = PyObject_CallOneArg(current_raw_stream, device);
    Py_DECREF(device);
    if (!raw) return false;
    stream = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    return !PyErr_Occurred();
}

template <typename F>
PyObject *guarded(F &&f)
{
    try {
        return f();
    } catch (...) {                                 // a tensor that has no memory to point to: the general path says so
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
template <typename F>
PyObject *status_of(F &&launch)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = launch();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// (src, dst, grid, tile)
PyObject *permute(PermuteFn fn, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        View v[2];
        int grid[3], tile[3], src_type, dst_type;
        void *stream;
        if (!fn || n != 4 || !dense(args[0], v[0]) || !dense(args[1], v[1]) || !same_shape4(v, 2) || !dtype_code(v[0], src_type) ||
            !dtype_code(v[1], dst_type) || !ints(args[2], 3, grid) || !ints(args[3], 3, tile) || !tokens_match(v[0].t->size(2), grid))
            Py_RETURN_NONE;
        if (!stream_of(stream)) return nullptr;
        const int B = (int)v[0].t->size(0), H = (int)v[0].t->size(1), D = (int)v[0].t->size(3);
        return status_of([&]() { return fn(v[0].ptr, v[1].ptr, src_type, dst_type, B, H, D, grid, tile, stream); });
    });
}
PyObject *py_tile_permute(PyObject *, PyObject *const *args, Py_ssize_t n) { return permute(entries.tile_permute, args, n); }
PyObject *py_untile(PyObject *, PyObject *const *args, Py_ssize_t n) { return permute(entries.untile, args, n); }

// (q, k, v, o, grid, tile, windows, scale, workspace or None)
PyObject *py_forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        View v[4], ws = {nullptr, nullptr};
        int grid[3], tile[3], win[3 * kMaxHeads];
        float scale;
        void *stream;
        if (!entries.forward || n != 9) Py_RETURN_NONE;
        for (int i = 0; i < 4; ++i)
            if (!dense(args[i], v[i])) Py_RETURN_NONE;
        if (!same_shape4(v, 4) || !all_bf16(v, 4) || !ints(args[4], 3, grid) || !ints(args[5], 3, tile) ||
            !tokens_match(v[0].t->size(2), grid) || !windows(args[6], v[0].t->size(1), win) || !number(args[7], scale) ||
            (args[8] != Py_None && !dense(args[8], ws)))
            Py_RETURN_NONE;
        const size_t ws_bytes = ws.t ? ws.t->numel() * ws.t->element_size() : 0;
        if (!stream_of(stream)) return nullptr;
        const int B = (int)v[0].t->size(0), H = (int)v[0].t->size(1), D = (int)v[0].t->size(3);
        return status_of([&]() {
            return entries.forward(v[0].ptr, v[1].ptr, v[2].ptr, v[3].ptr, B, H, D, grid, tile, win, scale, ws.ptr, ws_bytes, stream);
        });
    });
}

// lse: float32 [B, H, N] that goes with tensors of shape [B, H, N, D]
bool lse_of(PyObject *o, const View &like, View &lse)
{
    return dense(o, lse) && lse.t->scalar_type() == at::kFloat && lse.t->dim() == 3 && lse.t->sizes() == like.t->sizes().slice(0, 3);
}

// (q, k, v, o, lse, grid, tile, windows, scale)
PyObject *py_forward_lse(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        View v[4], lse;
        int grid[3], tile[3], win[3 * kMaxHeads];
        float scale;
        void *stream;
        if (!entries.forward_lse || n != 9) Py_RETURN_NONE;
        for (int i = 0; i < 4; ++i)
            if (!dense(args[i], v[i])) Py_RETURN_NONE;
        if (!same_shape4(v, 4) || !all_bf16(v, 4) || !lse_of(args[4], v[0], lse) || !ints(args[5], 3, grid) || !ints(args[6], 3, tile) ||
            !tokens_match(v[0].t->size(2), grid) || !windows(args[7], v[0].t->size(1), win) || !number(args[8], scale))
            Py_RETURN_NONE;
        if (!stream_of(stream)) return nullptr;
        const int B = (int)v[0].t->size(0), H = (int)v[0].t->size(1), D = (int)v[0].t->size(3);
        return status_of([&]() {
            return entries.forward_lse(v[0].ptr, v[1].ptr, v[2].ptr, v[3].ptr, static_cast<float *>(lse.ptr), B, H, D, grid, tile, win,
                                       scale, stream);
        });
    });
}

// (q, k, v, o, d_o, lse, d_q, d_k, d_v, grid, tile, windows, workspace, scale)
PyObject *py_backward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        View v[8], lse, ws;
        int grid[3], tile[3], win[3 * kMaxHeads];
        float scale;
        void *stream;
        if (!entries.backward || n != 14) Py_RETURN_NONE;
        for (int i = 0; i < 8; ++i)
            if (!dense(args[i < 5 ? i : i + 1], v[i])) Py_RETURN_NONE;
        if (!same_shape4(v, 8) || !all_bf16(v, 8) || !lse_of(args[5], v[0], lse) || !ints(args[9], 3, grid) || !ints(args[10], 3, tile) ||
            !tokens_match(v[0].t->size(2), grid) || !windows(args[11], v[0].t->size(1), win) || !dense(args[12], ws) ||
            !number(args[13], scale))
            Py_RETURN_NONE;
        const size_t ws_bytes = ws.t->numel() * ws.t->element_size();
        if (!stream_of(stream)) return nullptr;
        const int B = (int)v[0].t->size(0), H = (int)v[0].t->size(1), D = (int)v[0].t->size(3);
        return status_of([&]() {
            return entries.backward(v[0].ptr, v[1].ptr, v[2].ptr, v[3].ptr, v[4].ptr, static_cast<const float *>(lse.ptr), v[5].ptr,
                                    v[6].ptr, v[7].ptr, B, H, D, grid, tile, win, scale, ws.ptr, ws_bytes, stream);
        });
    });
}

// (addresses of the five entry points in the order of Entries, torch's current device and raw current stream)
PyObject *py_bind(PyObject *, PyObject *args)
{
    unsigned long long a[5];
    PyObject *device, *stream;
    if (!PyArg_ParseTuple(args, "KKKKKOO", &a[0], &a[1], &a[2], &a[3], &a[4], &device, &stream)) return nullptr;
    Py_INCREF(device);
    Py_INCREF(stream);
    Py_XSETREF(current_device, device);
    Py_XSETREF(current_raw_stream, stream);
    entries.tile_permute = reinterpret_cast<PermuteFn>(a[0]);
    entries.untile = reinterpret_cast<PermuteFn>(a[1]);
    entries.forward = reinterpret_cast<ForwardFn>(a[2]);
    entries.forward_lse = reinterpret_cast<ForwardLseFn>(a[3]);
    entries.backward = reinterpret_cast<BackwardFn>(a[4]);
    Py_RETURN_NONE;
}

#define STA_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr}, STA_FAST(tile_permute), STA_FAST(untile), STA_FAST(forward), STA_FAST(forward_lse),
    STA_FAST(backward), {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "sta_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_sta_fastcall(void) { return PyModule_Create(&module); }
