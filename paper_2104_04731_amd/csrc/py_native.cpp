// Python entry points of the tensor-taking calls, as a C extension (module `_native`): argument checks, the result
// tensor, the current stream and the library call in one step.  The calls themselves are those of
// include/conv2d_int8.h; nothing here computes.
//
// Why native: a small layer runs for 3-7 us on the GPU and its launch costs the host about 2.4 us (hipLaunchKernel,
// measured), but marshalling it in Python -- torch.cuda.current_stream() 2.9 us, torch.empty 1.7 us, a ctypes call
// with 13 arguments 1 us, attribute checks 1 us -- took another 7, so that a 3.5-us layer cost 10.3 us back to back.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/conv2d_int8.h"

namespace {

PyObject *g_error = nullptr;  // binding.ConvError

// The library's calls, looked up in the library that binding.load() loaded (which need not be the one beside this module).
#define LIBRARY_CALLS(X)                                                                                                  \
    X(conv2d_int8) X(conv2d_int8_static) X(conv2d_int8_nhwc) X(conv2d_int8_ex) X(conv2d_int8_packed) X(conv2d_int8_packed_nhwc) \
    X(conv2d_int8_packed_requant) X(pack_layout) X(pack_layout_nhwc) X(pack_layout_bytes) X(pack_weights) X(pack_weights_depth) \
    X(im2col_int8) X(im2col_nhwc_int8) X(unpack_nhwc_int32) X(requant_int8) X(requant_pack_layout) X(conv2d_int8_dilated)  \
    X(conv2d_int8_dilated_workspace_bytes) X(conv2d_int8_dilated_direct) X(conv2d_int8_dilated_direct_workspace_bytes)     \
    X(gemm_int8_nt)
struct Library {
#define CALL(name) decltype(&::name) name;
    LIBRARY_CALLS(CALL)
#undef CALL
} lib;
bool g_loaded = false;

struct PyFail {};  // a Python error is set

// ---- arguments -----------------------------------------------------------------------------------------------
const at::Tensor &tensor(PyObject *o, const char *what)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch.Tensor, not %.100s", what, Py_TYPE(o)->tp_name);
        throw PyFail{};
    }
    return THPVariable_Unpack(o);
}

const at::Tensor &require(PyObject *o, at::ScalarType dtype, const char *what)
{
    const at::Tensor &t = tensor(o, what);
    if (!(t.is_cuda() && t.scalar_type() == dtype && t.is_contiguous())) {
        PyErr_Format(PyExc_TypeError, "%s must be a contiguous torch.%s CUDA tensor", what,
                     dtype == at::kChar ? "int8" : "int32");
        throw PyFail{};
    }
    return t;
}

void require_dims(const at::Tensor &t, int64_t n, const char *what)
{
    if (t.dim() != n) {
        PyErr_Format(PyExc_ValueError, "%s must have %d dimensions, not %d", what, (int)n, (int)t.dim());
        throw PyFail{};
    }
}

int as_int(PyObject *o)
{
    if (PyLong_CheckExact(o)) return (int)PyLong_AsUnsignedLongMask(o);
    PyObject *i = PyNumber_Index(o);
    if (!i) throw PyFail{};
    const int v = (int)PyLong_AsUnsignedLongMask(i);
    Py_DECREF(i);
    return v;
}

// int(o): for the arguments that the binding has always passed through int() (whole-number floats among them).
int as_int_cast(PyObject *o)
{
    if (PyLong_CheckExact(o)) return (int)PyLong_AsUnsignedLongMask(o);
    PyObject *i = PyObject_CallFunctionObjArgs((PyObject *)&PyLong_Type, o, nullptr);
    if (!i) throw PyFail{};
    const int v = (int)PyLong_AsUnsignedLongMask(i);
    Py_DECREF(i);
    return v;
}

// int(o) as a flag: None and the like are refused
bool as_flag(PyObject *o)
{
    if (PyBool_Check(o)) return o == Py_True;
    return as_int_cast(o) != 0;
}

bool as_bool(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyFail{};
    return v != 0;
}

conv_desc_t as_desc(PyObject *o)
{
    PyObject *s = PySequence_Fast(o, "dims must be (N, C, H, W, K, R, S, stride, pad)");
    if (!s) throw PyFail{};
    if (PySequence_Fast_GET_SIZE(s) != 9) {
        Py_DECREF(s);
        PyErr_SetString(PyExc_TypeError, "dims must be (N, C, H, W, K, R, S, stride, pad)");
        throw PyFail{};
    }
    int v[9];
    try {
        for (int i = 0; i < 9; ++i) v[i] = as_int(PySequence_Fast_GET_ITEM(s, i));
    } catch (PyFail &) {
        Py_DECREF(s);
        throw;
    }
    Py_DECREF(s);
    return conv_desc_t{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8]};
}

// None: the current stream of the current device; else the handle of a torch stream
void *as_stream(PyObject *o)
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject *h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) throw PyFail{};
    void *p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (!p && PyErr_Occurred()) throw PyFail{};
    return p;
}

// Python's floor division of an output extent, never negative
int64_t extent(int64_t span, int stride)
{
    if (stride == 0) {
        PyErr_SetString(PyExc_ZeroDivisionError, "integer division or modulo by zero");
        throw PyFail{};
    }
    int64_t q = span / stride;
    if (span % stride != 0 && (span < 0) != (stride < 0)) --q;
    return q + 1 > 0 ? q + 1 : 0;
}

[[noreturn]] void fail(int status, const char *what)
{
    PyObject *e = PyObject_CallFunction(g_error, "is", status, what);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw PyFail{};
}

void check(int status, const char *what)
{
    if (status != CONV_OK) fail(status, what);
}

// ---- the result: the caller's tensor, or a new one; the interpreter lock is given up for allocation and call ----
struct Out {
    PyObject *given;
    at::Tensor made;
    explicit Out(PyObject *o) : given(o == Py_None ? nullptr : o) {}
    void *ptr() const { return (given ? THPVariable_Unpack(given) : made).data_ptr(); }
    PyObject *result()
    {
        if (given) {
            Py_INCREF(given);
            return given;
        }
        return THPVariable_Wrap(std::move(made));
    }
};

at::Tensor empty_like_device(const at::Tensor &on, at::IntArrayRef shape, at::ScalarType dtype)
{
    return at::empty(shape, at::TensorOptions().dtype(dtype).device(on.device()));
}

struct NoGil {
    PyThreadState *s = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(s); }
};

template <class F>
PyObject *guarded(Py_ssize_t n, Py_ssize_t want, F &&f)
{
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
        return nullptr;
    }
    if (!g_loaded) {
        PyErr_SetString(PyExc_RuntimeError, "no library has been loaded: use the functions of binding.py");
        return nullptr;
    }
    HANDLE_TH_ERRORS  // torch's own exceptions (out of memory among them) under their Python names
    try {
        return f();
    } catch (PyFail &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

#define NATIVE(name, count, ...)                                                    \
    PyObject *py_##name(PyObject *, PyObject *const *a, Py_ssize_t n)               \
    {                                                                               \
        return guarded(n, count, [&]() -> PyObject * __VA_ARGS__);                       \
    }

// ---- convolutions on whole tensors: (x, w, stride, pad, out, stream) ---------------------------------------
template <class F>
PyObject *one_shot(PyObject *const *a, const char *name, bool nhwc, bool given_only, F &&call)
{
    const at::Tensor &x = require(a[0], at::kChar, "input"), &w = require(a[1], at::kChar, "weights");
    if (given_only) require(a[4], at::kInt, "output");
    require_dims(x, 4, "input");
    require_dims(w, 4, "weights");
    const int64_t N = x.size(0), C = x.size(nhwc ? 3 : 1), H = x.size(nhwc ? 1 : 2), W = x.size(nhwc ? 2 : 3);
    const int64_t K = w.size(0), R = w.size(2), S = w.size(3);
    if (w.size(1) != C) {
        PyErr_SetString(PyExc_ValueError, "channel mismatch");
        throw PyFail{};
    }
    const int stride = as_int(a[2]), pad = as_int(a[3]);
    Out out(a[4]);
    if (out.given) tensor(a[4], "output");
    void *st = as_stream(a[5]);
    int64_t P = 0, Q = 0;
    if (!given_only) {
        P = extent(H + 2LL * pad - R, stride);
        Q = extent(W + 2LL * pad - S, stride);
    }
    int rc;
    {
        NoGil unlocked;
        if (!out.given) {
            const int64_t nkpq[4] = {N, K, P, Q}, npqk[4] = {N, P, Q, K};
            out.made = empty_like_device(x, nhwc ? npqk : nkpq, at::kInt);
        }
        rc = call((int)N, (int)C, (int)H, (int)W, (int)K, (int)R, (int)S, stride, pad, (const int8_t *)x.data_ptr(),
                  (const int8_t *)w.data_ptr(), (int32_t *)out.ptr(), st);
    }
    check(rc, name);
    return out.result();
}

NATIVE(conv2d_int8, 6, { return one_shot(a, "conv2d_int8", false, false, lib.conv2d_int8); })
NATIVE(conv2d_int8_static, 6, { return one_shot(a, "conv2d_int8_static", false, true, lib.conv2d_int8_static); })
NATIVE(conv2d_int8_nhwc, 6, { return one_shot(a, "conv2d_int8_nhwc", true, false, lib.conv2d_int8_nhwc); })

// (dims, layout, cb, x, w, out, workspace, wt_is_packed, stream)
NATIVE(conv2d_int8_ex, 9, {
    const conv_desc_t d = as_desc(a[0]);
    const int layout = as_int(a[1]), cb = as_int(a[2]);
    const at::Tensor &x = tensor(a[3], "input"), &w = tensor(a[4], "weights"), &o = tensor(a[5], "output");
    const at::Tensor *ws = a[6] == Py_None ? nullptr : &tensor(a[6], "workspace");
    const int packed = as_flag(a[7]);
    void *st = as_stream(a[8]);
    int rc;
    {
        NoGil unlocked;
        rc = lib.conv2d_int8_ex(&d, layout, cb, (const int8_t *)x.data_ptr(), (const int8_t *)w.data_ptr(), packed, (int32_t *)o.data_ptr(),
                            ws ? ws->data_ptr() : nullptr, ws ? (size_t)ws->numel() * ws->element_size() : 0, st);
    }
    check(rc, "conv2d_int8_ex");
    Py_INCREF(a[5]);
    return a[5];
})

// (dims, layout, cb, x_packed, w_packed, out, tile, split_k, stream)
template <class F>
PyObject *gemm_stage(PyObject *const *a, const char *name, F &&call)
{
    const conv_desc_t d = as_desc(a[0]);
    const int layout = as_int(a[1]), cb = as_int(a[2]), tile = as_int(a[6]), split = as_int(a[7]);
    const at::Tensor &x = tensor(a[3], "input"), &w = tensor(a[4], "weights"), &o = tensor(a[5], "output");
    void *st = as_stream(a[8]);
    int rc;
    {
        NoGil unlocked;
        rc = call(&d, layout, cb, (const int8_t *)x.data_ptr(), (const int8_t *)w.data_ptr(), (int32_t *)o.data_ptr(), tile, split, st);
    }
    check(rc, name);
    Py_INCREF(a[5]);
    return a[5];
}

NATIVE(conv2d_int8_packed, 9, { return gemm_stage(a, "conv2d_int8_packed", lib.conv2d_int8_packed); })
NATIVE(conv2d_int8_packed_nhwc, 9, { return gemm_stage(a, "conv2d_int8_packed_nhwc", lib.conv2d_int8_packed_nhwc); })

// (dims, layout, cb, x_packed, w_packed, out_cb, out_pad, shift, relu, out, stream)
NATIVE(conv2d_int8_packed_requant, 11, {
    const conv_desc_t d = as_desc(a[0]);
    const int layout = as_int_cast(a[1]), cb = as_int_cast(a[2]), shift = as_int_cast(a[7]);
    const at::Tensor &x = tensor(a[3], "input"), &w = tensor(a[4], "weights");
    const int relu = as_bool(a[8]);
    Out out(a[9]);
    if (out.given) tensor(a[9], "output");
    // (a result to be made has its shape from these two: integers only)
    const int out_cb = out.given ? as_int_cast(a[5]) : as_int(a[5]), out_pad = out.given ? as_int_cast(a[6]) : as_int(a[6]);
    void *st = as_stream(a[10]);
    int64_t P = 0, Q = 0;
    if (!out.given) {
        if (out_cb == 0) {
            PyErr_SetString(PyExc_ZeroDivisionError, "integer division or modulo by zero");
            throw PyFail{};
        }
        P = extent(d.H + 2LL * d.pad - d.R, d.stride);
        Q = extent(d.W + 2LL * d.pad - d.S, d.stride);
    }
    int rc;
    {
        NoGil unlocked;
        if (!out.given) {
            const int64_t shape[5] = {d.N, (d.K + (int64_t)out_cb - 1) / out_cb, P + 2LL * out_pad, Q + 2LL * out_pad, out_cb};
            out.made = empty_like_device(x, shape, at::kChar);
        }
        rc = lib.conv2d_int8_packed_requant(&d, layout, cb, (const int8_t *)x.data_ptr(), (const int8_t *)w.data_ptr(), (int8_t *)out.ptr(),
                                        out_cb, out_pad, shift, relu, st);
    }
    check(rc, "conv2d_int8_packed_requant");
    return out.result();
})

// ---- layout rewrites ----------------------------------------------------------------------------------------
// (x, cb, pad, out, stream)
template <class F>
PyObject *pack(PyObject *const *a, const char *name, bool nhwc, F &&call)
{
    const at::Tensor &x = require(a[0], at::kChar, "input");
    require_dims(x, 4, "input");
    const int cb = as_int(a[1]), pad = as_int(a[2]);
    Out out(a[3]);
    if (out.given) tensor(a[3], "output");
    void *st = as_stream(a[4]);
    const int64_t N = x.size(0), C = x.size(nhwc ? 3 : 1), H = x.size(nhwc ? 1 : 2), W = x.size(nhwc ? 2 : 3);
    if (!out.given && (lib.pack_layout_bytes((int)N, (int)C, (int)H, (int)W, cb, pad) == 0 || (nhwc && cb % 16)))
        fail(CONV_ERR_UNSUPPORTED, name);
    int rc;
    {
        NoGil unlocked;
        if (!out.given) {
            const int64_t shape[5] = {N, (C + cb - 1) / cb, H + 2LL * pad, W + 2LL * pad, cb};
            out.made = empty_like_device(x, shape, at::kChar);
        }
        rc = call((int)N, (int)C, (int)H, (int)W, cb, pad, (const int8_t *)x.data_ptr(), (int8_t *)out.ptr(), st);
    }
    check(rc, name);
    return out.result();
}

NATIVE(pack_layout, 5, { return pack(a, "pack_layout", false, lib.pack_layout); })
NATIVE(pack_layout_nhwc, 5, { return pack(a, "pack_layout_nhwc", true, lib.pack_layout_nhwc); })

// (w, layout, cb, out, stream)
NATIVE(pack_weights, 5, {
    const at::Tensor &w = require(a[0], at::kChar, "weights");
    require_dims(w, 4, "weights");
    const int layout = as_int(a[1]), cb = as_int(a[2]);
    const int K = (int)w.size(0), C = (int)w.size(1), R = (int)w.size(2), S = (int)w.size(3);
    Out out(a[3]);
    if (out.given) tensor(a[3], "output");
    void *st = as_stream(a[4]);
    const int depth = out.given ? 0 : lib.pack_weights_depth(C, R, S, layout, cb);
    if (!out.given && depth == 0) fail(CONV_ERR_UNSUPPORTED, "pack_weights");
    int rc;
    {
        NoGil unlocked;
        if (!out.given) out.made = empty_like_device(w, {(int64_t)K, (int64_t)depth}, at::kChar);
        rc = lib.pack_weights(K, C, R, S, layout, cb, (const int8_t *)w.data_ptr(), (int8_t *)out.ptr(), st);
    }
    check(rc, "pack_weights");
    return out.result();
})

// (x, R, S, stride, pad, kg_pad, out, stream)
template <class F>
PyObject *im2col(PyObject *const *a, const char *name, bool nhwc, F &&call)
{
    const at::Tensor &x = require(a[0], at::kChar, "input");
    require_dims(x, 4, "input");
    const int R = as_int(a[1]), S = as_int(a[2]), stride = as_int(a[3]), pad = as_int(a[4]);
    const int64_t N = x.size(0), C = x.size(nhwc ? 3 : 1), H = x.size(nhwc ? 1 : 2), W = x.size(nhwc ? 2 : 3);
    const int kg = a[5] == Py_None ? (int)((C * R * S + 63) / 64 * 64) : as_int(a[5]);
    Out out(a[6]);
    if (out.given) tensor(a[6], "output");
    void *st = as_stream(a[7]);
    int64_t P = 0, Q = 0;
    if (!out.given) {
        P = extent(H + 2LL * pad - R, stride);
        Q = extent(W + 2LL * pad - S, stride);
    }
    int rc;
    {
        NoGil unlocked;
        if (!out.given) out.made = empty_like_device(x, {N * P * Q, (int64_t)kg}, at::kChar);
        rc = call((int)N, (int)C, (int)H, (int)W, R, S, stride, pad, kg, (const int8_t *)x.data_ptr(), (int8_t *)out.ptr(), st);
    }
    check(rc, name);
    return out.result();
}

NATIVE(im2col_int8, 8, { return im2col(a, "im2col_int8", false, lib.im2col_int8); })
NATIVE(im2col_nhwc_int8, 8, { return im2col(a, "im2col_nhwc_int8", true, lib.im2col_nhwc_int8); })

// ---- between layers -----------------------------------------------------------------------------------------
// (x, out, stream)
NATIVE(unpack_nhwc_int32, 3, {
    const at::Tensor &x = require(a[0], at::kInt, "NKPQ tensor");
    require_dims(x, 4, "NKPQ tensor");
    const int64_t N = x.size(0), K = x.size(1), P = x.size(2), Q = x.size(3);
    Out out(a[1]);
    if (out.given) tensor(a[1], "output");
    void *st = as_stream(a[2]);
    int rc;
    {
        NoGil unlocked;
        if (!out.given) out.made = empty_like_device(x, {N, P, Q, K}, at::kInt);
        rc = lib.unpack_nhwc_int32((int)N, (int)K, (int)P, (int)Q, (const int32_t *)x.data_ptr(), (int32_t *)out.ptr(), st);
    }
    check(rc, "unpack_nhwc_int32");
    return out.result();
})

// (x, shift, relu, out, stream)
NATIVE(requant_int8, 5, {
    const at::Tensor &x = require(a[0], at::kInt, "accumulator tensor");
    const int shift = as_int(a[1]), relu = as_flag(a[2]);
    Out out(a[3]);
    if (out.given) tensor(a[3], "output");
    void *st = as_stream(a[4]);
    int rc;
    {
        NoGil unlocked;
        if (!out.given) out.made = empty_like_device(x, x.sizes(), at::kChar);
        rc = lib.requant_int8(x.numel(), (const int32_t *)x.data_ptr(), (int8_t *)out.ptr(), shift, relu, st);
    }
    check(rc, "requant_int8");
    return out.result();
})

// (x, cb, pad, shift, relu, out, stream)
NATIVE(requant_pack_layout, 7, {
    const at::Tensor &x = require(a[0], at::kInt, "accumulator tensor");
    require_dims(x, 4, "accumulator tensor");
    const int cb = as_int(a[1]), pad = as_int(a[2]), shift = as_int(a[3]), relu = as_flag(a[4]);
    const int64_t N = x.size(0), K = x.size(1), P = x.size(2), Q = x.size(3);
    Out out(a[5]);
    if (out.given) tensor(a[5], "output");
    void *st = as_stream(a[6]);
    if (!out.given && (cb <= 0 || cb % 16)) fail(CONV_ERR_UNSUPPORTED, "requant_pack_layout");
    int rc;
    {
        NoGil unlocked;
        if (!out.given) {
            const int64_t shape[5] = {N, (K + cb - 1) / cb, P + 2LL * pad, Q + 2LL * pad, cb};
            out.made = empty_like_device(x, shape, at::kChar);
        }
        rc = lib.requant_pack_layout((int)N, (int)K, (int)P, (int)Q, cb, pad, shift, relu, (const int32_t *)x.data_ptr(), (int8_t *)out.ptr(), st);
    }
    check(rc, "requant_pack_layout");
    return out.result();
})

// ---- dilated convolution: (dims, dilation, x, w, layout, cb, out, workspace, stream); `direct` ignores layout -----
at::Tensor aligned_workspace(const at::Tensor &on, size_t need)
{
    at::Tensor t = empty_like_device(on, {(int64_t)(need + 256)}, at::kChar);
    const int64_t skip = (int64_t)((-(uintptr_t)t.data_ptr()) & 255);
    return skip ? t.slice(0, skip) : t;
}

PyObject *dilated(PyObject *const *a, bool direct)
{
    const conv_desc_t d = as_desc(a[0]);
    const int layout = as_int_cast(a[4]), cb = as_int_cast(a[5]);
    const at::Tensor &x = require(a[2], at::kChar, "input"), &w = require(a[3], at::kChar, "weights");
    Out out(a[6]);
    if (out.given) tensor(a[6], "output");
    const int dil = out.given ? as_int_cast(a[1]) : as_int(a[1]);   // (a result to be made has its shape from it: integers only)
    at::Tensor ws;
    if (a[7] != Py_None) ws = tensor(a[7], "workspace");
    void *st = as_stream(a[8]);
    int64_t P = 0, Q = 0;
    if (!out.given) {
        const int64_t sp = d.H + 2LL * d.pad - (int64_t)dil * (d.R - 1), sq = d.W + 2LL * d.pad - (int64_t)dil * (d.S - 1);
        P = direct ? extent(sp - 1, d.stride) : sp > 0 ? sp : 0;
        Q = direct ? extent(sq - 1, d.stride) : sq > 0 ? sq : 0;
    }
    int rc;
    {
        NoGil unlocked;
        if (!out.given) out.made = empty_like_device(x, {d.N, d.K, P, Q}, at::kInt);
        if (!ws.defined())
            ws = aligned_workspace(x, direct ? lib.conv2d_int8_dilated_direct_workspace_bytes(&d, dil, cb)
                                             : lib.conv2d_int8_dilated_workspace_bytes(&d, dil, layout, cb));
        rc = direct ? lib.conv2d_int8_dilated_direct(&d, dil, cb, (const int8_t *)x.data_ptr(), (const int8_t *)w.data_ptr(), (int32_t *)out.ptr(),
                                                 ws.data_ptr(), ws.numel(), st)
                    : lib.conv2d_int8_dilated(&d, dil, layout, cb, (const int8_t *)x.data_ptr(), (const int8_t *)w.data_ptr(), (int32_t *)out.ptr(),
                                          ws.data_ptr(), ws.numel(), st);
    }
    check(rc, direct ? "conv2d_int8_dilated_direct" : "conv2d_int8_dilated");
    return out.result();
}

NATIVE(conv2d_int8_dilated, 9, { return dilated(a, false); })
NATIVE(conv2d_int8_dilated_direct, 9, { return dilated(a, true); })

// (A, B, out, stream)
NATIVE(gemm_int8_nt, 4, {
    const at::Tensor &A = require(a[0], at::kChar, "A"), &B = require(a[1], at::kChar, "B");
    require_dims(A, 2, "A");
    require_dims(B, 2, "B");
    if (A.size(1) != B.size(1)) {
        PyErr_SetString(PyExc_ValueError, "depth mismatch");
        throw PyFail{};
    }
    Out out(a[2]);
    if (out.given) tensor(a[2], "output");
    void *st = as_stream(a[3]);
    int rc;
    {
        NoGil unlocked;
        if (!out.given) out.made = empty_like_device(A, {A.size(0), B.size(0)}, at::kInt);
        rc = lib.gemm_int8_nt((int)A.size(0), (int)B.size(0), (int)A.size(1), (const int8_t *)A.data_ptr(), (const int8_t *)B.data_ptr(),
                          (int32_t *)out.ptr(), st);
    }
    check(rc, "gemm_int8_nt");
    return out.result();
})

PyObject *set_error_class(PyObject *, PyObject *cls)
{
    Py_XDECREF(g_error);
    Py_INCREF(cls);
    g_error = cls;
    Py_RETURN_NONE;
}

// The handle of the loaded library (an integer, as ctypes has it).
PyObject *set_library(PyObject *, PyObject *handle)
{
    void *const h = PyLong_AsVoidPtr(handle);
    if (!h) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a library handle is not null");
        return nullptr;
    }
    Library found;
#define CALL(name)                                                                        \
    if (!(found.name = reinterpret_cast<decltype(&::name)>(dlsym(h, #name)))) {          \
        PyErr_SetString(PyExc_RuntimeError, "the loaded library has no symbol " #name);    \
        return nullptr;                                                                    \
    }
    LIBRARY_CALLS(CALL)
#undef CALL
    lib = found;
    g_loaded = true;
    Py_RETURN_NONE;
}

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ENTRY(conv2d_int8), ENTRY(conv2d_int8_static), ENTRY(conv2d_int8_nhwc), ENTRY(conv2d_int8_ex), ENTRY(conv2d_int8_packed),
    ENTRY(conv2d_int8_packed_nhwc), ENTRY(conv2d_int8_packed_requant), ENTRY(pack_layout), ENTRY(pack_layout_nhwc), ENTRY(pack_weights),
    ENTRY(im2col_int8), ENTRY(im2col_nhwc_int8), ENTRY(unpack_nhwc_int32), ENTRY(requant_int8), ENTRY(requant_pack_layout),
    ENTRY(conv2d_int8_dilated), ENTRY(conv2d_int8_dilated_direct), ENTRY(gemm_int8_nt),
    {"set_error_class", set_error_class, METH_O, nullptr}, {"set_library", set_library, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
