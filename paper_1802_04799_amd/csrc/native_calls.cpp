// The call path from Python to libtvg as a CPython extension: argument unpacking, output
// allocation and the current-stream lookup of every operator call.
//
// What it is for: a batch-1 operator keeps the GPU busy for 3-10 us, and the same call through
// ctypes (marshalling of eleven arguments, a Stream object per call, a dozen attribute reads per
// tensor for the checks) took 8-13 us of host time, so launch-bound programs waited for Python.
// Here a tensor's address, shape and type are read from the C++ object behind it (about 10 ns
// each).  Nine depthwise layers at batch 1 through dwconv2d_fused: 106 us before (32 us of it
// kernels), 41 us now: a call costs 3.6 us, 2.5 of them the launch itself and 1.0 the output tensor.
//
// Only the ordinary case is handled natively.  A convenience call whose arguments are anything
// else (a wrong type, device, layout or dtype, a subclass of Tensor, objects that merely look like
// tensors) is handed to the Python implementation in binding.py, which raises the error that fits or
// handles it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "tvg.h"

namespace {

PyObject *g_desc_type = nullptr;       // binding.ConvDesc
PyObject *g_error_type = nullptr;      // binding.TvgError
PyObject *g_fallback = nullptr;        // name -> Python implementation of a convenience call

// ---------------------------------------------------------------------------------------
// arguments
// ---------------------------------------------------------------------------------------

// A function's parameters: `required` of them must be given, the first `positional` may be given
// by position, all by name.
struct Spec {
    const char *name;
    int count, positional, required;
    const char *const *names;
    PyObject **interned;               // filled when the module is made
};

bool parse(const Spec &s, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, PyObject **out)
{
    if (nargs > s.positional) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d positional arguments but %zd were given", s.name,
                     s.positional, nargs);
        return false;
    }
    for (Py_ssize_t i = 0; i < nargs; ++i) out[i] = args[i];
    for (int i = (int)nargs; i < s.count; ++i) out[i] = nullptr;
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject *key = PyTuple_GET_ITEM(kwnames, k);
        int at = -1;
        for (int i = 0; i < s.count && at < 0; ++i)
            if (s.interned[i] == key) at = i;
        for (int i = 0; i < s.count && at < 0; ++i)
            if (PyUnicode_Compare(s.interned[i], key) == 0) at = i;
        if (at < 0) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", s.name, key);
            return false;
        }
        if (out[at]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", s.name, key);
            return false;
        }
        out[at] = args[nargs + k];
    }
    for (int i = 0; i < s.required; ++i)
        if (!out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing a required argument: '%s'", s.name, s.names[i]);
            return false;
        }
    return true;
}

// An address: None, an int, a tensor, or any object with data_ptr().
bool address(PyObject *o, void **out)
{
    *out = nullptr;
    if (!o || o == Py_None) return true;
    if (THPVariable_CheckExact(o)) {       // (a subclass is asked like any other object: its answer may differ)
        *out = THPVariable_Unpack(o).data_ptr();
        return true;
    }
    PyObject *value = nullptr;
    if (PyLong_Check(o)) {
        value = o;
        Py_INCREF(value);
    } else {
        value = PyObject_CallMethod(o, "data_ptr", nullptr);
        if (!value) return false;
    }
    *out = PyLong_AsVoidPtr(value);
    Py_DECREF(value);
    return !(PyErr_Occurred() != nullptr);
}

// A stream handle: None (torch's current stream), an int, or an object with cuda_stream.
bool stream_handle(PyObject *o, void **out)
{
    if (!o || o == Py_None) {
        *out = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
        return !(PyErr_Occurred() != nullptr);
    }
    PyObject *value = PyObject_GetAttrString(o, "cuda_stream");
    if (!value) return false;
    *out = PyLong_AsVoidPtr(value);
    Py_DECREF(value);
    return !(PyErr_Occurred() != nullptr);
}

// An integer; values beyond the C type wrap around, as in ctypes.
bool integer(PyObject *o, long long fallback, long long *out)
{
    *out = fallback;
    if (!o) return true;
    PyObject *i = PyNumber_Index(o);
    if (!i) return false;
    *out = (long long)PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return !(*out == -1 && PyErr_Occurred());
}

// What int() makes an integer of, for the arguments that take it.
bool as_integer(PyObject *o, long long fallback, long long *out)
{
    if (!o || PyLong_Check(o)) return integer(o, fallback, out);
    PyObject *i = PyNumber_Long(o);
    const bool ok = i && integer(i, fallback, out);
    Py_XDECREF(i);
    return ok;
}

bool descriptor(PyObject *o, tvg_conv_desc *out)
{
    const int is = PyObject_IsInstance(o, g_desc_type);
    if (is < 0) return false;
    Py_buffer view;
    if (!is) {
        PyErr_Format(PyExc_TypeError, "desc must be a ConvDesc, not %s", Py_TYPE(o)->tp_name);
        return false;
    }
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
    const bool fits = view.len == (Py_ssize_t)sizeof(*out);
    if (fits) *out = *static_cast<const tvg_conv_desc *>(view.buf);
    PyBuffer_Release(&view);
    if (!fits) PyErr_SetString(PyExc_TypeError, "desc has the wrong size");
    return fits;
}

// Runs a library call without the GIL, which is held again on every way out.  Nothing of torch's
// belongs in `f`: reading a tensor's address may raise (tensors without storage), so callers read
// every address before.
template <typename F>
tvg_status without_gil(F &&f)
{
    struct Released {
        PyThreadState *state = PyEval_SaveThread();
        ~Released() { PyEval_RestoreThread(state); }
    } released;
    return f();
}

// Runs a call's body; C++ exceptions become the Python ones that torch's own calls raise for them
// (OutOfMemoryError where an allocation failed, else RuntimeError and the like).
template <typename F>
PyObject *guarded(F &&f)
{
    try {
        return f();
    } catch (...) {
        if (!PyErr_Occurred()) torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

PyObject *raise_status(tvg_status st, const char *where)
{
    PyObject *e = PyObject_CallFunction(g_error_type, "is", (int)st, where);
    if (e) {
        PyErr_SetObject(g_error_type, e);
        Py_DECREF(e);
    }
    return nullptr;
}

PyObject *fall_back(const char *name, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    PyObject *f = PyDict_GetItemString(g_fallback, name);      // borrowed
    if (!f) {
        PyErr_SetString(PyExc_RuntimeError, "the native call path was not set up");
        return nullptr;
    }
    return PyObject_Vectorcall(f, args, (size_t)nargs, kwnames);
}

// ---------------------------------------------------------------------------------------
// the C entry points: addresses in, status code out
// ---------------------------------------------------------------------------------------

#define SPEC(fn, pos, req, ...)                                                                    \
    const char *const fn##_names[] = {__VA_ARGS__};                                                \
    PyObject *fn##_interned[sizeof(fn##_names) / sizeof(char *)];                                  \
    const Spec fn##_spec = {#fn, (int)(sizeof(fn##_names) / sizeof(char *)), pos, req, fn##_names, fn##_interned}

SPEC(tvg_conv2d_fused, 11, 8, "desc", "x", "w", "scale", "shift", "bias", "residual", "y", "workspace",
     "workspace_bytes", "stream");
SPEC(tvg_dwconv2d_fused, 11, 8, "desc", "x", "w", "scale", "shift", "bias", "residual", "y", "workspace",
     "workspace_bytes", "stream");
SPEC(tvg_conv2d_fused_static, 9, 8, "desc", "x", "w", "scale", "shift", "bias", "residual", "y", "stream");
SPEC(tvg_conv2d_fused_dual, 12, 11, "desc", "k1", "flags2", "x", "w", "scale", "shift", "bias", "residual1", "y1",
     "y2", "stream");
SPEC(tvg_conv2d_fused_prepacked, 11, 10, "desc", "x", "packed", "scale", "shift", "bias", "residual", "y",
     "workspace", "workspace_bytes", "stream");
SPEC(tvg_dwpw_fused, 16, 13, "dw_desc", "pw_k", "pw_flags", "x", "w_dw", "scale_dw", "shift_dw", "w_pw", "scale_pw",
     "shift_pw", "bias_pw", "residual", "y", "workspace", "workspace_bytes", "stream");
SPEC(tvg_maxpool2d_3x3s2, 8, 7, "n", "c", "h", "w", "dtype", "x", "y", "stream");

#define ARGS PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames

typedef tvg_status (*conv_entry)(const tvg_conv_desc *, const void *, const void *, const float *, const float *,
                                 const float *, const void *, void *, void *, size_t, void *);

PyObject *conv_like(conv_entry fn, const Spec &spec, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames,
                    bool prepacked = false)
{
    return guarded([&]() -> PyObject * {
        PyObject *v[11];
        tvg_conv_desc d;
        void *p[8], *stream;
        long long bytes;
        if (!parse(spec, args, nargs, kwnames, v) || !descriptor(v[0], &d)) return nullptr;
        for (int i = 0; i < 8; ++i)
            if (!address(v[1 + i], &p[i])) return nullptr;
        if (!(prepacked ? as_integer : integer)(v[9], 0, &bytes) || !stream_handle(v[10], &stream)) return nullptr;
        const tvg_status st = without_gil([&] {
            return fn(&d, p[0], p[1], static_cast<float *>(p[2]), static_cast<float *>(p[3]),
                      static_cast<float *>(p[4]), p[5], p[6], p[7], (size_t)bytes, stream);
        });
        return PyLong_FromLong(st);
    });
}

PyObject *py_tvg_conv2d_fused(ARGS) { return conv_like(tvg_conv2d_fused, tvg_conv2d_fused_spec, args, nargs, kwnames); }
PyObject *py_tvg_dwconv2d_fused(ARGS)
{
    return conv_like(tvg_dwconv2d_fused, tvg_dwconv2d_fused_spec, args, nargs, kwnames);
}
PyObject *py_tvg_conv2d_fused_prepacked(ARGS)
{
    return conv_like(tvg_conv2d_fused_prepacked, tvg_conv2d_fused_prepacked_spec, args, nargs, kwnames, true);
}

PyObject *py_tvg_conv2d_fused_static(ARGS)
{
    return guarded([&]() -> PyObject * {
        PyObject *v[9];
        tvg_conv_desc d;
        void *p[7], *stream;
        if (!parse(tvg_conv2d_fused_static_spec, args, nargs, kwnames, v) || !descriptor(v[0], &d)) return nullptr;
        for (int i = 0; i < 7; ++i)
            if (!address(v[1 + i], &p[i])) return nullptr;
        if (!stream_handle(v[8], &stream)) return nullptr;
        const tvg_status st = without_gil([&] {
            return tvg_conv2d_fused_static(&d, p[0], p[1], static_cast<float *>(p[2]), static_cast<float *>(p[3]),
                                           static_cast<float *>(p[4]), p[5], p[6], stream);
        });
        return PyLong_FromLong(st);
    });
}

PyObject *py_tvg_conv2d_fused_dual(ARGS)
{
    return guarded([&]() -> PyObject * {
        PyObject *v[12];
        tvg_conv_desc d;
        void *p[8], *stream;
        long long k1, flags2;
        if (!parse(tvg_conv2d_fused_dual_spec, args, nargs, kwnames, v) || !descriptor(v[0], &d) ||
            !as_integer(v[1], 0, &k1) || !as_integer(v[2], 0, &flags2))
            return nullptr;
        for (int i = 0; i < 8; ++i)
            if (!address(v[3 + i], &p[i])) return nullptr;
        if (!stream_handle(v[11], &stream)) return nullptr;
        const tvg_status st = without_gil([&] {
            return tvg_conv2d_fused_dual(&d, (int32_t)k1, (uint32_t)flags2, p[0], p[1], static_cast<float *>(p[2]),
                                         static_cast<float *>(p[3]), static_cast<float *>(p[4]), p[5], p[6], p[7],
                                         stream);
        });
        return PyLong_FromLong(st);
    });
}

PyObject *py_tvg_dwpw_fused(ARGS)
{
    return guarded([&]() -> PyObject * {
        PyObject *v[16];
        tvg_conv_desc d;
        void *p[11], *stream;
        long long k, flags, bytes;
        if (!parse(tvg_dwpw_fused_spec, args, nargs, kwnames, v) || !descriptor(v[0], &d) ||
            !as_integer(v[1], 0, &k) || !as_integer(v[2], 0, &flags))
            return nullptr;
        for (int i = 0; i < 11; ++i)
            if (!address(v[3 + i], &p[i])) return nullptr;
        if (!integer(v[14], 0, &bytes) || !stream_handle(v[15], &stream)) return nullptr;
        const tvg_status st = without_gil([&] {
            return tvg_dwpw_fused(&d, (int32_t)k, (uint32_t)flags, p[0], p[1], static_cast<float *>(p[2]),
                                  static_cast<float *>(p[3]), p[4], static_cast<float *>(p[5]),
                                  static_cast<float *>(p[6]), static_cast<float *>(p[7]), p[8], p[9], p[10],
                                  (size_t)bytes, stream);
        });
        return PyLong_FromLong(st);
    });
}

PyObject *py_tvg_maxpool2d_3x3s2(ARGS)
{
    return guarded([&]() -> PyObject * {
        PyObject *v[8];
        void *x, *y, *stream;
        long long d[5];
        if (!parse(tvg_maxpool2d_3x3s2_spec, args, nargs, kwnames, v)) return nullptr;
        for (int i = 0; i < 5; ++i)
            if (!integer(v[i], 0, &d[i])) return nullptr;
        if (!address(v[5], &x) || !address(v[6], &y) || !stream_handle(v[7], &stream)) return nullptr;
        const tvg_status st = without_gil([&] {
            return tvg_maxpool2d_3x3s2((int32_t)d[0], (int32_t)d[1], (int32_t)d[2], (int32_t)d[3], (int32_t)d[4], x, y,
                                       stream);
        });
        return PyLong_FromLong(st);
    });
}

// ---------------------------------------------------------------------------------------
// the conveniences: tensors in, the output tensor back
// ---------------------------------------------------------------------------------------

SPEC(conv2d_fused, 6, 4, "x", "w", "scale", "shift", "bias", "residual", "stride", "pad", "relu", "out", "workspace",
     "stream", "stream_out");
SPEC(dwconv2d_fused, 6, 4, "x", "w", "scale", "shift", "bias", "residual", "stride", "pad", "relu", "out", "stream",
     "stream_out");
SPEC(dwpw_fused, 9, 7, "x", "w_dw", "scale_dw", "shift_dw", "w_pw", "scale_pw", "shift_pw", "bias_pw", "residual",
     "stride", "relu_dw", "relu_pw", "out", "workspace", "stream", "stream_out", "one_kernel");

bool absent(PyObject *o) { return !o || o == Py_None; }

// A contiguous device tensor of the given type; `optional` ones may be None.
bool plain_tensor(PyObject *o, bool optional, c10::ScalarType dtype, const at::Tensor **out)
{
    *out = nullptr;
    if (absent(o)) return optional;
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous() || t.scalar_type() != dtype) return false;
    *out = &t;
    return true;
}

// None or a tensor (an output or a workspace: of any type and shape, the bytes are what counts).
bool plain_buffer(PyObject *o, const at::Tensor **out)
{
    *out = nullptr;
    if (absent(o)) return true;
    if (!THPVariable_CheckExact(o)) return false;
    *out = &THPVariable_Unpack(o);
    return true;
}

size_t bytes_of(const at::Tensor *t) { return t ? (size_t)t->numel() * t->element_size() : 0; }

bool dense_on_device(const at::Tensor &t) { return t.is_cuda() && t.is_contiguous(); }

bool flag(PyObject *o, bool fallback, bool *out)
{
    if (!o) {
        *out = fallback;
        return true;
    }
    if (o != Py_True && o != Py_False) return false;
    *out = o == Py_True;
    return true;
}

bool extent(PyObject *o, int32_t *out)
{
    if (!PyLong_CheckExact(o)) return false;
    const long v = PyLong_AsLong(o);
    if ((v == -1 && PyErr_Occurred()) || v < INT32_MIN || v > INT32_MAX) {
        PyErr_Clear();
        return false;
    }
    *out = (int32_t)v;
    return true;
}

// An int for both directions, or a tuple of two.
bool extent_pair(PyObject *o, int fallback, int32_t *a, int32_t *b)
{
    *a = *b = fallback;
    if (!o) return true;
    if (PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2)
        return extent(PyTuple_GET_ITEM(o, 0), a) && extent(PyTuple_GET_ITEM(o, 1), b);
    if (!extent(o, a)) return false;
    *b = *a;
    return true;
}

bool known_dtype(const at::Tensor &x, int32_t *code)
{
    if (x.scalar_type() == at::kFloat) *code = TVG_F32;
    else if (x.scalar_type() == at::kBFloat16) *code = TVG_BF16;
    else return false;
    return true;
}

bool describe(const at::Tensor &x, const at::Tensor &w, PyObject *stride, PyObject *pad, int pad_default, uint32_t flags,
              tvg_conv_desc *d)
{
    if (x.dim() != 4 || w.dim() != 4) return false;
    const int64_t e[7] = {x.size(0), x.size(1), x.size(2), x.size(3), w.size(0), w.size(2), w.size(3)};
    for (int64_t v : e)
        if (v < 1 || v > INT32_MAX) return false;
    d->n = (int32_t)e[0]; d->c = (int32_t)e[1]; d->h = (int32_t)e[2]; d->w = (int32_t)e[3];
    d->k = (int32_t)e[4]; d->r = (int32_t)e[5]; d->s = (int32_t)e[6];
    if (!extent_pair(stride, 1, &d->stride_h, &d->stride_w) || !extent_pair(pad, pad_default, &d->pad_h, &d->pad_w))
        return false;
    d->flags = flags;
    // what the output extents are computed from (the library validates the rest)
    return d->stride_h > 0 && d->stride_w > 0 && d->pad_h >= 0 && d->pad_w >= 0 && d->pad_h < 64 && d->pad_w < 64 &&
           known_dtype(x, &d->dtype);
}

int64_t out_extent(int64_t in, int32_t pad, int32_t taps, int32_t stride) { return (in + 2 * pad - taps) / stride + 1; }

// Memory for a launch on a stream of the caller's choice.  torch's allocator hands a block out again in
// the order of the stream it was allocated on: from the current stream's pool it could still be in use
// there when the launch writes it, and a workspace released on return would be the next allocation's
// while the launch works in it.  So it comes from the pool of the launch's stream; a result, which the
// caller goes on to use on the current stream, is marked as used there too.
class Allocator {
public:
    // `stream`: the call's argument (absent: the current stream), `handle`: what it stands for
    Allocator(const at::Tensor &x, PyObject *stream, void *handle)
        : device_(x.device()), chosen_(stream && stream != Py_None), handle_(handle) {}
    at::Tensor workspace(size_t bytes) const { return make({(int64_t)bytes}, at::kByte, false); }
    at::Tensor result(at::IntArrayRef shape, c10::ScalarType type) const { return make(shape, type, true); }

private:
    at::Tensor make(at::IntArrayRef shape, c10::ScalarType type, bool result) const
    {
        const at::TensorOptions options = at::TensorOptions().dtype(type).device(device_);
        if (!chosen_) return at::empty(shape, options);
        struct Restored {
            c10::hip::HIPStream current;
            ~Restored() { c10::hip::setCurrentHIPStream(current); }
        } restored{c10::hip::getCurrentHIPStream(device_.index())};
        if (restored.current.stream() == handle_) return at::empty(shape, options);
        c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal(static_cast<hipStream_t>(handle_), device_.index()));
        at::Tensor t = at::empty(shape, options);
        if (result) c10::hip::HIPCachingAllocator::recordStream(t.storage().data_ptr(), restored.current);
        return t;
    }
    c10::Device device_;
    bool chosen_;
    void *handle_;
};

// The tensor that receives the result: the caller's, or a new one.
at::Tensor result(const at::Tensor *given, const Allocator &memory, const at::Tensor &x, const tvg_conv_desc &d, int64_t k)
{
    if (given) return *given;
    return memory.result({d.n, k, out_extent(d.h, d.pad_h, d.r, d.stride_h), out_extent(d.w, d.pad_w, d.s, d.stride_w)},
                         x.scalar_type());
}

// Whether an output of the caller's holds the result.
bool holds_result(const at::Tensor *out, const at::Tensor &x, const tvg_conv_desc &d, int64_t k)
{
    if (!out) return true;
    const int64_t oh = out_extent(d.h, d.pad_h, d.r, d.stride_h), ow = out_extent(d.w, d.pad_w, d.s, d.stride_w);
    return dense_on_device(*out) && (oh < 1 || ow < 1 || bytes_of(out) >= (size_t)(d.n * k * oh * ow) * x.element_size());
}

// Whether a workspace of the caller's that is large enough to be used can be used.
bool usable(const at::Tensor *ws, size_t need) { return bytes_of(ws) < need || !need || dense_on_device(*ws); }

// The workspace to pass: the caller's if it is large enough, else a new one.
at::Tensor enough_workspace(const at::Tensor *given, size_t need, const Allocator &memory)
{
    return given && bytes_of(given) >= need ? *given : memory.workspace(need);
}

const float *floats(const at::Tensor *t) { return t ? static_cast<const float *>(t->data_ptr()) : nullptr; }
const void *data(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }

// conv2d_fused and dwconv2d_fused
PyObject *convolution(bool depthwise, const Spec &spec, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    return guarded([&]() -> PyObject * {
        PyObject *v[13];
        if (!parse(spec, args, nargs, kwnames, v)) return nullptr;
        if (depthwise) {               // no workspace argument: the later ones move up by one
            v[12] = v[11];
            v[11] = v[10];
            v[10] = nullptr;
        }
        const at::Tensor *x, *w, *scale, *shift, *bias, *residual, *out, *ws;
        bool relu, stream_out;
        tvg_conv_desc d;
        const char *where = depthwise ? "dwconv2d_fused" : "conv2d_fused";
        if (!THPVariable_CheckExact(v[0])) return fall_back(where, args, nargs, kwnames);
        const c10::ScalarType dtype = THPVariable_Unpack(v[0]).scalar_type();
        if (!plain_tensor(v[0], false, dtype, &x) || !plain_tensor(v[1], false, dtype, &w) ||
            !plain_tensor(v[2], false, at::kFloat, &scale) || !plain_tensor(v[3], false, at::kFloat, &shift) ||
            !plain_tensor(v[4], true, at::kFloat, &bias) || !plain_tensor(v[5], true, dtype, &residual) ||
            !flag(v[8], false, &relu) || !plain_buffer(v[9], &out) || !plain_buffer(v[10], &ws) ||
            !flag(v[12], false, &stream_out) ||
            !describe(*x, *w, v[6], v[7], depthwise ? 1 : 0,
                      (relu ? (uint32_t)TVG_RELU : 0u) | (stream_out ? (uint32_t)TVG_STREAM_OUT : 0u), &d) ||
            (!depthwise && w->size(1) != x->size(1)) || !holds_result(out, *x, d, d.k))
            return fall_back(where, args, nargs, kwnames);
        void *stream;
        if (!stream_handle(v[11], &stream)) return nullptr;
        size_t need = 0;
        if (!depthwise) {
            const tvg_status st = tvg_conv2d_workspace_size(&d, &need);
            if (st != TVG_OK) return raise_status(st, "tvg_conv2d_workspace_size");
            if (!usable(ws, need)) return fall_back(where, args, nargs, kwnames);
        } else {
            const tvg_status st = tvg_dwconv2d_workspace_size(&d, &need);      // validates the descriptor
            if (st != TVG_OK) return fall_back(where, args, nargs, kwnames);
        }
        const Allocator memory(*x, v[11], stream);
        at::Tensor y = result(out, memory, *x, d, d.k);
        at::Tensor scratch;
        if (need) scratch = enough_workspace(ws, need, memory);
        else if (ws) scratch = *ws;
        void *scratch_ptr = scratch.defined() ? scratch.data_ptr() : nullptr;
        const size_t scratch_bytes = scratch.defined() ? bytes_of(&scratch) : 0;
        void *yp = y.data_ptr();
        const void *xp = data(x), *wp = data(w), *rp = data(residual);
        const float *sp = floats(scale), *hp = floats(shift), *bp = floats(bias);
        const tvg_status st = without_gil([&] {
            return (depthwise ? tvg_dwconv2d_fused : tvg_conv2d_fused)(&d, xp, wp, sp, hp, bp, rp, yp, scratch_ptr,
                                                                      scratch_bytes, stream);
        });
        if (st != TVG_OK) return raise_status(st, depthwise ? "tvg_dwconv2d_fused" : "tvg_conv2d_fused");
        if (out) {
            Py_INCREF(v[9]);
            return v[9];
        }
        return THPVariable_Wrap(std::move(y));
    });
}

PyObject *py_conv2d_fused(ARGS) { return convolution(false, conv2d_fused_spec, args, nargs, kwnames); }
PyObject *py_dwconv2d_fused(ARGS) { return convolution(true, dwconv2d_fused_spec, args, nargs, kwnames); }

PyObject *py_dwpw_fused(ARGS)
{
    return guarded([&]() -> PyObject * {
        PyObject *v[17];
        if (!parse(dwpw_fused_spec, args, nargs, kwnames, v)) return nullptr;
        const at::Tensor *x, *wd, *scd, *shd, *wp, *scp, *shp, *bias, *residual, *out, *ws;
        bool relu_dw, relu_pw, stream_out, one_kernel;
        tvg_conv_desc d;
        if (!THPVariable_CheckExact(v[0])) return fall_back("dwpw_fused", args, nargs, kwnames);
        const c10::ScalarType dtype = THPVariable_Unpack(v[0]).scalar_type();
        if (!plain_tensor(v[0], false, dtype, &x) || !plain_tensor(v[1], false, dtype, &wd) ||
            !plain_tensor(v[2], false, at::kFloat, &scd) || !plain_tensor(v[3], false, at::kFloat, &shd) ||
            !plain_tensor(v[4], false, dtype, &wp) || !plain_tensor(v[5], false, at::kFloat, &scp) ||
            !plain_tensor(v[6], false, at::kFloat, &shp) || !plain_tensor(v[7], true, at::kFloat, &bias) ||
            !plain_tensor(v[8], true, dtype, &residual) || !flag(v[10], true, &relu_dw) ||
            !flag(v[11], true, &relu_pw) || !plain_buffer(v[12], &out) || !plain_buffer(v[13], &ws) ||
            !flag(v[15], false, &stream_out) || !flag(v[16], false, &one_kernel) ||
            !describe(*x, *wd, v[9], nullptr, 1, relu_dw ? (uint32_t)TVG_RELU : 0u, &d) || wp->dim() != 4 ||
            wp->size(0) > INT32_MAX || wp->size(1) != x->size(1) || wp->size(2) != 1 || wp->size(3) != 1)
            return fall_back("dwpw_fused", args, nargs, kwnames);
        const int32_t k = (int32_t)wp->size(0);
        size_t need = 0;
        if (tvg_dwpw_workspace_size(&d, k, &need) != TVG_OK || !holds_result(out, *x, d, k) ||
            (!one_kernel && !usable(ws, need)))
            return fall_back("dwpw_fused", args, nargs, kwnames);
        void *stream;
        if (!stream_handle(v[14], &stream)) return nullptr;
        const Allocator memory(*x, v[14], stream);
        at::Tensor y = result(out, memory, *x, d, k);
        at::Tensor scratch;
        if (!one_kernel) scratch = enough_workspace(ws, need, memory);
        void *scratch_ptr = scratch.defined() ? scratch.data_ptr() : nullptr;
        const size_t scratch_bytes = scratch.defined() ? bytes_of(&scratch) : 0;
        void *yp = y.data_ptr();
        const uint32_t flags = (relu_pw ? (uint32_t)TVG_RELU : 0u) | (stream_out ? (uint32_t)TVG_STREAM_OUT : 0u);
        const void *xp = data(x), *wdp = data(wd), *wpp = data(wp), *rp = data(residual);
        const float *scdp = floats(scd), *shdp = floats(shd), *scpp = floats(scp), *shpp = floats(shp), *bp = floats(bias);
        const tvg_status st = without_gil([&] {
            return tvg_dwpw_fused(&d, k, flags, xp, wdp, scdp, shdp, wpp, scpp, shpp, bp, rp, yp, scratch_ptr,
                                  scratch_bytes, stream);
        });
        if (st != TVG_OK) return raise_status(st, "tvg_dwpw_fused");
        if (out) {
            Py_INCREF(v[12]);
            return v[12];
        }
        return THPVariable_Wrap(std::move(y));
    });
}

// setup(ConvDesc, TvgError, {name: Python implementation})
PyObject *py_setup(PyObject *, PyObject *args)
{
    PyObject *desc, *error, *fallback;
    if (!PyArg_ParseTuple(args, "OOO!", &desc, &error, &PyDict_Type, &fallback)) return nullptr;
    Py_INCREF(desc);
    Py_INCREF(error);
    Py_INCREF(fallback);
    Py_XDECREF(g_desc_type);
    Py_XDECREF(g_error_type);
    Py_XDECREF(g_fallback);
    g_desc_type = desc;
    g_error_type = error;
    g_fallback = fallback;
    Py_RETURN_NONE;
}

#define METHOD(fn, doc) {#fn, (PyCFunction)(void (*)(void))py_##fn, METH_FASTCALL | METH_KEYWORDS, doc}
PyMethodDef g_methods[] = {
    METHOD(tvg_conv2d_fused, "tvg_conv2d_fused($module, desc, x, w, scale, shift, bias, residual, y, workspace=None, workspace_bytes=0, stream=None)\n--\n\nThe C entry point (include/tvg.h); returns its status code."),
    METHOD(tvg_dwconv2d_fused, "tvg_dwconv2d_fused($module, desc, x, w, scale, shift, bias, residual, y, workspace=None, workspace_bytes=0, stream=None)\n--\n\nThe C entry point (include/tvg.h); returns its status code."),
    METHOD(tvg_conv2d_fused_static, "tvg_conv2d_fused_static($module, desc, x, w, scale, shift, bias, residual, y, stream=None)\n--\n\ntvg_conv2d_fused with the library's own static scratch instead of a workspace."),
    METHOD(tvg_conv2d_fused_dual, "tvg_conv2d_fused_dual($module, desc, k1, flags2, x, w, scale, shift, bias, residual1, y1, y2, stream=None)\n--\n\nTwo fused 3x3 convolutions of the same input in one launch (include/tvg.h)."),
    METHOD(tvg_conv2d_fused_prepacked, "tvg_conv2d_fused_prepacked($module, desc, x, packed, scale, shift, bias, residual, y, workspace, workspace_bytes, stream=None)\n--\n\nThe C entry point (include/tvg.h); returns its status code."),
    METHOD(tvg_dwpw_fused, "tvg_dwpw_fused($module, dw_desc, pw_k, pw_flags, x, w_dw, scale_dw, shift_dw, w_pw, scale_pw, shift_pw, bias_pw, residual, y, workspace=None, workspace_bytes=0, stream=None)\n--\n\nThe C entry point (include/tvg.h); returns its status code."),
    METHOD(tvg_maxpool2d_3x3s2, "tvg_maxpool2d_3x3s2($module, n, c, h, w, dtype, x, y, stream=None)\n--\n\nThe C entry point (include/tvg.h); returns its status code."),
    METHOD(conv2d_fused, "conv2d_fused($module, x, w, scale, shift, bias=None, residual=None, *, stride=1, pad=0, relu=False, out=None, workspace=None, stream=None, stream_out=False)\n--\n\ny = tail(conv2d(x, w)); allocates y (and the workspace when needed) with torch."),
    METHOD(dwconv2d_fused, "dwconv2d_fused($module, x, w, scale, shift, bias=None, residual=None, *, stride=1, pad=1, relu=False, out=None, stream=None, stream_out=False)\n--\n\ny = tail(depthwise conv2d(x, w)); allocates y with torch."),
    METHOD(dwpw_fused, "dwpw_fused($module, x, w_dw, scale_dw, shift_dw, w_pw, scale_pw, shift_pw, bias_pw=None, residual=None, *, stride=1, relu_dw=True, relu_pw=True, out=None, workspace=None, stream=None, stream_out=False, one_kernel=False)\n--\n\nMobileNet block (depthwise 3x3 + tail, 1x1 conv + tail) through tvg_dwpw_fused; allocates y with torch, and the workspace of the two-kernel form unless one_kernel asks for the form that needs none."),
    {"setup", py_setup, METH_VARARGS, "setup(ConvDesc, TvgError, fallbacks): called once by binding.py."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", "Native call path of the libtvg binding.", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

bool intern(const Spec &s)
{
    for (int i = 0; i < s.count; ++i) {
        s.interned[i] = PyUnicode_InternFromString(s.names[i]);
        if (!s.interned[i]) return false;
    }
    return true;
}

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    for (const Spec *s : {&tvg_conv2d_fused_spec, &tvg_dwconv2d_fused_spec, &tvg_conv2d_fused_static_spec,
                          &tvg_conv2d_fused_dual_spec, &tvg_conv2d_fused_prepacked_spec, &tvg_dwpw_fused_spec,
                          &tvg_maxpool2d_3x3s2_spec, &conv2d_fused_spec, &dwconv2d_fused_spec, &dwpw_fused_spec})
        if (!intern(*s)) return nullptr;
    return PyModule_Create(&g_module);
}
