// Argument marshalling between Python and the C ABI (include/hq.h): checks of the tensors, allocation of the
// results, PyTorch's current stream.  No arithmetic and no device code.
//
// Why native: interpreted, a call spent about 11 us on attribute look-ups, checks and the foreign-function layer
// before its kernel was launched - more than most of the kernels take; here it is about 4 us, most of it the launch.
// (Two calls back to back on small layers: 23 .. 24 us a layer before, 9.8 .. 10.4 us with this; linear
// 8192 x 384 -> 1152: 23.4 -> 15.1 us, bound by its kernels.)
//
// The entry points of the library are handed over as addresses (bind), so that the library is loaded in one place.
#include <Python.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/EmptyTensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>

#include <initializer_list>
#include <string>

#include "hq.h"

// (build.py looks for this text in the file)
extern "C" __attribute__((used, visibility("default"))) const char hq_marshal_built_for[] = HQ_BUILT_FOR;

namespace {

// ---- the library ------------------------------------------------------------------------------------------
#define HQ_ENTRY_POINTS(X)                                                                                          \
    X(hq_status_string) X(hq_quantize_weights) X(hq_act_hadamard_quant) X(hq_int_linear) X(hq_int_conv2d)            \
    X(hq_act_hadamard_quant_static) X(hq_int_linear_static) X(hq_int_conv2d_static) X(hq_quantize_weights_single)    \
    X(hq_int_linear_single) X(hq_act_hadamard_quant_width) X(hq_int_conv2d_width) X(hq_int_linear_i8)                \
    X(hq_int_conv2d_i8) X(hq_act_hadamard_quant_i8) X(hq_act_quant_int_conv2d) X(hq_act_quant_int_linear)

struct Library {
#define X(name) decltype(&::name) name;
    HQ_ENTRY_POINTS(X)
#undef X
} lib;
PyObject *error_class = nullptr;   // HqError(fn, code, text)

// ---- errors -----------------------------------------------------------------------------------------------
struct PythonError {};   // the interpreter's error indicator is set

[[noreturn]] void refuse(const std::string &text) {
    PyErr_SetString(PyExc_ValueError, text.c_str());
    throw PythonError();
}

void check(const char *fn, hq_status st) {
    if (st == HQ_OK) return;
    PyObject *e = PyObject_CallFunction(error_class, "sis", fn, static_cast<int>(st), lib.hq_status_string(st));
    if (e) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    }
    throw PythonError();
}

// The library only enqueues work; other threads may run meanwhile.  Its arguments are values: all that can fail (sizes that do
// not fit, storage without memory, the stream) is evaluated by the caller, with the interpreter's lock held.
struct Unlocked {
    PyThreadState *const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class... Parameters, class... Values>
hq_status call(hq_status (*f)(Parameters...), Values... values) {
    const Unlocked unlocked;
    return f(values...);
}

// ---- arguments --------------------------------------------------------------------------------------------
struct Args {
    PyObject *const *v;
    Py_ssize_t n, at = 0;
    PyObject *next() {
        if (at >= n) {
            PyErr_SetString(PyExc_TypeError, "too few arguments");
            throw PythonError();
        }
        return v[at++];
    }
    int integer() {
        const long x = PyLong_AsLong(next());
        if (x == -1 && PyErr_Occurred()) throw PythonError();
        if (x > 0x7FFFFFFFL || x < -0x7FFFFFFFL) refuse("an integer argument does not fit 32 bits");
        return static_cast<int>(x);
    }
    at::ScalarType dtype() {
        PyObject *o = next();
        if (!THPDtype_Check(o)) {
            PyErr_SetObject(PyExc_KeyError, o);
            throw PythonError();
        }
        return reinterpret_cast<THPDtype *>(o)->scalar_type;
    }
    bool none() const { return at < n && v[at] == Py_None; }
    // a tensor; must be one
    const at::Tensor &tensor(const char *name) {
        PyObject *o = next();
        if (!THPVariable_Check(o)) {
            PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
            throw PythonError();
        }
        return THPVariable_Unpack(o);
    }
    // contiguous, on the device
    const at::Tensor &device(const char *name) {
        const at::Tensor &t = tensor(name);
        if (!t.is_cuda() || !t.is_contiguous()) refuse(std::string(name) + " must be a contiguous device tensor");
        return t;
    }
    const at::Tensor &codes(at::ScalarType dt, const char *name) {
        const at::Tensor &t = device(name);
        if (t.scalar_type() != dt)
            refuse(std::string(name) + " must hold " + (dt == at::kByte ? "torch.uint8" : "torch.int8") + " codes");
        return t;
    }
    // an optional vector: exactly n elements of dt; the pointer, or null for None
    const void *vec(int64_t count, at::ScalarType dt, const char *name) {
        if (none()) {
            next();
            return nullptr;
        }
        const at::Tensor &t = tensor(name);
        if (!t.is_cuda() || !t.is_contiguous() || t.scalar_type() != dt || t.numel() != count)
            refuse(std::string(name) + " must be a contiguous device tensor of " + c10::toString(dt) + " with " +
                   std::to_string(count) + " elements");
        return t.const_data_ptr();
    }
    // one float32 on the device
    const float *scalar() {
        if (none()) refuse("x_scale must be a device tensor holding one float32");
        const at::Tensor &t = tensor("x_scale");
        if (!t.is_cuda() || t.scalar_type() != at::kFloat || t.numel() != 1)
            refuse("x_scale must be a device tensor holding one float32");
        return static_cast<const float *>(t.const_data_ptr());
    }
};

const float *f32(const void *p) { return static_cast<const float *>(p); }
const uint8_t *u8(const at::Tensor &t) { return static_cast<const uint8_t *>(t.const_data_ptr()); }

hq_dtype hq_type(at::ScalarType dt) {
    switch (dt) {
        case at::kHalf: return HQ_F16;
        case at::kFloat: return HQ_F32;
        case at::kInt: return HQ_I32;
        default:
            PyErr_SetString(PyExc_KeyError, c10::toString(dt));
            throw PythonError();
    }
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

at::Tensor empty(at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like) {
    return at::detail::empty_cuda(shape, dt, like.device(), std::nullopt);
}

// A caller's result buffer (the argument `o`; must hold exactly the result) or a new one.
at::Tensor result(PyObject *o, at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like) {
    if (o == Py_None) return empty(shape, dt, like);
    if (!THPVariable_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "out must be a tensor");
        throw PythonError();
    }
    const at::Tensor &t = THPVariable_Unpack(o);
    int64_t count = 1;
    for (const int64_t d : shape) count *= d;
    if (!t.is_cuda() || t.scalar_type() != dt || t.numel() != count || !t.is_contiguous())
        refuse(std::string("out must be a contiguous device tensor of ") + c10::toString(dt) + " with " +
               std::to_string(count) + " elements");
    return t;
}

// out = None or a pair of buffers (any sequence of them)
struct Pair {
    PyObject *a = Py_None, *b = Py_None;
    explicit Pair(PyObject *o) {
        if (o == Py_None) return;
        owned = true;
        a = PySequence_GetItem(o, 0);
        b = a ? PySequence_GetItem(o, 1) : nullptr;
        if (!b) {
            Py_XDECREF(a);
            throw PythonError();
        }
    }
    ~Pair() {
        if (!owned) return;
        Py_DECREF(a);
        Py_DECREF(b);
    }
    Pair(const Pair &) = delete;

private:
    bool owned = false;
};

using Shape = c10::SmallVector<int64_t, 6>;

Shape with_last(const at::Tensor &t, int64_t last) {
    Shape s(t.sizes().begin(), t.sizes().end());
    s.back() = last;
    return s;
}
Shape without_last(const at::Tensor &t) { return Shape(t.sizes().begin(), t.sizes().end() - 1); }

PyObject *wrap(const at::Tensor &t) { return THPVariable_Wrap(t); }
PyObject *wrap(const at::Tensor &a, const at::Tensor &b) {
    PyObject *pa = THPVariable_Wrap(a), *pb = THPVariable_Wrap(b);
    PyObject *p = pa && pb ? PyTuple_Pack(2, pa, pb) : nullptr;
    Py_XDECREF(pa);
    Py_XDECREF(pb);
    return p;
}

// The library takes sizes of 32 bits (but for the rows of a matrix).
void expect_32bit(std::initializer_list<int64_t> sizes) {
    for (const int64_t v : sizes)
        if (v > 0x7FFFFFFFLL) refuse("a size does not fit 32 bits");
}
int narrow(int64_t v) { return static_cast<int>(v); }

void expect_dims(const at::Tensor &t, int64_t dims, const char *text) {
    if (t.dim() != dims) refuse(text);
}

struct ConvOut {
    int64_t h, w;
};
ConvOut conv_out(int64_t h, int64_t w, int ksize, int stride, int pad) {
    if (stride < 1 || pad < 0 || ksize < 1) refuse("bad convolution geometry");
    // (rounded down, as for positive sizes; a window larger than the padded image is refused by the library)
    auto out = [&](int64_t n) {
        const int64_t d = n + int64_t{2} * pad - ksize;
        return (d >= 0 ? d / stride : -((-d + stride - 1) / stride)) + 1;
    };
    return {out(h), out(w)};
}
void expect_result(const ConvOut &o) {
    if (o.h < 0 || o.w < 0) refuse("bad convolution geometry");
}
int padding(Args &a, int ksize) {
    if (a.none()) {
        a.next();
        return (ksize - 1) / 2;
    }
    return a.integer();
}

// ---- calls: arguments in the order of the functions of binding.py -----------------------------------------------
PyObject *quantize_weights(Args a) {
    const at::Tensor &w = a.device("w");
    const int block = a.integer(), bits = a.integer();
    expect_dims(w, 3, "w must be [n_out, taps, k_in]");
    const int64_t n = w.size(0), taps = w.size(1), k = w.size(2);
    expect_32bit({n, taps, k});
    const at::Tensor wq = empty({n, taps, bits == 8 ? k : k / 2}, bits == 8 ? at::kChar : at::kByte, w);
    const at::Tensor ws = empty({n}, at::kFloat, w);
    const hq_dtype dt = hq_type(w.scalar_type());
    check("hq_quantize_weights", call(lib.hq_quantize_weights, w.const_data_ptr(), dt, narrow(n), narrow(taps),
                                      narrow(k), block, bits, static_cast<uint8_t *>(wq.data_ptr()),
                                      static_cast<float *>(ws.data_ptr()), stream()));
    return wrap(wq, ws);
}

PyObject *act_hadamard_quant(Args a) {
    const at::Tensor &x = a.device("x");
    const int block = a.integer(), bits = a.integer();
    const Pair out(a.next());
    if (x.dim() < 1) refuse("x must have a channel axis");
    const int64_t k = x.size(-1), m = k ? x.numel() / k : 0;
    expect_32bit({k});
    const at::Tensor xq = result(out.a, with_last(x, bits == 8 ? k : k / 2), bits == 8 ? at::kChar : at::kByte, x);
    const at::Tensor xs = result(out.b, without_last(x), at::kFloat, x);
    const hq_dtype dt = hq_type(x.scalar_type());
    check("hq_act_hadamard_quant", call(lib.hq_act_hadamard_quant, x.const_data_ptr(), dt, m, narrow(k), block, bits,
                                        static_cast<uint8_t *>(xq.data_ptr()), static_cast<float *>(xs.data_ptr()),
                                        stream()));
    return wrap(xq, xs);
}

PyObject *act_hadamard_quant_i8(Args a) {
    const at::Tensor &x = a.device("x");
    const int block = a.integer(), bits = a.integer();
    if (x.dim() < 1) refuse("x must have a channel axis");
    const int64_t k = x.size(-1), m = k ? x.numel() / k : 0;
    expect_32bit({k});
    const at::Tensor xq = empty(x.sizes(), at::kChar, x);
    const at::Tensor xs = empty(without_last(x), at::kFloat, x);
    const hq_dtype dt = hq_type(x.scalar_type());
    check("hq_act_hadamard_quant_i8", call(lib.hq_act_hadamard_quant_i8, x.const_data_ptr(), dt, m, narrow(k), block,
                                           bits, static_cast<int8_t *>(xq.data_ptr()),
                                           static_cast<float *>(xs.data_ptr()), stream()));
    return wrap(xq, xs);
}

PyObject *act_hadamard_quant_static(Args a) {
    const at::Tensor &x = a.device("x");
    PyObject *scale = a.next();
    const int block = a.integer(), bits = a.integer();
    if (x.dim() < 1) refuse("x must have a channel axis");
    const int64_t k = x.size(-1), m = k ? x.numel() / k : 0;
    expect_32bit({k});
    const at::Tensor xq = result(a.next(), with_last(x, k / 2), at::kByte, x);
    Args one{&scale, 1};
    const float *s = one.scalar();
    const hq_dtype dt = hq_type(x.scalar_type());
    check("hq_act_hadamard_quant_static", call(lib.hq_act_hadamard_quant_static, x.const_data_ptr(), dt, m, narrow(k),
                                               block, bits, s, static_cast<uint8_t *>(xq.data_ptr()), stream()));
    return wrap(xq);
}

// hq_int_linear, hq_int_linear_static, hq_int_linear_i8
enum class Scales { dynamic, fixed };

template <class Code>
PyObject *int_linear(Args &a, const char *fn, hq_status (*f)(const Code *, const float *, const Code *, const float *, const void *,
                                                              int64_t, int, int, void *, hq_dtype, void *), Scales scales) {
    constexpr bool bytes = std::is_same<Code, int8_t>::value;   // one code per byte
    constexpr at::ScalarType code = bytes ? at::kChar : at::kByte;
    const at::Tensor &xq = a.codes(code, "xq");
    PyObject *x_scale = a.next();
    const at::Tensor &wq = a.codes(code, "wq");
    PyObject *w_scale = a.next(), *bias = a.next();
    const at::ScalarType ydt = a.dtype();
    expect_dims(xq, 2, "xq must be [m, k]");
    const int64_t m = xq.size(0), kb = xq.size(1), n = wq.dim() ? wq.size(0) : 0;
    expect_32bit({n, bytes ? kb : kb * 2});
    if (wq.numel() != n * kb) refuse("wq does not match xq in k");
    const void *sx = Args{&x_scale, 1}.vec(scales == Scales::fixed ? 1 : m, at::kFloat, "x_scale");
    const void *sw = Args{&w_scale, 1}.vec(n, at::kFloat, "w_scale");
    const void *b = Args{&bias, 1}.vec(n, ydt, "bias");
    const at::Tensor y = result(a.next(), {m, n}, ydt, xq);
    const hq_dtype dt = hq_type(ydt);
    check(fn, call(f, static_cast<const Code *>(xq.const_data_ptr()), f32(sx),
                   static_cast<const Code *>(wq.const_data_ptr()), f32(sw), b, m, narrow(n),
                   narrow(bytes ? kb : kb * 2), y.data_ptr(), dt, stream()));
    return wrap(y);
}
PyObject *linear(Args a) { return int_linear<uint8_t>(a, "hq_int_linear", lib.hq_int_linear, Scales::dynamic); }
PyObject *linear_static(Args a) { return int_linear<uint8_t>(a, "hq_int_linear_static", lib.hq_int_linear_static, Scales::fixed); }
PyObject *linear_i8(Args a) { return int_linear<int8_t>(a, "hq_int_linear_i8", lib.hq_int_linear_i8, Scales::dynamic); }

// hq_int_conv2d, hq_int_conv2d_static, hq_int_conv2d_i8
template <class Code>
PyObject *int_conv2d(Args &a, const char *fn,
                     hq_status (*f)(const Code *, const float *, const Code *, const float *, const void *, int, int, int, int,
                                    int, int, int, int, int, void *, hq_dtype, void *),
                     Scales scales) {
    constexpr bool bytes = std::is_same<Code, int8_t>::value;
    constexpr at::ScalarType code = bytes ? at::kChar : at::kByte;
    const at::Tensor &xq = a.codes(code, "xq");
    PyObject *x_scale = a.next();
    const at::Tensor &wq = a.codes(code, "wq");
    PyObject *w_scale = a.next(), *bias = a.next();
    const int ksize = a.integer(), stride = a.integer(), pad = padding(a, ksize);
    const at::ScalarType ydt = a.dtype();
    expect_dims(xq, 4, "xq must be [nb, h, w, c]");
    const int64_t nb = xq.size(0), h = xq.size(1), w = xq.size(2), cb = xq.size(3), n = wq.dim() ? wq.size(0) : 0;
    const int64_t taps = static_cast<int64_t>(ksize) * ksize;
    expect_32bit({nb, h, w, bytes ? cb : cb * 2, n});
    if (wq.numel() != n * taps * cb) refuse("wq does not match xq / ksize");
    const void *sx = Args{&x_scale, 1}.vec(scales == Scales::fixed ? 1 : nb * h * w, at::kFloat, "x_scale");
    const void *sw = Args{&w_scale, 1}.vec(n, at::kFloat, "w_scale");
    const void *b = Args{&bias, 1}.vec(n, ydt, "bias");
    const ConvOut o = conv_out(h, w, ksize, stride, pad);
    expect_result(o);
    Shape shape{nb, o.h, o.w};
    if (ydt == at::kInt && scales == Scales::dynamic && (!bytes || taps > 1)) shape.push_back(taps);   // per-tap sums
    shape.push_back(n);
    const at::Tensor y = result(a.next(), shape, ydt, xq);
    const hq_dtype dt = hq_type(ydt);
    check(fn, call(f, static_cast<const Code *>(xq.const_data_ptr()), f32(sx),
                   static_cast<const Code *>(wq.const_data_ptr()), f32(sw), b, narrow(nb), narrow(h), narrow(w),
                   narrow(bytes ? cb : cb * 2), narrow(n), ksize, ksize, stride, pad, y.data_ptr(), dt, stream()));
    return wrap(y);
}
PyObject *conv2d(Args a) { return int_conv2d<uint8_t>(a, "hq_int_conv2d", lib.hq_int_conv2d, Scales::dynamic); }
PyObject *conv2d_static(Args a) { return int_conv2d<uint8_t>(a, "hq_int_conv2d_static", lib.hq_int_conv2d_static, Scales::fixed); }
PyObject *conv2d_i8(Args a) { return int_conv2d<int8_t>(a, "hq_int_conv2d_i8", lib.hq_int_conv2d_i8, Scales::dynamic); }

PyObject *act_quant_conv2d(Args a) {
    const at::Tensor &x = a.device("x"), &wq = a.codes(at::kByte, "wq");
    PyObject *w_scale = a.next(), *bias = a.next();
    const int block = a.integer(), bits = a.integer(), ksize = a.integer(), stride = a.integer(), pad = padding(a, ksize);
    const at::ScalarType ydt = a.dtype();
    PyObject *out = a.next(), *codes = a.next();
    const Pair codes_out(codes);
    expect_dims(x, 4, "x must be [nb, h, w, c]");
    const int64_t nb = x.size(0), h = x.size(1), w = x.size(2), cin = x.size(3), n = wq.dim() ? wq.size(0) : 0;
    const int64_t taps = static_cast<int64_t>(ksize) * ksize;
    expect_32bit({nb, h, w, cin, n});
    if (wq.numel() != n * taps * (cin / 2)) refuse("wq does not match x / ksize");
    const void *sw = Args{&w_scale, 1}.vec(n, at::kFloat, "w_scale");
    const void *b = Args{&bias, 1}.vec(n, ydt, "bias");
    const ConvOut o = conv_out(h, w, ksize, stride, pad);
    expect_result(o);
    Shape shape{nb, o.h, o.w};
    if (ydt == at::kInt) shape.push_back(taps);
    shape.push_back(n);
    const at::Tensor y = result(out, shape, ydt, x);
    at::Tensor xq, sx;
    if (codes != Py_None) {
        xq = result(codes_out.a, {nb, h, w, cin / 2}, at::kByte, x);
        sx = result(codes_out.b, {nb, h, w}, at::kFloat, x);
    }
    const hq_dtype xdt = hq_type(x.scalar_type()), dt = hq_type(ydt);
    check("hq_act_quant_int_conv2d", call(lib.hq_act_quant_int_conv2d, x.const_data_ptr(), xdt, u8(wq), f32(sw), b,
                                          narrow(nb), narrow(h), narrow(w), narrow(cin), narrow(n), ksize, ksize,
                                          stride, pad, block, bits, y.data_ptr(), dt,
                                          xq.defined() ? static_cast<uint8_t *>(xq.data_ptr()) : nullptr,
                                          sx.defined() ? static_cast<float *>(sx.data_ptr()) : nullptr, stream()));
    return wrap(y);
}

PyObject *act_quant_linear(Args a) {
    const at::Tensor &x = a.device("x"), &wq = a.codes(at::kByte, "wq");
    PyObject *w_scale = a.next(), *bias = a.next();
    const int block = a.integer(), bits = a.integer();
    const at::ScalarType ydt = a.dtype();
    PyObject *out = a.next(), *codes = a.next();
    const Pair codes_out(codes);
    if (x.dim() < 1) refuse("x must have a channel axis");
    const int64_t k = x.size(-1), m = k ? x.numel() / k : 0, n = wq.dim() ? wq.size(0) : 0;
    expect_32bit({n, k});
    if (wq.numel() != n * (k / 2)) refuse("wq does not match x");
    const void *sw = Args{&w_scale, 1}.vec(n, at::kFloat, "w_scale");
    const void *b = Args{&bias, 1}.vec(n, ydt, "bias");
    const at::Tensor y = result(out, with_last(x, n), ydt, x);
    at::Tensor xq, sx;
    if (codes != Py_None) {
        xq = result(codes_out.a, with_last(x, k / 2), at::kByte, x);
        sx = result(codes_out.b, without_last(x), at::kFloat, x);
    }
    const hq_dtype xdt = hq_type(x.scalar_type()), dt = hq_type(ydt);
    check("hq_act_quant_int_linear", call(lib.hq_act_quant_int_linear, x.const_data_ptr(), xdt, u8(wq), f32(sw), b, m,
                                          narrow(n), narrow(k), block, bits, y.data_ptr(), dt,
                                          xq.defined() ? static_cast<uint8_t *>(xq.data_ptr()) : nullptr,
                                          sx.defined() ? static_cast<float *>(sx.data_ptr()) : nullptr, stream()));
    return wrap(y);
}

PyObject *quantize_weights_single(Args a) {
    const at::Tensor &w = a.device("w");
    const int block = a.integer(), bits = a.integer();
    expect_dims(w, 2, "w must be [n_out, k_in]");
    const int64_t n = w.size(0), k = w.size(1);
    expect_32bit({n, k});
    const at::Tensor wq3 = empty({n, 3, k / 2}, at::kByte, w);
    const at::Tensor ws = empty({n}, at::kFloat, w);
    const hq_dtype dt = hq_type(w.scalar_type());
    check("hq_quantize_weights_single", call(lib.hq_quantize_weights_single, w.const_data_ptr(), dt, narrow(n),
                                             narrow(k), block, bits, static_cast<uint8_t *>(wq3.data_ptr()),
                                             static_cast<float *>(ws.data_ptr()), stream()));
    return wrap(wq3, ws);
}

PyObject *linear_single(Args a) {
    const at::Tensor &xq = a.codes(at::kByte, "xq");
    PyObject *x_scale = a.next();
    const at::Tensor &wq3 = a.codes(at::kByte, "wq3");
    PyObject *w_scale = a.next(), *bias = a.next();
    const int block = a.integer();
    const at::ScalarType ydt = a.dtype();
    expect_dims(xq, 2, "xq must be [m, k]");
    const int64_t m = xq.size(0), kb = xq.size(1), n = wq3.dim() ? wq3.size(0) : 0;
    expect_32bit({n, kb * 2});
    if (wq3.numel() != n * 3 * kb) refuse("wq3 does not match xq in k");
    const void *sx = Args{&x_scale, 1}.vec(m, at::kFloat, "x_scale");
    const void *sw = Args{&w_scale, 1}.vec(n, at::kFloat, "w_scale");
    const void *b = Args{&bias, 1}.vec(n, ydt, "bias");
    Shape shape{m, n};
    if (ydt == at::kInt) shape = {m, 3, n};
    const at::Tensor y = result(a.next(), shape, ydt, xq);
    const hq_dtype dt = hq_type(ydt);
    check("hq_int_linear_single", call(lib.hq_int_linear_single, u8(xq), f32(sx), u8(wq3), f32(sw), b, m, narrow(n),
                                       narrow(kb * 2), block, y.data_ptr(), dt, stream()));
    return wrap(y);
}

PyObject *act_hadamard_quant_width(Args a) {
    const at::Tensor &x = a.device("x");
    const float *scale = a.scalar();
    const int block = a.integer(), bits = a.integer();
    expect_dims(x, 4, "x must be [N, H, W, C]");
    const int64_t nb = x.size(0), h = x.size(1), w = x.size(2), c = x.size(3);
    expect_32bit({nb, h, w, c});
    const at::Tensor xu3 = result(a.next(), {3, nb, h, w, c / 2}, at::kByte, x);
    const hq_dtype dt = hq_type(x.scalar_type());
    check("hq_act_hadamard_quant_width", call(lib.hq_act_hadamard_quant_width, x.const_data_ptr(), dt, narrow(nb),
                                              narrow(h), narrow(w), narrow(c), block, bits, scale,
                                              static_cast<uint8_t *>(xu3.data_ptr()), stream()));
    return wrap(xu3);
}

PyObject *conv2d_width(Args a) {
    const at::Tensor &xu3 = a.codes(at::kByte, "xu3");
    PyObject *x_scale = a.next();
    const at::Tensor &wq = a.codes(at::kByte, "wq");
    PyObject *w_scale = a.next(), *bias = a.next();
    const int block = a.integer();
    const at::ScalarType ydt = a.dtype();
    PyObject *out = a.next();
    const int stride = a.integer();
    if (xu3.dim() != 5 || xu3.size(0) != 3) refuse("xu3 must be [3, N, H, W, Cin/2]");
    const int64_t nb = xu3.size(1), h = xu3.size(2), w = xu3.size(3), kb = xu3.size(4), n = wq.dim() ? wq.size(0) : 0;
    expect_32bit({nb, h, w, kb * 2, n});
    if (wq.numel() != n * 9 * kb) refuse("wq does not match xu3 in Cin or is not a 3x3 kernel");
    const void *sx = Args{&x_scale, 1}.vec(1, at::kFloat, "x_scale");
    const void *sw = Args{&w_scale, 1}.vec(n, at::kFloat, "w_scale");
    const void *b = Args{&bias, 1}.vec(n, ydt, "bias");
    const ConvOut o = conv_out(h, w, 3, stride, 1);
    expect_result(o);
    const at::Tensor y = result(out, {nb, o.h, o.w, n}, ydt, xu3);
    const hq_dtype dt = hq_type(ydt);
    check("hq_int_conv2d_width", call(lib.hq_int_conv2d_width, u8(xu3), f32(sx), u8(wq), f32(sw), b, narrow(nb),
                                      narrow(h), narrow(w), narrow(kb * 2), narrow(n), 3, 3, stride, 1, block,
                                      y.data_ptr(), dt, stream()));
    return wrap(y);
}

// ---- module -----------------------------------------------------------------------------------------------------
template <PyObject *(*F)(Args)>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    try {
        return F(Args{args, n});
    } catch (const PythonError &) {
        return nullptr;
    } catch (const std::exception &e) {   // (an allocation that failed)
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// bind({name: address}, HqError)
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 2 || !PyDict_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "bind(addresses, error class)");
        return nullptr;
    }
    Library l{};
#define X(name)                                                                   \
    {                                                                             \
        PyObject *v = PyDict_GetItemString(args[0], #name);                       \
        void *p = v ? PyLong_AsVoidPtr(v) : nullptr;                              \
        if (!p) {                                                                 \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);        \
            return nullptr;                                                       \
        }                                                                         \
        l.name = reinterpret_cast<decltype(l.name)>(p);                           \
    }
    HQ_ENTRY_POINTS(X)
#undef X
    lib = l;
    Py_INCREF(args[1]);
    Py_XDECREF(error_class);
    error_class = args[1];
    Py_RETURN_NONE;
}

#define HQ_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<f>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    HQ_METHOD(quantize_weights), HQ_METHOD(act_hadamard_quant), HQ_METHOD(act_hadamard_quant_i8),
    HQ_METHOD(act_hadamard_quant_static), HQ_METHOD(linear), HQ_METHOD(linear_static), HQ_METHOD(linear_i8),
    HQ_METHOD(conv2d), HQ_METHOD(conv2d_static), HQ_METHOD(conv2d_i8),
    HQ_METHOD(act_quant_conv2d), HQ_METHOD(act_quant_linear), HQ_METHOD(quantize_weights_single), HQ_METHOD(linear_single),
    HQ_METHOD(act_hadamard_quant_width), HQ_METHOD(conv2d_width),
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Argument marshalling of the HIP library.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
