// The entry points of include/q8t.h that a training step calls, as functions of a Python module over torch tensors: argument
// checks, output tensors, scratch memory and the stream in native code.  binding.py wraps every function here under its public
// name, arguments and defaults and documents it; the calls that a step makes once or not at all stay on ctypes there.
//
// Why: a step of small layers waits for the host.  Through ctypes and torch's Python functions a call cost its launches (2.6 us
// each) and as much again or more: 1.6 us per output tensor, 1.5 for the argument conversion, 0.8 for the scratch memory.  Host
// time of a call, us, before / now: quantize 9.2 / 5.4, quantize_bifurcate 13.3 / 7.3, qgemm 7.6 / 4.3, a small convolution with
// statistics 19.6 / 15.4, Range BN + ReLU backward with codes 23.8 / 16.0; the step of a 64x256x128 FC layer 78.6 / 42.2.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "q8t.h"

namespace {

PyObject *g_workspace = nullptr;   // binding.workspace(nbytes, device)
PyObject *g_cache = nullptr;       // its buffers, {(device, stream): tensor}
PyObject *g_error = nullptr;       // binding.Q8TError(code, name)

struct Raised {};   // a Python exception is set

[[noreturn]] void raise(PyObject *type, const char *text)
{
    PyErr_SetString(type, text);
    throw Raised();
}
void require(bool ok)
{
    if (!ok) raise(PyExc_AssertionError, "");
}

struct Ref {   // owned reference
    PyObject *o;
    explicit Ref(PyObject *p) : o(p)
    {
        if (!p) throw Raised();
    }
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

struct Unlocked {   // the interpreter runs other threads meanwhile
    PyThreadState *s = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(s); }
};

// ---- arguments ----
const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "q8t: a tensor is expected");
    return THPVariable_Unpack(o);
}
const at::Tensor &dev(PyObject *o)
{
    const at::Tensor &t = tensor(o);
    if (!t.is_cuda()) raise(PyExc_ValueError, "q8t works on device tensors only (got a CPU tensor)");
    if (!t.is_contiguous()) raise(PyExc_ValueError, "q8t needs contiguous tensors");
    return t;
}
template <class T>
T *ptr(PyObject *o)
{
    return o == Py_None ? nullptr : static_cast<T *>(tensor(o).data_ptr());
}
template <class T>
T *ptr(const at::Tensor &t)
{
    return t.defined() ? static_cast<T *>(t.data_ptr()) : nullptr;
}
bool truth(PyObject *o)
{
    const int r = PyObject_IsTrue(o);
    if (r < 0) throw Raised();
    return r != 0;
}
int integer(PyObject *o, bool convert = false)   // convert: int(o)
{
    const Ref n(convert ? PyNumber_Long(o) : PyNumber_Index(o));
    const long v = PyLong_AsLong(n.o);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    if (v != (int)v) raise(PyExc_OverflowError, "q8t: integer argument out of range");
    return (int)v;
}
uint64_t seed(PyObject *o)   // int(o) modulo 2^64
{
    const Ref n(PyNumber_Long(o));
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(n.o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Raised();
    return v;
}
float real(PyObject *o)   // float(o)
{
    const Ref f(PyNumber_Float(o));
    return (float)PyFloat_AS_DOUBLE(f.o);
}
struct Desc {   // binding.ConvDesc
    Py_buffer b;
    explicit Desc(PyObject *o)
    {
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE)) throw Raised();
        if (b.len != (Py_ssize_t)sizeof(q8t_conv_desc)) {
            PyBuffer_Release(&b);
            raise(PyExc_TypeError, "q8t: a ConvDesc is expected");
        }
    }
    ~Desc() { PyBuffer_Release(&b); }
    Desc(const Desc &) = delete;
    const q8t_conv_desc *operator->() const { return static_cast<const q8t_conv_desc *>(b.buf); }
    const q8t_conv_desc *get() const { return static_cast<const q8t_conv_desc *>(b.buf); }
    int64_t P() const { return out(get()->H, get()->R); }
    int64_t Q() const { return out(get()->W, get()->S); }

  private:
    int64_t out(int64_t in, int64_t f) const   // the quotient is rounded down, as in Python
    {
        const int64_t n = in + 2 * (int64_t)get()->pad - f, s = get()->stride;
        if (s == 0) raise(PyExc_ZeroDivisionError, "integer division or modulo by zero");
        return n / s - (n % s != 0 && (n < 0) != (s < 0)) + 1;
    }
};
void shape_is(const at::Tensor &t, std::initializer_list<int64_t> want)
{
    require(t.sizes().equals(at::IntArrayRef(want.begin(), want.size())));
}
struct Plane {   // N, C, H, W of a tensor
    int N, C, H, W;
    explicit Plane(const at::Tensor &t)
    {
        if (t.dim() != 4) raise(PyExc_ValueError, "q8t: a tensor of four dimensions is expected");
        N = dim(t.size(0));
        C = dim(t.size(1));
        H = dim(t.size(2));
        W = dim(t.size(3));
    }
    static int dim(int64_t v)
    {
        if (v != (int)v) raise(PyExc_OverflowError, "q8t: dimension out of range");
        return (int)v;
    }
};

// ---- outputs and scratch memory ----
at::Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like)
{
    const Unlocked u;
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}
at::Tensor make_params(const at::Tensor &like) { return make({6}, at::kInt, like); }
at::Tensor same(const at::Tensor &like)
{
    const Unlocked u;
    return at::empty_like(like);
}
// the tensor handed in, or a new one
template <class F>
at::Tensor given(PyObject *o, F fresh)
{
    return o == Py_None ? fresh() : tensor(o);
}
struct Scratch {
    PyObject *o = nullptr;
    Scratch(PyObject *ws, size_t need, PyObject *like, bool none_if_zero = false)
    {
        if (ws != Py_None) {
            Py_INCREF(ws);
            o = ws;
            return;
        }
        if (none_if_zero && need == 0) return;
        const Ref device(PyObject_GetAttrString(like, "device"));
        const uintptr_t stream = reinterpret_cast<uintptr_t>(c10::hip::getCurrentHIPStream().stream());
        // a kept buffer of the stream; a call that is being captured and one that needs a larger buffer go through Python
        if (!stream || c10::hip::currentStreamCaptureStatusMayInitCtx() == c10::hip::CaptureStatus::None) {
            const Ref handle(PyLong_FromUnsignedLongLong(stream)), key(PyTuple_Pack(2, device.o, handle.o));
            PyObject *hit = PyDict_GetItemWithError(g_cache, key.o);
            if (!hit && PyErr_Occurred()) throw Raised();
            if (hit && (size_t)tensor(hit).numel() >= need) {
                Py_INCREF(hit);
                o = hit;
                return;
            }
        }
        const Ref n(PyLong_FromSize_t(need));
        o = PyObject_CallFunctionObjArgs(g_workspace, n.o, device.o, nullptr);
        if (!o) throw Raised();
    }
    ~Scratch() { Py_XDECREF(o); }
    Scratch(const Scratch &) = delete;
    void *get() const { return o ? tensor(o).data_ptr() : nullptr; }
};

template <class F>
void run(const char *name, F call)
{
    void *stream = static_cast<void *>(c10::hip::getCurrentHIPStream().stream());
    int rc;
    {
        const Unlocked u;
        rc = call(stream);
    }
    if (rc == Q8T_OK) return;
    const Ref e(PyObject_CallFunction(g_error, "is", rc, name));
    PyErr_SetObject(g_error, e.o);
    throw Raised();
}

// ---- results: a tuple of tensors, None where one is not defined ----
PyObject *wrap(const at::Tensor &t)
{
    if (!t.defined()) Py_RETURN_NONE;
    PyObject *o = THPVariable_Wrap(t);
    if (!o) throw Raised();
    return o;
}
PyObject *results(std::initializer_list<const at::Tensor *> ts)
{
    PyObject *r = PyTuple_New((Py_ssize_t)ts.size());
    if (!r) throw Raised();
    Py_ssize_t i = 0;
    for (const at::Tensor *t : ts) {
        PyObject *o = nullptr;
        try {
            o = wrap(*t);
        } catch (...) {
            Py_DECREF(r);
            throw;
        }
        PyTuple_SET_ITEM(r, i++, o);
    }
    return r;
}

typedef PyObject *const *Argv;

// x, bits, stochastic, seed, q_out, qp_out, ws
PyObject *quantize(Argv a)
{
    const at::Tensor &x = dev(a[0]);
    const int64_t n = x.numel();
    const int bits = integer(a[1]), st = truth(a[2]);
    const uint64_t s = seed(a[3]);
    const at::Tensor q = given(a[4], [&] { return make(x.sizes(), bits <= 8 ? at::kChar : at::kShort, x); });
    const at::Tensor p = given(a[5], [&] { return make_params(x); });
    const Scratch ws(a[6], q8t_quantize_workspace_size(n), a[0]);
    run("q8t_quantize", [&, w = ws.get()](void *stream) {
        return q8t_quantize(ptr<float>(x), n, bits, st, s, ptr<void>(q), ptr<q8t_qparams>(p), w, stream);
    });
    return results({&q, &p});
}

// x, vmin_vmax, bits, stochastic, seed, q_out, qp_out
PyObject *quantize_with_range(Argv a)
{
    const at::Tensor &x = dev(a[0]), &r = dev(a[1]);
    const int bits = integer(a[2]), st = truth(a[3]);
    const uint64_t s = seed(a[4]);
    const at::Tensor q = given(a[5], [&] { return make(x.sizes(), bits <= 8 ? at::kChar : at::kShort, x); });
    const at::Tensor p = given(a[6], [&] { return make_params(x); });
    run("q8t_quantize_with_range", [&](void *stream) {
        return q8t_quantize_with_range(ptr<float>(x), x.numel(), bits, st, s, ptr<float>(r), ptr<void>(q), ptr<q8t_qparams>(p), stream);
    });
    return results({&q, &p});
}

// g, seed8, seed16, q8_out, qp8_out, q16_out, qp16_out, ws
PyObject *quantize_bifurcate(Argv a)
{
    const at::Tensor &g = dev(a[0]);
    const int64_t n = g.numel();
    const uint64_t s8 = seed(a[1]), s16 = seed(a[2]);
    const at::Tensor q8 = given(a[3], [&] { return make(g.sizes(), at::kChar, g); });
    const at::Tensor q16 = given(a[5], [&] { return make(g.sizes(), at::kShort, g); });
    const at::Tensor p8 = given(a[4], [&] { return make_params(g); }), p16 = given(a[6], [&] { return make_params(g); });
    const Scratch ws(a[7], q8t_quantize_workspace_size(n), a[0]);
    run("q8t_quantize_bifurcate", [&, w = ws.get()](void *stream) {
        return q8t_quantize_bifurcate(ptr<float>(g), n, s8, s16, ptr<int8_t>(q8), ptr<q8t_qparams>(p8), ptr<int16_t>(q16),
                                      ptr<q8t_qparams>(p16), w, stream);
    });
    return results({&q8, &p8, &q16, &p16});
}

// x, K, ws
PyObject *chunk_range(Argv a)
{
    const at::Tensor &x = dev(a[0]);
    const int64_t n = x.numel();
    const int K = integer(a[1], true);
    const at::Tensor out = make({2}, at::kFloat, x);
    const Scratch ws(a[2], q8t_chunk_range_workspace_size(n, K), a[0]);
    run("q8t_chunk_range", [&, w = ws.get()](void *stream) { return q8t_chunk_range(ptr<float>(x), n, K, ptr<float>(out), w, stream); });
    return wrap(out);
}

// a, pa, b, pb, want_acc, out, ws; which: 0 forward, 1 layer gradient, 2 weight gradient
template <int WHICH>
PyObject *qgemm(Argv a)
{
    const at::Tensor &x = dev(a[0]), &w = dev(a[2]);
    if (x.dim() != 2 || w.dim() != 2) raise(PyExc_ValueError, "q8t: matrices are expected");
    int M, N, K;
    if (WHICH == 0) {
        M = Plane::dim(x.size(0)), K = Plane::dim(x.size(1)), N = Plane::dim(w.size(1));
        require(w.size(0) == K);
    } else if (WHICH == 1) {
        M = Plane::dim(x.size(0)), N = Plane::dim(x.size(1)), K = Plane::dim(w.size(0));
        require(w.size(1) == N);
    } else {
        M = Plane::dim(x.size(0)), K = Plane::dim(x.size(1)), N = Plane::dim(w.size(1));
        require(w.size(0) == M && w.scalar_type() == at::kShort);
    }
    const int64_t rows = WHICH == 2 ? K : M, cols = WHICH == 1 ? K : N;
    at::Tensor acc;
    const at::Tensor y = given(a[5], [&] { return make({rows, cols}, at::kFloat, x); });
    if (truth(a[4])) acc = make({rows, cols}, WHICH == 2 ? at::kLong : at::kInt, x);
    const Scratch ws(a[6], q8t_qgemm_workspace_size(M, N, K, WHICH), a[0], true);
    const q8t_qparams *pa = ptr<q8t_qparams>(a[1]), *pb = ptr<q8t_qparams>(a[3]);
    run(WHICH == 0 ? "q8t_qgemm_fwd" : (WHICH == 1 ? "q8t_qgemm_dgrad" : "q8t_qgemm_wgrad"), [&, s = ws.get()](void *stream) {
        if (WHICH == 0)
            return q8t_qgemm_fwd(ptr<int8_t>(x), pa, ptr<int8_t>(w), pb, M, N, K, ptr<float>(y), ptr<int32_t>(acc), s, stream);
        if (WHICH == 1)
            return q8t_qgemm_dgrad(ptr<int8_t>(x), pa, ptr<int8_t>(w), pb, M, N, K, ptr<float>(y), ptr<int32_t>(acc), s, stream);
        return q8t_qgemm_wgrad(ptr<int8_t>(x), pa, ptr<int16_t>(w), pb, M, N, K, ptr<float>(y), ptr<int64_t>(acc), s, stream);
    });
    return results({&y, &acc});
}

// d, qx, px, qw, pw, want_acc, out, stats_out, ws, packed
PyObject *qconv_fwd_bn_stats(Argv a)
{
    const Desc d(a[0]);
    const at::Tensor &x = dev(a[1]), &w = dev(a[3]);
    shape_is(x, {d->N, d->C, d->H, d->W});
    shape_is(w, {d->K, d->C, d->R, d->S});
    at::Tensor acc;
    const at::Tensor y = given(a[6], [&] { return make({d->N, d->K, d.P(), d.Q()}, at::kFloat, x); });
    if (truth(a[5])) acc = make({d->N, d->K, d.P(), d.Q()}, at::kInt, x);
    const at::Tensor stats = given(a[7], [&] { return make({3, d->K}, at::kFloat, x); });
    const Scratch ws(a[8], q8t_qconv_fwd_bn_stats_workspace_size(d.get()), a[1]);
    const q8t_qparams *px = ptr<q8t_qparams>(a[2]), *pw = ptr<q8t_qparams>(a[4]);
    const void *packed = ptr<void>(a[9]);
    run(packed ? "q8t_qconv_fwd_bn_stats_packed" : "q8t_qconv_fwd_bn_stats", [&, s = ws.get()](void *stream) {
        if (packed)
            return q8t_qconv_fwd_bn_stats_packed(d.get(), ptr<int8_t>(x), px, ptr<int8_t>(w), pw, packed, ptr<float>(y), ptr<int32_t>(acc),
                                                 ptr<float>(stats), s, stream);
        return q8t_qconv_fwd_bn_stats(d.get(), ptr<int8_t>(x), px, ptr<int8_t>(w), pw, ptr<float>(y), ptr<int32_t>(acc),
                                      ptr<float>(stats), s, stream);
    });
    return results({&y, &acc, &stats});
}

// d, a, pa, b, pb, want_acc, out, ws, packed (layer gradient only); which as for qgemm
template <int WHICH>
PyObject *qconv(Argv a)
{
    const Desc d(a[0]);
    const at::Tensor &x = dev(a[1]), &w = dev(a[3]);
    if (WHICH == 1) shape_is(x, {d->N, d->K, d.P(), d.Q()});
    else shape_is(x, {d->N, d->C, d->H, d->W});
    if (WHICH == 2) shape_is(w, {d->N, d->K, d.P(), d.Q()});
    else shape_is(w, {d->K, d->C, d->R, d->S});
    require(WHICH < 2 || w.scalar_type() == at::kShort);
    const int64_t fwd[4] = {d->N, d->K, d.P(), d.Q()}, dgrad[4] = {d->N, d->C, d->H, d->W}, wgrad[4] = {d->K, d->C, d->R, d->S};
    const at::IntArrayRef shape(WHICH == 0 ? fwd : (WHICH == 1 ? dgrad : wgrad), 4);
    at::Tensor acc;
    const at::Tensor y = given(a[6], [&] { return make(shape, at::kFloat, x); });
    if (truth(a[5])) acc = make(shape, WHICH == 2 ? at::kLong : at::kInt, x);
    const Scratch ws(a[7], q8t_qconv_workspace_size(d.get(), WHICH), a[1]);
    const q8t_qparams *pa = ptr<q8t_qparams>(a[2]), *pb = ptr<q8t_qparams>(a[4]);
    const void *packed = WHICH == 1 ? ptr<void>(a[8]) : nullptr;
    run(WHICH == 0 ? "q8t_qconv_fwd" : (WHICH == 2 ? "q8t_qconv_wgrad" : (packed ? "q8t_qconv_dgrad_packed" : "q8t_qconv_dgrad")),
        [&, s = ws.get()](void *stream) {
            if (WHICH == 0)
                return q8t_qconv_fwd(d.get(), ptr<int8_t>(x), pa, ptr<int8_t>(w), pb, ptr<float>(y), ptr<int32_t>(acc), s, stream);
            if (WHICH == 2)
                return q8t_qconv_wgrad(d.get(), ptr<int8_t>(x), pa, ptr<int16_t>(w), pb, ptr<float>(y), ptr<int64_t>(acc), s, stream);
            if (packed)
                return q8t_qconv_dgrad_packed(d.get(), ptr<int8_t>(x), pa, ptr<int8_t>(w), pb, packed, ptr<float>(y),
                                              ptr<int32_t>(acc), s, stream);
            return q8t_qconv_dgrad(d.get(), ptr<int8_t>(x), pa, ptr<int8_t>(w), pb, ptr<float>(y), ptr<int32_t>(acc), s, stream);
        });
    return results({&y, &acc});
}

// d, qdy, pg, qw, pw, other, act, out, ws, packed; act None: nothing to mask (other is then required)
PyObject *qconv_dgrad_sum(Argv a)
{
    const Desc d(a[0]);
    const at::Tensor &g = dev(a[1]), &w = dev(a[3]);
    shape_is(g, {d->N, d->K, d.P(), d.Q()});
    shape_is(w, {d->K, d->C, d->R, d->S});
    for (int i = 5; i < 7; ++i)
        if (a[i] != Py_None) {
            const at::Tensor &t = dev(a[i]);
            shape_is(t, {d->N, d->C, d->H, d->W});
            require(t.scalar_type() == at::kFloat);
        }
    const at::Tensor dx = given(a[7], [&] { return make({d->N, d->C, d->H, d->W}, at::kFloat, g); });
    const Scratch ws(a[8], q8t_qconv_workspace_size(d.get(), 1), a[1]);
    const q8t_qparams *pg = ptr<q8t_qparams>(a[2]), *pw = ptr<q8t_qparams>(a[4]);
    const float *other = ptr<float>(a[5]), *act = ptr<float>(a[6]);
    const void *packed = ptr<void>(a[9]);
    run(!act ? "q8t_qconv_dgrad_sum" : (packed ? "q8t_qconv_dgrad_relu_sum_packed" : "q8t_qconv_dgrad_relu_sum"),
        [&, s = ws.get()](void *stream) {
            if (!act)
                return q8t_qconv_dgrad_sum(d.get(), ptr<int8_t>(g), pg, ptr<int8_t>(w), pw, packed, other, ptr<float>(dx), s, stream);
            if (packed)
                return q8t_qconv_dgrad_relu_sum_packed(d.get(), ptr<int8_t>(g), pg, ptr<int8_t>(w), pw, packed, other, act,
                                                       ptr<float>(dx), s, stream);
            return q8t_qconv_dgrad_relu_sum(d.get(), ptr<int8_t>(g), pg, ptr<int8_t>(w), pw, other, act, ptr<float>(dx), s, stream);
        });
    return wrap(dx);
}

// x, gamma, beta, eps, quantized, want_y, y_out, stats_out, q_out, qp_out, ws
PyObject *range_bn_fwd(Argv a)
{
    const at::Tensor &x = dev(a[0]);
    const Plane s(x);
    const float eps = real(a[3]);
    const bool quantized = truth(a[4]), want = truth(a[5]);
    at::Tensor y, q, p;
    if (a[6] != Py_None || want) y = given(a[6], [&] { return same(x); });
    const at::Tensor stats = given(a[7], [&] { return make({3, s.C}, at::kFloat, x); });
    if (quantized) {
        q = given(a[8], [&] { return make(x.sizes(), at::kChar, x); });
        p = given(a[9], [&] { return make_params(x); });
    }
    const Scratch ws(a[10], q8t_range_bn_workspace_size(s.N, s.C, s.H, s.W), a[0]);
    const float *gamma = ptr<float>(a[1]), *beta = ptr<float>(a[2]);
    run("q8t_range_bn_fwd", [&, w = ws.get()](void *stream) {
        return q8t_range_bn_fwd(ptr<float>(x), s.N, s.C, s.H, s.W, gamma, beta, eps, ptr<float>(y), ptr<float>(stats), ptr<int8_t>(q),
                                ptr<q8t_qparams>(p), w, stream);
    });
    return results({&y, &stats, &q, &p});
}

// x, stats, gamma, beta, eps, quantized, want_y, y_out, q_out, qp_out
template <bool RELU>
PyObject *range_bn_fwd_apply(Argv a)
{
    const at::Tensor &x = dev(a[0]), &stats = dev(a[1]);
    const Plane s(x);
    const float eps = real(a[4]);
    const bool quantized = truth(a[5]), want = truth(a[6]);
    at::Tensor y, q, p;
    if (a[7] != Py_None || want) y = given(a[7], [&] { return same(x); });
    if (quantized) {
        q = given(a[8], [&] { return make(x.sizes(), at::kChar, x); });
        p = given(a[9], [&] { return make_params(x); });
    }
    const float *gamma = ptr<float>(a[2]), *beta = ptr<float>(a[3]);
    run(RELU ? "q8t_range_bn_relu_fwd_apply" : "q8t_range_bn_fwd_apply", [&](void *stream) {
        return (RELU ? q8t_range_bn_relu_fwd_apply : q8t_range_bn_fwd_apply)(ptr<float>(x), s.N, s.C, s.H, s.W, gamma, beta, eps,
                                                                             ptr<float>(stats), ptr<float>(y), ptr<int8_t>(q),
                                                                             ptr<q8t_qparams>(p), stream);
    });
    return results({&y, &q, &p});
}

// x, dy, stats, gamma, eps, dx_out, ws
PyObject *range_bn_bwd(Argv a)
{
    const at::Tensor &x = dev(a[0]), &dy = dev(a[1]), &stats = dev(a[2]);
    const Plane s(x);
    const float eps = real(a[4]);
    const at::Tensor dx = given(a[5], [&] { return same(x); });
    const at::Tensor dgamma = make({s.C}, at::kFloat, x), dbeta = make({s.C}, at::kFloat, x);
    const Scratch ws(a[6], q8t_range_bn_workspace_size(s.N, s.C, s.H, s.W), a[0]);
    const float *gamma = ptr<float>(a[3]);
    run("q8t_range_bn_bwd", [&, w = ws.get()](void *stream) {
        return q8t_range_bn_bwd(ptr<float>(x), ptr<float>(dy), ptr<float>(stats), s.N, s.C, s.H, s.W, gamma, eps, ptr<float>(dx),
                                ptr<float>(dgamma), ptr<float>(dbeta), w, stream);
    });
    return results({&dx, &dgamma, &dbeta});
}

// x, dy, stats, gamma, beta, eps, seed8, seed16, dx_out, q8_out, qp8_out, q16_out, qp16_out, ws, want_dx, want_q8, act;
// act: the gradient is masked where it is not positive (or, bytes: where the bits of q8t_range_bn_add_relu_pass say so) and the
// masked gradient takes the place of dx in the results
template <bool RELU>
PyObject *range_bn_bwd_bifurcate(Argv a)
{
    const at::Tensor &x = dev(a[0]), &dy = dev(a[1]), &stats = dev(a[2]);
    const Plane s(x);
    const float eps = real(a[5]);
    const uint64_t s8 = seed(a[6]), s16 = seed(a[7]);
    const bool masked = !RELU && a[16] != Py_None, want_q8 = truth(a[15]);
    const float *act = nullptr;
    const uint8_t *pass = nullptr;
    if (masked) {
        const at::Tensor &t = dev(a[16]);
        require(dy.sizes().equals(x.sizes()) && dy.scalar_type() == at::kFloat);
        if (t.scalar_type() == at::kByte) {
            require(t.numel() * 4 == x.numel());
            pass = ptr<uint8_t>(t);
        } else {
            require(t.sizes().equals(x.sizes()) && t.scalar_type() == at::kFloat);
            act = ptr<float>(t);
        }
    }
    at::Tensor dx, q8, p8;
    if (a[8] != Py_None || truth(a[14]) || masked) dx = given(a[8], [&] { return same(x); });
    const at::Tensor dgamma = make({s.C}, at::kFloat, x), dbeta = make({s.C}, at::kFloat, x);
    if (want_q8) {
        q8 = given(a[9], [&] { return make(x.sizes(), at::kChar, x); });
        p8 = given(a[10], [&] { return make_params(x); });
    }
    const at::Tensor q16 = given(a[11], [&] { return make(x.sizes(), at::kShort, x); });
    const at::Tensor p16 = given(a[12], [&] { return make_params(x); });
    const Scratch ws(a[13], q8t_range_bn_bwd_bifurcate_workspace_size(s.N, s.C, s.H, s.W), a[0]);
    const float *gamma = ptr<float>(a[3]), *beta = ptr<float>(a[4]);
    run(RELU ? "q8t_range_bn_relu_bwd_bifurcate" : (pass ? "q8t_range_bn_bwd_bifurcate_pass" : (masked ? "q8t_range_bn_bwd_bifurcate_masked" : "q8t_range_bn_bwd_bifurcate")),
        [&, w = ws.get()](void *stream) {
            const float *px = ptr<float>(x), *pdy = ptr<float>(dy), *pst = ptr<float>(stats);
            float *dg = ptr<float>(dgamma), *db = ptr<float>(dbeta);
            int8_t *o8 = ptr<int8_t>(q8);
            int16_t *o16 = ptr<int16_t>(q16);
            q8t_qparams *r8 = ptr<q8t_qparams>(p8), *r16 = ptr<q8t_qparams>(p16);
            if (RELU)
                return q8t_range_bn_relu_bwd_bifurcate(px, pdy, pst, s.N, s.C, s.H, s.W, gamma, beta, eps, ptr<float>(dx), dg, db, s8,
                                                       s16, o8, r8, o16, r16, w, stream);
            if (pass)
                return q8t_range_bn_bwd_bifurcate_pass(px, pdy, pass, pst, s.N, s.C, s.H, s.W, gamma, eps, ptr<float>(dx), dg, db, s8,
                                                       s16, o8, r8, o16, r16, w, stream);
            if (masked)
                return q8t_range_bn_bwd_bifurcate_masked(px, pdy, act, pst, s.N, s.C, s.H, s.W, gamma, eps, ptr<float>(dx), dg, db, s8,
                                                         s16, o8, r8, o16, r16, w, stream);
            return q8t_range_bn_bwd_bifurcate(px, pdy, pst, s.N, s.C, s.H, s.W, gamma, eps, ptr<float>(dx), dg, db, s8, s16, o8, r8,
                                              o16, r16, w, stream);
        });
    return results({&dx, &dgamma, &dbeta, &q8, &p8, &q16, &p16});
}

// x, stats, other, gamma, beta, other_stats, other_gamma, other_beta, eps, quantized
PyObject *range_bn_add_relu_quantize(Argv a)
{
    const at::Tensor &x = dev(a[0]), &other = dev(a[2]), &stats = dev(a[1]);
    const Plane s(x);
    const float eps = real(a[8]);
    at::Tensor q, p;
    const at::Tensor out = same(x);
    if (truth(a[9])) {
        q = make(x.sizes(), at::kChar, x);
        p = make_params(x);
    }
    const Scratch ws(Py_None, q8t_add_relu_quantize_workspace_size(x.numel()), a[0]);
    const float *ga = ptr<float>(a[3]), *be = ptr<float>(a[4]), *os = ptr<float>(a[5]), *og = ptr<float>(a[6]), *ob = ptr<float>(a[7]);
    run("q8t_range_bn_add_relu_quantize", [&, w = ws.get()](void *stream) {
        return q8t_range_bn_add_relu_quantize(ptr<float>(x), ptr<float>(stats), ga, be, ptr<float>(other), os, og, ob, s.N, s.C, s.H,
                                              s.W, eps, ptr<float>(out), ptr<int8_t>(q), ptr<q8t_qparams>(p), w, stream);
    });
    return results({&out, &q, &p});
}

template <PyObject *(*F)(Argv), int N>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "q8t: %d arguments are expected, %zd given", N, n);
        return nullptr;
    }
    HANDLE_TH_ERRORS
    try {
        return F(args);
    } catch (const Raised &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject *setup(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "q8t: workspace, its cache and the error type are expected");
        return nullptr;
    }
    PyObject **slot[3] = {&g_workspace, &g_cache, &g_error};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(args[i]);
        Py_XSETREF(*slot[i], args[i]);
    }
    Py_RETURN_NONE;
}

#define CALL(name, f, n) {name, (PyCFunction)(void (*)(void))entry<f, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"setup", (PyCFunction)(void (*)(void))setup, METH_FASTCALL, nullptr},
    CALL("quantize", quantize, 7),
    CALL("quantize_with_range", quantize_with_range, 7),
    CALL("quantize_bifurcate", quantize_bifurcate, 8),
    CALL("chunk_range", chunk_range, 3),
    CALL("qgemm_fwd", qgemm<0>, 7),
    CALL("qgemm_dgrad", qgemm<1>, 7),
    CALL("qgemm_wgrad", qgemm<2>, 7),
    CALL("qconv_fwd", qconv<0>, 9),
    CALL("qconv_dgrad", qconv<1>, 9),
    CALL("qconv_wgrad", qconv<2>, 9),
    CALL("qconv_fwd_bn_stats", qconv_fwd_bn_stats, 10),
    CALL("qconv_dgrad_sum", qconv_dgrad_sum, 10),
    CALL("range_bn_fwd", range_bn_fwd, 11),
    CALL("range_bn_fwd_apply", range_bn_fwd_apply<false>, 10),
    CALL("range_bn_relu_fwd_apply", range_bn_fwd_apply<true>, 10),
    CALL("range_bn_bwd", range_bn_bwd, 7),
    CALL("range_bn_bwd_bifurcate", range_bn_bwd_bifurcate<false>, 17),
    CALL("range_bn_relu_bwd_bifurcate", range_bn_bwd_bifurcate<true>, 17),
    CALL("range_bn_add_relu_quantize", range_bn_add_relu_quantize, 10),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_q8t_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__q8t_calls(void) { return PyModule_Create(&module); }
