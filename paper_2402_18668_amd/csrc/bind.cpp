// Native half of the Python binding: argument checks, output allocation and the library call of the hot
// entry points in one C++ function each.
//
// A small call is bound by the host, not by the GPU: one token of the fused decode step is 3-6 us of kernel, and
// marshalling its 25 arguments in Python (ctypes boxes, tensor attributes, the stream object) took 20 us.
// Here a tensor's pointer, shape and dtype are field reads (the same checks as before: 23 -> 10 us for a fused step
// and the advance of its positions).
// based.py keeps the public functions (names, defaults, documentation) and hands their arguments over
// positionally; the entry points' addresses come from the library it has loaded, so that there is one library
// in the process whichever build of it the user points the binding at.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/DimVector.h>
#include <ATen/core/LegacyTypeDispatch.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>

#include "../../include/based.h"

namespace {

#define BASED_FNS(X)                                                                                              \
    X(based_prefill) X(based_prefill_packed) X(based_prefill_numerator) X(based_prefill_workspace_bytes)           \
    X(based_decode_step) X(based_decode_step_packed) X(based_decode_step_numerator) X(based_state_bytes)           \
    X(based_packed_state_bytes) X(based_swa_prefill) X(based_swa_prefill_rotary) X(based_swa_decode)               \
    X(based_swa_decode_ragged) X(based_swa_decode_rotary) X(based_decode_fused) X(based_decode_fused_packed)       \
    X(based_decode_fused_ragged) X(based_decode_fused_rotary) X(based_positions_advance) X(based_linear)           \
    X(based_project_qkv) X(based_project_out) X(based_short_conv_gate)
struct Fns {
#define X(name) decltype(&::name) name;
    BASED_FNS(X)
#undef X
} fn = {};
PyObject *g_raise = nullptr;   // Python callable (status, what): raises the package's error

struct PyError {};   // a Python exception is set

[[noreturn]] void fail(PyObject *type, const char *msg)
{
    PyErr_SetString(type, msg);
    throw PyError{};
}
[[noreturn]] void bad(const char *msg) { fail(PyExc_ValueError, msg); }

void check(int status, const char *what)
{
    if (status == BASED_OK) return;
    PyObject *r = PyObject_CallFunction(g_raise, "is", status, what);
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, what);
    throw PyError{};
}

// Allocates what a call returns and makes the call, without the interpreter lock: a launch into a full queue and an allocation
// that has to wait for the GPU would otherwise stop every Python thread.  (Both in one stretch without the lock: giving it up and
// taking it back costs 0.1 us, and longer with other threads running.)  f touches nothing of Python.
template <typename F> void call(const char *what, F &&f)
{
    int status;
    {
        struct Unlocked {
            PyThreadState *state = PyEval_SaveThread();
            ~Unlocked() { PyEval_RestoreThread(state); }
        } unlocked;
        status = f();
    }
    check(status, what);
}

// A tensor argument: a borrowed handle, checked to live on the GPU and to be contiguous.
using Arg = const at::Tensor *;
Arg tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch.Tensor");
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda()) bad("tensors must live on the GPU");
    if (!t.is_contiguous()) bad("tensors must be contiguous");
    return &t;
}
Arg optional(PyObject *o) { return o == Py_None ? nullptr : tensor(o); }

void *ptr(Arg t) { return t ? t->data_ptr() : nullptr; }
int code_of(Arg t)
{
    if (t->scalar_type() == at::kFloat) return BASED_F32;
    if (t->scalar_type() == at::kBFloat16) return BASED_BF16;
    fail(PyExc_TypeError, "unsupported tensor dtype");
}
bool shape_is(Arg t, std::initializer_list<int64_t> s) { return t->sizes() == at::IntArrayRef(s.begin(), s.size()); }
bool same_type(Arg a, Arg b) { return a->scalar_type() == b->scalar_type(); }
void want_dim(Arg t, int64_t d, const char *msg)
{
    if (t->dim() != d) bad(msg);
}
size_t nbytes(Arg t) { return (size_t)t->numel() * t->element_size(); }

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

long as_long(PyObject *o)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyError{};
    return v;
}
int as_int(PyObject *o)
{
    long v;
    if (PyLong_Check(o)) {
        v = as_long(o);
    } else {   // whatever int() takes
        PyObject *n = PyNumber_Long(o);
        if (!n) throw PyError{};
        v = PyLong_AsLong(n);
        Py_DECREF(n);
        if (v == -1 && PyErr_Occurred()) throw PyError{};
    }
    if (v != (long)(int)v) fail(PyExc_OverflowError, "integer argument out of range");
    return (int)v;
}
int as_bool(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyError{};
    return v;
}
float as_float(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PyError{};
    return (float)v;
}

// A new tensor of like's type and device, of the given shape (null: like's own).  Straight from the device's allocation function
// (two trips through the dispatcher are a third of what an allocation costs, 0.9 us), unless somebody looks at operators or has a
// say in them: a mode or transformation, the tracer, like's own class, a profiler's callbacks, the fill of uninitialised memory.
// (Asking takes 0.02 us.)
at::Tensor new_tensor(Arg like, const at::IntArrayRef *shape)
{
    using c10::DispatchKey;
    constexpr c10::DispatchKeySet classes({DispatchKey::Python, DispatchKey::PythonTLSSnapshot, DispatchKey::PythonDispatcher,
                                           DispatchKey::FuncTorchDynamicLayerFrontMode, DispatchKey::FuncTorchDynamicLayerBackMode,
                                           DispatchKey::Functionalize, DispatchKey::FuncTorchBatched, DispatchKey::Tracer});
    const at::Context &context = at::globalContext();
    if ((c10::impl::tls_local_dispatch_key_set().included_ | like->key_set()).has_any(classes) ||
        at::getStepCallbacksUnlessEmpty(at::RecordScope::FUNCTION).has_value() ||
        (context.deterministicAlgorithms() && context.deterministicFillUninitializedMemory()))
        return shape ? at::empty(*shape, like->options()) : at::empty_like(*like);
    return at::Tensor(at::detail::empty_cuda(shape ? *shape : like->sizes(), like->scalar_type(), like->device(), std::nullopt));
}

// A result: the tensor the caller gave (of the same shape and type where `msg` says what to answer otherwise, else any
// buffer that is large enough), or one that make() allocates (inside call()), shaped like `like` or of the given shape.
struct Out {
    PyObject *given = nullptr;
    void *data = nullptr;
    at::Tensor made;
    Arg like;
    at::DimVector shape;   // (empty: like's own)
    Out(PyObject *o, Arg like_, const char *msg = nullptr) : like(like_)
    {
        if (o == Py_None) return;
        Arg t = tensor(o);
        if (msg ? t->sizes() != like->sizes() || !same_type(t, like) : nbytes(t) < nbytes(like))
            bad(msg ? msg : "output buffer too small");
        given = o;
        data = t->data_ptr();
    }
    Out(Arg like_, std::initializer_list<int64_t> shape_) : like(like_), shape(shape_) {}
    void make()
    {
        if (given) return;
        const at::IntArrayRef own(shape);
        made = new_tensor(like, shape.empty() ? nullptr : &own);
        data = made.data_ptr();
    }
    PyObject *take()
    {
        if (given) { Py_INCREF(given); return given; }
        return THPVariable_Wrap(std::move(made));
    }
};
PyObject *pair(Out &a, Out &b)
{
    PyObject *t = PyTuple_New(2);
    if (!t) throw PyError{};
    PyTuple_SET_ITEM(t, 0, a.take());
    PyTuple_SET_ITEM(t, 1, b.take());
    return t;
}

void check_state(Arg st, size_t need)
{
    if (st->scalar_type() != at::kFloat || nbytes(st) < need) bad("state buffer too small or not fp32");
}

// q, k, v, y, state, has_init, workspace, packed, numerator_only
PyObject *prefill(PyObject *const *a)
{
    Arg q = tensor(a[0]), k = tensor(a[1]), v = tensor(a[2]), state = optional(a[4]), ws = optional(a[6]);
    const int has_init = as_bool(a[5]), packed = as_bool(a[7]), numer = as_bool(a[8]);
    want_dim(q, 4, "q must be [B, H, N, d']");
    want_dim(v, 4, "v must be [B, H, N, d_v]");
    const int B = q->size(0), H = q->size(1), N = q->size(2), dp = q->size(3), dv = v->size(3);
    if (k->sizes() != q->sizes() || !shape_is(v, {B, H, N, dv}) || !same_type(k, q) || !same_type(v, q))
        bad("q, k, v shapes / dtypes disagree");
    const int code = code_of(q);
    Out y(a[3], v, "y must match v");
    if (state) check_state(state, packed ? fn.based_packed_state_bytes(B, H, dp, dv) : fn.based_state_bytes(B, H, dp, dv));
    const size_t need = fn.based_prefill_workspace_bytes(B, H, N, dp, dv, code);
    if (need && ws && nbytes(ws) < need) bad("workspace too small");
    if (packed && numer) bad("there is no packed numerator-only prefill");
    auto f = numer ? fn.based_prefill_numerator : packed ? fn.based_prefill_packed : fn.based_prefill;
    call(numer ? "based_prefill_numerator" : packed ? "based_prefill_packed" : "based_prefill", [&] {
        y.make();
        at::Tensor own;
        if (need && !ws) {   // zero-filled once, as the library asks
            own = at::zeros({(int64_t)((need + 3) / 4)}, q->options().dtype(at::kFloat));
            ws = &own;
        }
        return f(ptr(q), ptr(k), ptr(v), y.data, ptr(state), has_init, ptr(ws), B, H, N, dp, dv, code, stream());
    });
    return y.take();
}

// q, k, v, state, y, packed, numerator_only
PyObject *decode_step(PyObject *const *a)
{
    Arg q = tensor(a[0]), k = tensor(a[1]), v = tensor(a[2]), state = tensor(a[3]);
    const int packed = as_bool(a[5]), numer = as_bool(a[6]);
    want_dim(q, 3, "q must be [B, H, d']");
    want_dim(v, 3, "v must be [B, H, d_v]");
    const int B = q->size(0), H = q->size(1), dp = q->size(2), dv = v->size(2);
    if (k->sizes() != q->sizes() || !shape_is(v, {B, H, dv}) || !same_type(k, q) || !same_type(v, q))
        bad("q, k, v shapes / dtypes disagree");
    check_state(state, packed ? fn.based_packed_state_bytes(B, H, dp, dv) : fn.based_state_bytes(B, H, dp, dv));
    Out y(a[4], v);
    if (packed && numer) bad("there is no packed numerator-only decode step");
    const int code = code_of(q);
    auto f = numer ? fn.based_decode_step_numerator : packed ? fn.based_decode_step_packed : fn.based_decode_step;
    call(numer ? "based_decode_step_numerator" : packed ? "based_decode_step_packed" : "based_decode_step", [&] {
        y.make();
        return f(ptr(q), ptr(k), ptr(v), y.data, ptr(state), B, H, dp, dv, code, stream());
    });
    return y.take();
}

// a rotary table for head dim dh: [rows][dh / 2][2] fp32 (rows < 0: any number)
Arg rotary_table(PyObject *o, int64_t rows, int64_t dh)
{
    Arg t = optional(o);
    if (t && (t->scalar_type() != at::kFloat || t->dim() != 3 || (rows >= 0 && t->size(0) != rows) ||
              t->size(1) != dh / 2 || t->size(2) != 2))
        bad(rows >= 0 ? "rotary table must be contiguous fp32 [N, d_h / 2, 2]"
                      : "rotary table must be contiguous fp32 [rows, d_h / 2, 2]");
    return t;
}

// q, k, v, w, scale, y, ring, rotary
PyObject *swa_prefill(PyObject *const *a)
{
    Arg q = tensor(a[0]), k = tensor(a[1]), v = tensor(a[2]), ring = optional(a[6]);
    const int w = as_int(a[3]);
    const float scale = as_float(a[4]);
    want_dim(q, 4, "q must be [B, H, N, d_h]");
    const int B = q->size(0), H = q->size(1), N = q->size(2), dh = q->size(3);
    if (k->sizes() != q->sizes() || v->sizes() != q->sizes() || !same_type(k, q) || !same_type(v, q))
        bad("q, k, v shapes / dtypes disagree");
    if (ring && (!same_type(ring, q) || ring->numel() != (int64_t)B * H * 2 * w * dh))
        bad("ring must be [B,H,2,w,d_h] of the input dtype");
    Arg rot = rotary_table(a[7], N, dh);
    const int code = code_of(q);
    Out y(a[5], v);
    call(rot ? "based_swa_prefill_rotary" : "based_swa_prefill", [&] {
        y.make();
        return rot ? fn.based_swa_prefill_rotary(ptr(q), ptr(k), ptr(v), y.data, ptr(ring), (const float *)ptr(rot), B, H, N, dh,
                                                 w, scale, code, stream())
                   : fn.based_swa_prefill(ptr(q), ptr(k), ptr(v), y.data, ptr(ring), B, H, N, dh, w, scale, code, stream());
    });
    return y.take();
}

// The position argument of a decode call: a number, or an int32 device tensor of one position per sequence.
struct Pos {
    int value = 0;
    const int *per_seq = nullptr;
};
Pos position(PyObject *o, int64_t B)
{
    Pos p;
    if (!THPVariable_Check(o)) {
        p.value = as_int(o);
        return p;
    }
    const at::Tensor &t = THPVariable_Unpack(o);
    if (t.scalar_type() != at::kInt || t.numel() != B || !t.is_cuda() || !t.is_contiguous())
        bad("per-sequence positions must be a contiguous int32 device tensor of B elements");
    p.per_seq = (const int *)t.data_ptr();
    return p;
}

// q, k, v, ring, pos, w, scale, y, rotary
PyObject *swa_decode(PyObject *const *a)
{
    Arg q = tensor(a[0]), k = tensor(a[1]), v = tensor(a[2]), ring = tensor(a[3]);
    const int w = as_int(a[5]);
    const float scale = as_float(a[6]);
    want_dim(q, 3, "q must be [B, H, d_h]");
    const int B = q->size(0), H = q->size(1), dh = q->size(2);
    if (k->sizes() != q->sizes() || v->sizes() != q->sizes() || !same_type(k, q) || !same_type(v, q))
        bad("q, k, v shapes / dtypes disagree");
    if (!same_type(ring, q) || ring->numel() != (int64_t)B * H * 2 * w * dh)
        bad("ring must be [B,H,2,w,d_h] of the input dtype");
    Arg rot = rotary_table(a[8], -1, dh);
    const Pos pos = position(a[4], B);
    const int code = code_of(q);
    Out y(a[7], v);
    call(rot ? "based_swa_decode_rotary" : pos.per_seq ? "based_swa_decode_ragged" : "based_swa_decode", [&] {
        y.make();
        if (rot)
            return fn.based_swa_decode_rotary(ptr(q), ptr(k), ptr(v), y.data, ptr(ring), (const float *)ptr(rot),
                                              (int)rot->size(0), pos.value, pos.per_seq, B, H, dh, w, scale, code, stream());
        if (pos.per_seq)
            return fn.based_swa_decode_ragged(ptr(q), ptr(k), ptr(v), y.data, ptr(ring), pos.per_seq, B, H, dh, w, scale, code,
                                              stream());
        return fn.based_swa_decode(ptr(q), ptr(k), ptr(v), y.data, ptr(ring), pos.value, B, H, dh, w, scale, code, stream());
    });
    return y.take();
}

// q, k, v, state, swa_q, swa_k, swa_v, ring, pos, w, scale, y_lin, y_swa, packed, rotary
PyObject *decode_fused(PyObject *const *a)
{
    Arg q = tensor(a[0]), k = tensor(a[1]), v = tensor(a[2]), state = tensor(a[3]);
    Arg sq = tensor(a[4]), sk = tensor(a[5]), sv = tensor(a[6]), ring = tensor(a[7]);
    const int w = as_int(a[9]), packed = as_bool(a[13]);
    const float scale = as_float(a[10]);
    want_dim(q, 3, "q must be [B, H, d']");
    want_dim(v, 3, "v must be [B, H, d_v]");
    want_dim(sq, 3, "the window attention q must be [B, H, d_h]");
    const int B = q->size(0), H = q->size(1), dp = q->size(2), dv = v->size(2), dh = sq->size(2);
    if (k->sizes() != q->sizes() || !shape_is(v, {B, H, dv}) || !shape_is(sq, {B, H, dh})) bad("shapes disagree");
    if (sk->sizes() != sq->sizes() || sv->sizes() != sq->sizes()) bad("window attention shapes disagree");
    for (Arg t : {k, v, sq, sk, sv, ring})
        if (!same_type(t, q)) bad("dtypes disagree");
    check_state(state, packed ? fn.based_packed_state_bytes(B, H, dp, dv) : fn.based_state_bytes(B, H, dp, dv));
    if (ring->numel() != (int64_t)B * H * 2 * w * dh) bad("ring must be [B,H,2,w,d_h]");
    Arg rot = rotary_table(a[14], -1, dh);
    const Pos pos = position(a[8], B);
    const int code = code_of(q);
    Out yl(a[11], v), ys(a[12], sv);
    call(rot ? "based_decode_fused_rotary" : pos.per_seq ? "based_decode_fused_ragged"
                                           : packed      ? "based_decode_fused_packed"
                                                         : "based_decode_fused", [&] {
        yl.make();
        ys.make();
        if (rot)
            return fn.based_decode_fused_rotary(ptr(q), ptr(k), ptr(v), yl.data, ptr(state), packed, dp, dv, ptr(sq), ptr(sk),
                                                ptr(sv), ys.data, ptr(ring), (const float *)ptr(rot), (int)rot->size(0),
                                                pos.value, pos.per_seq, dh, w, scale, B, H, code, stream());
        if (pos.per_seq)
            return fn.based_decode_fused_ragged(ptr(q), ptr(k), ptr(v), yl.data, ptr(state), packed, dp, dv, ptr(sq), ptr(sk),
                                                ptr(sv), ys.data, ptr(ring), pos.per_seq, dh, w, scale, B, H, code, stream());
        return (packed ? fn.based_decode_fused_packed : fn.based_decode_fused)(
            ptr(q), ptr(k), ptr(v), yl.data, ptr(state), dp, dv, ptr(sq), ptr(sk), ptr(sv), ys.data, ptr(ring), pos.value, dh, w,
            scale, B, H, code, stream());
    });
    return pair(yl, ys);
}

// pos
PyObject *positions_advance(PyObject *const *a)
{
    if (!THPVariable_Check(a[0])) fail(PyExc_TypeError, "expected a torch.Tensor");
    const int B = (int)THPVariable_Unpack(a[0]).numel();
    const Pos pos = position(a[0], B);
    call("based_positions_advance", [&] { return fn.based_positions_advance(const_cast<int *>(pos.per_seq), B, stream()); });
    Py_RETURN_NONE;
}

// x, W, y
PyObject *linear(PyObject *const *a)
{
    Arg x = tensor(a[0]), W = tensor(a[1]), y_given = optional(a[2]);
    if (x->dim() < 1 || W->dim() != 2 || x->size(-1) != W->size(1) || x->size(-1) < 1 || !same_type(W, x))
        bad("x [..., K] and W [N, K] must be contiguous and of one dtype");
    const int64_t K = W->size(1), N = W->size(0), M = x->numel() / K;
    if (y_given && (y_given->numel() != M * N || !same_type(y_given, x)))
        bad("y must be [..., N], contiguous, of x's dtype");
    auto shape = x->sizes().vec();
    shape.back() = N;
    const int code = code_of(x);
    at::Tensor made;
    call("based_linear", [&] {
        const at::IntArrayRef sizes(shape);
        if (!y_given) made = new_tensor(x, &sizes);
        return fn.based_linear(ptr(x), ptr(W), y_given ? ptr(y_given) : made.data_ptr(), (int)M, (int)K, (int)N, code, stream());
    });
    if (y_given) { Py_INCREF(a[2]); return a[2]; }
    return THPVariable_Wrap(std::move(made));
}

// x, W, H, d_feat, d_v
PyObject *project_qkv(PyObject *const *a)
{
    Arg x = tensor(a[0]), W = tensor(a[1]);
    const int H = as_int(a[2]), dp = as_int(a[3]), dv = as_int(a[4]);
    want_dim(x, 3, "x must be [B, N, d_model]");
    const int B = x->size(0), N = x->size(1), dm = x->size(2);
    if (!shape_is(W, {(int64_t)H * (2 * dp + dv), dm}) || !same_type(W, x))
        bad("x [B, N, d_model] and W [H (2 d' + d_v), d_model] must be contiguous and of one dtype");
    Out q(x, {B, H, N, dp}), k(x, {B, H, N, dp}), v(x, {B, H, N, dv});
    const int code = code_of(x);
    call("based_project_qkv", [&] {
        q.make();
        k.make();
        v.make();
        return fn.based_project_qkv(ptr(x), ptr(W), q.data, k.data, v.data, B, N, dm, H, dp, dv, code, stream());
    });
    PyObject *t = PyTuple_New(3);
    if (!t) throw PyError{};
    PyTuple_SET_ITEM(t, 0, q.take());
    PyTuple_SET_ITEM(t, 1, k.take());
    PyTuple_SET_ITEM(t, 2, v.take());
    return t;
}

// y_heads, W
PyObject *project_out(PyObject *const *a)
{
    Arg y = tensor(a[0]), W = tensor(a[1]);
    want_dim(y, 4, "y must be [B, H, N, d_v]");
    const int B = y->size(0), H = y->size(1), N = y->size(2), dv = y->size(3);
    if (W->dim() != 2 || W->size(1) != (int64_t)H * dv || !same_type(W, y))
        bad("y [B, H, N, d_v] and W [d_model, H d_v] must be contiguous and of one dtype");
    const int dm = W->size(0);
    Out out(y, {B, N, dm});
    const int code = code_of(y);
    call("based_project_out", [&] {
        out.make();
        return fn.based_project_out(ptr(y), ptr(W), out.data, B, N, H, dv, dm, code, stream());
    });
    return out.take();
}

// a, c, h, b1, b2, c_prev, c_last, out
PyObject *short_conv_gate(PyObject *const *p)
{
    Arg a = tensor(p[0]), c = tensor(p[1]), h = tensor(p[2]), b1 = tensor(p[3]), b2 = tensor(p[4]);
    Arg prev = optional(p[5]), last = optional(p[6]);
    want_dim(a, 3, "a, c must be contiguous [B, N, Dc] of one dtype");
    const int64_t B = a->size(0), N = a->size(1), Dc = a->size(2);
    if (c->sizes() != a->sizes() || !same_type(c, a)) bad("a, c must be contiguous [B, N, Dc] of one dtype");
    if (!shape_is(h, {3, Dc}) || !shape_is(b1, {Dc}) || !shape_is(b2, {Dc}) || h->scalar_type() != at::kFloat ||
        b1->scalar_type() != at::kFloat || b2->scalar_type() != at::kFloat)
        bad("h [3, Dc], b1, b2 [Dc] must be contiguous fp32");
    for (Arg t : {prev, last})
        if (t && (!shape_is(t, {B, 2, Dc}) || !same_type(t, a)))
            bad("c_prev / c_last must be contiguous [B, 2, Dc] of a's dtype");
    Out out(p[7], a, "out must match a");
    const int code = code_of(a);
    call("based_short_conv_gate", [&] {
        out.make();
        return fn.based_short_conv_gate(ptr(a), ptr(c), (const float *)ptr(h), (const float *)ptr(b1), (const float *)ptr(b2),
                                        ptr(prev), out.data, ptr(last), (int)B, (int)N, (int)Dc, code, stream());
    });
    return out.take();
}

// Python entry: the argument count is fixed (based.py passes every argument), C++ exceptions become Python ones.
template <PyObject *(*F)(PyObject *const *), Py_ssize_t NARGS>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != NARGS) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", NARGS, nargs);
        return nullptr;
    }
    try {
        // plain buffers: nothing here is recorded for autograd
        at::AutoDispatchBelowADInplaceOrView guard;
        return F(args);
    } catch (const PyError &) {
    } catch (const c10::OutOfMemoryError &e) {
        PyObject *torch_mod = PyImport_ImportModule("torch");
        PyObject *oom = torch_mod ? PyObject_GetAttrString(torch_mod, "OutOfMemoryError") : nullptr;
        PyErr_Clear();
        PyErr_SetString(oom ? oom : PyExc_MemoryError, e.what_without_backtrace());
        Py_XDECREF(oom);
        Py_XDECREF(torch_mod);
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// init(addresses, raise): addresses maps every entry point's name to its address
PyObject *init(PyObject *, PyObject *args)
{
    PyObject *addr, *raise;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &addr, &raise)) return nullptr;
#define X(name)                                                                                            \
    {                                                                                                      \
        PyObject *v = PyDict_GetItemString(addr, #name);                                                   \
        if (!v) { PyErr_SetString(PyExc_KeyError, #name); return nullptr; }                                \
        void *p = PyLong_AsVoidPtr(v);                                                                     \
        if (!p) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, #name); return nullptr; }       \
        fn.name = reinterpret_cast<decltype(&::name)>(p);                                                  \
    }
    BASED_FNS(X)
#undef X
    Py_INCREF(raise);
    Py_XDECREF(g_raise);
    g_raise = raise;
    Py_RETURN_NONE;
}

#define M(name, n) {#name, (PyCFunction)(void (*)(void))entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"init", init, METH_VARARGS, nullptr},
                         M(prefill, 9),
                         M(decode_step, 7),
                         M(swa_prefill, 8),
                         M(swa_decode, 9),
                         M(decode_fused, 15),
                         M(positions_advance, 1),
                         M(linear, 3),
                         M(project_qkv, 5),
                         M(project_out, 2),
                         M(short_conv_gate, 8),
                         {nullptr, nullptr, 0, nullptr}};
#undef M
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_bind", "Native half of the binding in based.py.", -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind(void) { return PyModule_Create(&module_def); }
