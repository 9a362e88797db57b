// Native half of the Python binding: takes torch tensors and scalars, checks them, and calls the C
// ABI of libmp8.so on the current HIP stream.  The Python module keeps the signatures, defaults
// and documentation; everything that has to happen on every call happens here, because a layer's
// step is five or six launches of a few microseconds each and the host has to stay ahead of them:
// one call through ctypes and Python-level checks cost 8-11 us, about twice what the launch costs.
//
// libmp8.so itself stays free of torch and Python.  Its entry points are handed over by address
// (init), so that whichever build of the library the Python module has loaded is the one called.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstdarg>
#include <cstring>
#include <exception>

#include "../../include/mp8.h"

namespace {

PyObject *g_error = nullptr;  // Mp8Error

// The entry points this module calls.
#define MP8_ENTRIES(X)                                                                              \
    X(mp8_quantize_e5m2) X(mp8_gemm_fp8_tuned) X(mp8_gemm_fp8_static) X(mp8_quantize_gemm_fwd_fp8)   \
    X(mp8_conv3x3_fp8) X(mp8_conv3x3_wgrad_update_fp16_sr) X(mp8_conv3x3_wgrad_momentum_fp16_sr)     \
    X(mp8_wgrad_update_fp16_sr) X(mp8_wgrad_momentum_fp16_sr) X(mp8_wgrad_adam_fp16_sr)              \
    X(mp8_sgd_update_fp16_sr) X(mp8_sgd_momentum_fp16_sr) X(mp8_adam_fp16_sr) X(mp8_status_string)
#define MP8_POINTER(name) decltype(&name) p_##name = nullptr;
MP8_ENTRIES(MP8_POINTER)
#undef MP8_POINTER

// Thrown after a Python exception has been set.
struct Raised {};

[[noreturn]] void fail(const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    PyErr_FormatV(g_error, fmt, ap);
    va_end(ap);
    throw Raised{};
}

// What a tensor argument may hold.
enum Kind { kF32, kU8, kSource /* float32 or float16 */, kHalf /* float16 or its bits */ };

struct Arg {
    void *p = nullptr;
    int64_t n = 0;         // elements
    int64_t itemsize = 0;  // bytes of one
    const at::Tensor *t = nullptr;
    bool given = false;
    explicit operator bool() const { return given; }
};

// Sizes are formed from what the caller passes: they saturate instead of wrapping, so that no product of
// large dimensions passes for a small one.
int64_t mul(int64_t a, int64_t b) {
    int64_t r;
    return __builtin_mul_overflow(a, b, &r) ? ((a < 0) == (b < 0) ? INT64_MAX : INT64_MIN) : r;
}
int64_t add(int64_t a, int64_t b) {
    int64_t r;
    return __builtin_add_overflow(a, b, &r) ? (a < 0 ? INT64_MIN : INT64_MAX) : r;
}

// The arguments of one call, read in order.
struct Args {
    PyObject *const *at_;
    Py_ssize_t left;
    PyObject *next() {
        if (left-- <= 0) {
            PyErr_SetString(PyExc_TypeError, "too few arguments");
            throw Raised{};
        }
        return *at_++;
    }
    // seeds, offsets, enumerations and flags wrap, as they do through ctypes
    uint64_t u64() {
        const uint64_t v = PyLong_AsUnsignedLongLongMask(next());
        if (v == (uint64_t)-1 && PyErr_Occurred()) throw Raised{};
        return v;
    }
    int i32() { return (int)u64(); }
    // dimensions do not: the sizes that are checked are the ones that are passed on
    int64_t as_i64(PyObject *o) {
        int overflow = 0;
        const int64_t v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow) fail("%S does not fit 64 bits", o);
        if (v == -1 && PyErr_Occurred()) throw Raised{};
        return v;
    }
    int64_t i64() { return as_i64(next()); }
    // what int() takes: the step counters that optimizers keep may be floats or tensors
    int64_t whole() {
        PyObject *o = PyNumber_Long(next());
        if (!o) throw Raised{};
        try {
            const int64_t v = as_i64(o);
            Py_DECREF(o);
            return v;
        } catch (const Raised &) {
            Py_DECREF(o);
            throw;
        }
    }
    // what float() takes
    float f32() {
        PyObject *o = next();
        if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
        PyObject *f = PyNumber_Float(o);
        if (!f) throw Raised{};
        const double v = PyFloat_AS_DOUBLE(f);
        Py_DECREF(f);
        return (float)v;
    }
    int op() {
        PyObject *o = next();
        const int64_t v = as_i64(o);
        if (v < 0 || v > 2) {
            PyErr_SetObject(PyExc_KeyError, o);
            throw Raised{};
        }
        return (int)v;
    }
    int64_t i64_or(int64_t otherwise) {  // None: the default
        if (left > 0 && *at_ == Py_None) {
            next();
            return otherwise;
        }
        return i64();
    }
    bool flag() {
        const int v = PyObject_IsTrue(next());
        if (v < 0) throw Raised{};
        return v != 0;
    }
    // a GPU tensor (or None), contiguous, of the expected type
    Arg tensor(const char *name, Kind kind) {
        PyObject *o = next();
        Arg a;
        if (o == Py_None) return a;
        if (!THPVariable_Check(o)) {
            PyErr_Format(PyExc_TypeError, "%s must be a tensor or None", name);
            throw Raised{};
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda()) fail("%s must be a GPU tensor", name);
        if (!t.is_contiguous()) fail("%s must be contiguous", name);
        const at::ScalarType s = t.scalar_type();
        bool ok = true;
        const char *expected = "";
        switch (kind) {
            case kF32: ok = s == at::kFloat; expected = "torch.float32"; break;
            case kU8: ok = s == at::kByte; expected = "torch.uint8"; break;
            case kSource: ok = s == at::kFloat || s == at::kHalf; expected = "(torch.float32, torch.float16)"; break;
            case kHalf:
                ok = s == at::kHalf || s == at::kShort || s == at::kUInt16;
                expected = "(torch.float16, torch.int16, torch.uint16)";
                break;
        }
        if (!ok) {
            PyObject *d = PyObject_GetAttrString(o, "dtype");
            if (!d) throw Raised{};
            PyErr_Format(g_error, "%s has dtype %S, expected %s", name, d, expected);
            Py_DECREF(d);
            throw Raised{};
        }
        a.t = &t;
        a.given = true;
        a.p = t.data_ptr();
        a.n = t.numel();
        a.itemsize = t.element_size();
        return a;
    }
    // A pointer that is passed on as it is (statistics, flags, scratch): a tensor, or any object with the
    // methods of one that are needed here.
    Arg raw(bool sized = false) {
        PyObject *o = next();
        Arg a;
        if (o == Py_None) return a;
        a.given = true;
        if (THPVariable_Check(o)) {
            a.t = &THPVariable_Unpack(o);
            a.p = a.t->data_ptr();
            a.n = a.t->numel();
            a.itemsize = a.t->element_size();
            return a;
        }
        auto call = [&](const char *method) {
            PyObject *v = PyObject_CallMethod(o, method, nullptr);
            const uint64_t x = v ? PyLong_AsUnsignedLongLongMask(v) : 0;
            Py_XDECREF(v);
            if (PyErr_Occurred()) throw Raised{};
            return x;
        };
        a.p = (void *)call("data_ptr");
        if (sized) a.n = (int64_t)call("numel"), a.itemsize = (int64_t)call("element_size");
        return a;
    }
    size_t bytes(const Arg &a) const { return (size_t)a.n * (size_t)a.itemsize; }
};

void must_be(const Arg &a, const char *name) {
    if (!a) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
        throw Raised{};
    }
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

void check(mp8_status st, const char *what) {
    if (st != MP8_OK) fail("%s: %s (status %d)", what, p_mp8_status_string(st), (int)st);
}

// Runs a call without the interpreter lock, as ctypes does.
template <class F>
mp8_status unlocked(F f) {
    mp8_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return st;
}

// Elements an operand of `n` rows and contraction length kc spans with leading dimension ld.
int64_t span(bool contraction_major, int64_t n, int64_t kc, int64_t ld) {
    if (n <= 0 || kc <= 0) return 0;
    return contraction_major ? add(mul(kc - 1, ld), n) : add(mul(n - 1, ld), kc);
}

void op_dims(int op, int64_t M, int64_t N, int64_t K, int64_t &rows, int64_t &cols, int64_t &kc) {
    switch (op) {
        case MP8_FWD: rows = M; cols = N; kc = K; break;
        case MP8_BWD_DATA: rows = M; cols = K; kc = N; break;
        default: rows = K; cols = N; kc = M; break;  // MP8_WGRAD
    }
}

void at_least(const Arg &a, int64_t n, const char *name, const char *what) {
    if (a && a.n < n) fail("%s is smaller than %s", name, what);
}
void exactly(const Arg &a, int64_t n, const char *name, const char *what) {
    if (a && a.n != n) fail("%s must have %s elements", name, what);
}

// ---------------------------------------------------------------------------------------
void quantize(Args a) {
    const Arg src = a.tensor("src", kSource), dst = a.tensor("dst", kU8), dst_t = a.tensor("dst_t", kU8);
    const float scale = a.f32();
    const int round = a.i32(), flags = a.i32();
    const uint64_t seed = a.u64(), offset = a.u64();
    const Arg stats = a.raw();
    must_be(src, "src");
    must_be(dst, "dst");
    if (src.t->dim() != 2) fail("src must be 2-D");
    const int64_t rows = src.t->size(0), cols = src.t->size(1);
    if (dst.n != src.n || (dst_t && dst_t.n != src.n)) fail("dst / dst_t size does not match src");
    const int f16 = src.t->scalar_type() == at::kHalf;
    void *s = stream();
    check(unlocked([&] {
        return p_mp8_quantize_e5m2(src.p, f16, (uint8_t *)dst.p, (uint8_t *)dst_t.p, rows, cols, scale, (mp8_round)round,
                                   flags, seed, offset, (mp8_stats *)stats.p, s);
    }), "mp8_quantize_e5m2");
}

void gemm(Args a) {
    const int op = a.op();
    const int64_t M = a.i64(), N = a.i64(), K = a.i64();
    const Arg x = a.tensor("a", kU8), y = a.tensor("b", kU8), out8 = a.tensor("out8", kU8), out8_t = a.tensor("out8_t", kU8),
              acc = a.tensor("acc", kF32);
    const int acc_mode = a.i32();
    const float alpha = a.f32();
    const int round = a.i32(), flags = a.i32();
    const uint64_t seed = a.u64(), offset = a.u64();
    const Arg stats = a.raw(), ws = a.raw(true);
    int64_t rows, cols, kc;
    op_dims(op, M, N, K, rows, cols, kc);
    const bool a_km = (flags & MP8_FLAG_A_CONTRACTION_MAJOR) != 0, b_km = (flags & MP8_FLAG_B_CONTRACTION_MAJOR) != 0;
    const int64_t lda = a.i64_or(a_km ? rows : kc), ldb = a.i64_or(b_km ? cols : kc);
    const int tile = a.i32(), split = a.i32();
    const bool fixed = a.flag();
    must_be(x, "a");
    must_be(y, "b");
    at_least(x, span(a_km, rows, kc, lda), "a", "its shape and leading dimension require");
    at_least(y, span(b_km, cols, kc, ldb), "b", "its shape and leading dimension require");
    const int64_t no = mul(rows, cols);
    at_least(out8, no, "out8", "rows*cols");
    at_least(out8_t, no, "out8_t", "rows*cols");
    at_least(acc, no, "acc", "rows*cols");
    void *s = stream();
    if (fixed) {
        if (ws || tile || split) fail("static_scratch takes no workspace, tile_config or split_k");
        check(unlocked([&] {
            return p_mp8_gemm_fp8_static((mp8_op)op, M, N, K, (const uint8_t *)x.p, lda, (const uint8_t *)y.p, ldb, alpha,
                                         (float *)acc.p, acc_mode, (uint8_t *)out8.p, (uint8_t *)out8_t.p,
                                         (mp8_round)round, flags, seed, offset, (mp8_stats *)stats.p, s);
        }), "mp8_gemm_fp8_static");
        return;
    }
    const size_t ws_bytes = a.bytes(ws);
    check(unlocked([&] {
        return p_mp8_gemm_fp8_tuned((mp8_op)op, M, N, K, (const uint8_t *)x.p, lda, (const uint8_t *)y.p, ldb, alpha,
                                    (float *)acc.p, acc_mode, (uint8_t *)out8.p, (uint8_t *)out8_t.p, (mp8_round)round,
                                    flags, seed, offset, (mp8_stats *)stats.p, ws.p, ws_bytes, s, tile, split);
    }), "mp8_gemm_fp8");
}

void quantize_gemm_fwd(Args a) {
    const int64_t M = a.i64(), N = a.i64(), K = a.i64();
    const Arg x = a.tensor("x", kF32), x8 = a.tensor("x8_out", kU8), w8 = a.tensor("w8", kU8), out8 = a.tensor("out8", kU8),
              out8_t = a.tensor("out8_t", kU8), acc = a.tensor("acc", kF32);
    const int acc_mode = a.i32();
    const float x_scale = a.f32();
    const int x_round = a.i32(), x_flags = a.i32();
    const uint64_t x_seed = a.u64(), x_offset = a.u64();
    const Arg x_stats = a.raw();
    const float alpha = a.f32();
    const int round = a.i32(), flags = a.i32();
    const uint64_t seed = a.u64(), offset = a.u64();
    const Arg stats = a.raw(), ws = a.raw(true);
    const int64_t ldw = a.i64_or(N);
    must_be(x, "x");
    must_be(x8, "x8_out");
    must_be(w8, "w8");
    const int64_t nx = mul(M, K), no = mul(M, N);
    if (x.n != nx || x8.n != nx) fail("x and x8_out must have M*K elements");
    at_least(w8, span(true, N, K, ldw), "w8", "its shape and leading dimension require");
    at_least(out8, no, "out8", "M*N");
    at_least(out8_t, no, "out8_t", "M*N");
    at_least(acc, no, "acc", "M*N");
    void *s = stream();
    const size_t ws_bytes = a.bytes(ws);
    check(unlocked([&] {
        return p_mp8_quantize_gemm_fwd_fp8(M, N, K, (const float *)x.p, x_scale, (mp8_round)x_round, x_flags, x_seed, x_offset,
                                           (mp8_stats *)x_stats.p, (uint8_t *)x8.p, (const uint8_t *)w8.p, ldw, alpha,
                                           (float *)acc.p, acc_mode, (uint8_t *)out8.p, (uint8_t *)out8_t.p,
                                           (mp8_round)round, flags, seed, offset, (mp8_stats *)stats.p, ws.p, ws_bytes, s);
    }), "mp8_quantize_gemm_fwd_fp8");
}

struct ConvDims {
    int64_t B, H, W, Cin, Cout;
    explicit ConvDims(Args &a) : B(a.i64()), H(a.i64()), W(a.i64()), Cin(a.i64()), Cout(a.i64()) {}
    int64_t prows(Args &a) const {  // default: B*(H+2)*(W+2) up to a multiple of 128
        return a.i64_or(mul(add(mul(mul(B, add(H, 2)), add(W, 2)), 127) / 128, 128));
    }
};

// W + 3 rows of `channels` elements are readable on both sides of the padded tensor.
bool has_guard(const Arg &a, int64_t guard) {
    const int64_t first = a.t->storage_offset();
    const int64_t after = (int64_t)(a.t->storage().nbytes() / a.t->element_size()) - (first + a.n);
    return first >= guard && after >= guard;
}

void conv(Args a) {
    const int op = a.op();
    const ConvDims d(a);
    const Arg x = a.tensor("a", kU8), y = a.tensor("b", kU8), out8 = a.tensor("out8", kU8), acc = a.tensor("acc", kF32);
    const int acc_mode = a.i32();
    const float alpha = a.f32();
    const int round = a.i32(), flags = a.i32();
    const uint64_t seed = a.u64(), offset = a.u64();
    const Arg stats = a.raw(), ws = a.raw(true);
    const int64_t prows = d.prows(a);
    must_be(x, "a");
    must_be(y, "b");
    const int64_t w = mul(mul(9, d.Cin), d.Cout), px = mul(prows, d.Cin), py = mul(prows, d.Cout);
    int64_t na, nb, no;
    switch (op) {
        case MP8_FWD: na = px; nb = w; no = py; break;
        case MP8_BWD_DATA: na = py; nb = w; no = px; break;
        default: na = px; nb = py; no = w; break;  // MP8_WGRAD
    }
    if (x.n != na || y.n != nb) fail("a / b do not have the sizes the operation implies");
    at_least(out8, no, "out8", "the output");
    at_least(acc, no, "acc", "the output");
    if (!has_guard(x, mul(add(d.W, 3), op == MP8_BWD_DATA ? d.Cout : d.Cin)))
        fail("the padded tensor `a` needs W+3 readable guard rows before and after (allocate it with conv_buffer)");
    void *s = stream();
    const size_t ws_bytes = a.bytes(ws);
    check(unlocked([&] {
        return p_mp8_conv3x3_fp8((mp8_op)op, d.B, d.H, d.W, d.Cin, d.Cout, prows, (const uint8_t *)x.p, (const uint8_t *)y.p,
                                 alpha, (float *)acc.p, acc_mode, (uint8_t *)out8.p, (mp8_round)round, flags, seed, offset,
                                 (mp8_stats *)stats.p, ws.p, ws_bytes, s);
    }), "mp8_conv3x3_fp8");
}

// What the weight-gradient calls with an update share, after their operands: g8_out, alpha,
// g_round, flags, g_seed, g_offset, stats, w_round, w_seed, w_offset, skip, w8_out, workspace.
struct UpdateArgs {
    Arg g8;
    float alpha;
    int g_round, flags;
    uint64_t g_seed, g_offset;
    Arg stats;
    int w_round;
    uint64_t w_seed, w_offset;
    Arg skip, w8, ws;
    explicit UpdateArgs(Args &a) {
        g8 = a.tensor("g8_out", kU8);
        alpha = a.f32();
        g_round = a.i32();
        flags = a.i32();
        g_seed = a.u64();
        g_offset = a.u64();
        stats = a.raw();
        w_round = a.i32();
        w_seed = a.u64();
        w_offset = a.u64();
        skip = a.raw();
        w8 = a.tensor("w8_out", kU8);
        ws = a.raw(true);
    }
};

// rule: 0 plain SGD, 1 momentum, 2 ADAM
template <int RULE>
void wgrad_update(Args a) {
    const int64_t M = a.i64(), N = a.i64(), K = a.i64();
    const Arg x = a.tensor("a", kU8), y = a.tensor("b", kU8), w16 = a.tensor("w16", kHalf);
    Arg s0, s1;
    if (RULE == 1) s0 = a.tensor("velocity", kF32);
    if (RULE == 2) s0 = a.tensor("m", kF32), s1 = a.tensor("v", kF32);
    const float lr = a.f32(), inv = a.f32();
    float mu = 0, wd = 0, b1 = 0, b2 = 0, eps = 0;
    int64_t step = 0;
    if (RULE == 1) mu = a.f32(), wd = a.f32();
    if (RULE == 2) step = a.whole(), b1 = a.f32(), b2 = a.f32(), eps = a.f32(), wd = a.f32();
    const UpdateArgs u(a);
    const bool a_km = (u.flags & MP8_FLAG_A_CONTRACTION_MAJOR) != 0, b_km = (u.flags & MP8_FLAG_B_CONTRACTION_MAJOR) != 0;
    const int64_t lda = a.i64_or(a_km ? K : M), ldb = a.i64_or(b_km ? N : M);
    must_be(x, "a");
    must_be(y, "b");
    if (x.n < span(a_km, K, M, lda) || y.n < span(b_km, N, M, ldb))
        fail("a / b is smaller than its shape and leading dimension require");
    const int64_t n = mul(K, N);
    exactly(w16, n, "w16", "K*N");
    exactly(s0, n, RULE == 1 ? "velocity" : "m", "K*N");
    exactly(s1, n, "v", "K*N");
    exactly(u.g8, n, "g8_out", "K*N");
    exactly(u.w8, n, "w8_out", "K*N");
    void *s = stream();
    const size_t ws_bytes = a.bytes(u.ws);
    const uint8_t *ap = (const uint8_t *)x.p, *bp = (const uint8_t *)y.p;
    uint8_t *g8 = (uint8_t *)u.g8.p, *w8 = (uint8_t *)u.w8.p;
    mp8_stats *st = (mp8_stats *)u.stats.p;
    const uint32_t *skip = (const uint32_t *)u.skip.p;
    const mp8_round gr = (mp8_round)u.g_round, wr = (mp8_round)u.w_round;
    uint16_t *w = (uint16_t *)w16.p;
    if (RULE == 0)
        check(unlocked([&] {
            return p_mp8_wgrad_update_fp16_sr(M, N, K, ap, lda, bp, ldb, u.alpha, g8, gr, u.flags, u.g_seed, u.g_offset, st,
                                              w, lr, inv, wr, u.w_seed, u.w_offset, skip, w8, u.ws.p, ws_bytes, s);
        }), "mp8_wgrad_update_fp16_sr");
    else if (RULE == 1)
        check(unlocked([&] {
            return p_mp8_wgrad_momentum_fp16_sr(M, N, K, ap, lda, bp, ldb, u.alpha, g8, gr, u.flags, u.g_seed, u.g_offset, st,
                                                w, (float *)s0.p, lr, inv, mu, wd, wr, u.w_seed, u.w_offset, skip, w8,
                                                u.ws.p, ws_bytes, s);
        }), "mp8_wgrad_momentum_fp16_sr");
    else
        check(unlocked([&] {
            return p_mp8_wgrad_adam_fp16_sr(M, N, K, ap, lda, bp, ldb, u.alpha, g8, gr, u.flags, u.g_seed, u.g_offset, st, w,
                                            (float *)s0.p, (float *)s1.p, lr, inv, b1, b2, eps, wd, step, wr, u.w_seed,
                                            u.w_offset, skip, w8, u.ws.p, ws_bytes, s);
        }), "mp8_wgrad_adam_fp16_sr");
}

// rule: 0 plain SGD, 1 momentum
template <int RULE>
void conv_wgrad_update(Args a) {
    const ConvDims d(a);
    const Arg x8 = a.tensor("x8", kU8), e8 = a.tensor("e8", kU8), w16 = a.tensor("w16", kHalf);
    Arg vel;
    if (RULE == 1) vel = a.tensor("velocity", kF32);
    const float lr = a.f32(), inv = a.f32();
    float mu = 0, wd = 0;
    if (RULE == 1) mu = a.f32(), wd = a.f32();
    const UpdateArgs u(a);
    const int64_t prows = d.prows(a), n = mul(mul(9, d.Cin), d.Cout);
    must_be(x8, "x8");
    must_be(e8, "e8");
    if (x8.n != mul(prows, d.Cin) || e8.n != mul(prows, d.Cout)) fail("x8 / e8 do not have the sizes the operation implies");
    exactly(w16, n, "w16", "9*Cin*Cout");
    exactly(vel, n, "velocity", "9*Cin*Cout");
    exactly(u.g8, n, "g8_out", "9*Cin*Cout");
    exactly(u.w8, n, "w8_out", "9*Cin*Cout");
    if (!has_guard(x8, mul(add(d.W, 3), d.Cin)))
        fail("the padded tensor x8 needs W+3 readable guard rows before and after (allocate it with conv_buffer)");
    void *s = stream();
    const size_t ws_bytes = a.bytes(u.ws);
    const uint8_t *xp = (const uint8_t *)x8.p, *ep = (const uint8_t *)e8.p;
    uint8_t *g8 = (uint8_t *)u.g8.p, *w8 = (uint8_t *)u.w8.p;
    mp8_stats *st = (mp8_stats *)u.stats.p;
    const uint32_t *skip = (const uint32_t *)u.skip.p;
    const mp8_round gr = (mp8_round)u.g_round, wr = (mp8_round)u.w_round;
    uint16_t *w = (uint16_t *)w16.p;
    if (RULE == 0)
        check(unlocked([&] {
            return p_mp8_conv3x3_wgrad_update_fp16_sr(d.B, d.H, d.W, d.Cin, d.Cout, prows, xp, ep, u.alpha, g8, gr, u.flags,
                                                      u.g_seed, u.g_offset, st, w, lr, inv, wr, u.w_seed, u.w_offset, skip,
                                                      w8, u.ws.p, ws_bytes, s);
        }), "mp8_conv3x3_wgrad_update_fp16_sr");
    else
        check(unlocked([&] {
            return p_mp8_conv3x3_wgrad_momentum_fp16_sr(d.B, d.H, d.W, d.Cin, d.Cout, prows, xp, ep, u.alpha, g8, gr, u.flags,
                                                        u.g_seed, u.g_offset, st, w, (float *)vel.p, lr, inv, mu, wd, wr,
                                                        u.w_seed, u.w_offset, skip, w8, u.ws.p, ws_bytes, s);
        }), "mp8_conv3x3_wgrad_momentum_fp16_sr");
}

// rule: 0 plain SGD, 1 momentum, 2 ADAM
template <int RULE>
void update(Args a) {
    const Arg w16 = a.tensor("w16", kHalf);
    Arg s0, s1;
    if (RULE == 1) s0 = a.tensor("velocity", kF32);
    if (RULE == 2) s0 = a.tensor("m", kF32), s1 = a.tensor("v", kF32);
    const Arg g8 = a.tensor("g8", kU8);
    const float lr = a.f32(), inv = a.f32();
    float mu = 0, wd = 0, b1 = 0, b2 = 0, eps = 0;
    int64_t step = 0;
    if (RULE == 1) mu = a.f32(), wd = a.f32();
    if (RULE == 2) step = a.whole(), b1 = a.f32(), b2 = a.f32(), eps = a.f32(), wd = a.f32();
    const int round = a.i32();
    const uint64_t seed = a.u64(), offset = a.u64();
    const Arg skip = a.raw(), w8 = a.tensor("w8_out", kU8), stats = a.raw();
    must_be(w16, "w16");
    must_be(g8, "g8");
    if (RULE > 0) must_be(s0, RULE == 1 ? "velocity" : "m");
    if (RULE > 1) must_be(s1, "v");
    const int64_t n = w16.n;
    if (g8.n != n || (RULE > 0 && s0.n != n) || (RULE > 1 && s1.n != n) || (w8 && w8.n != n))
        fail(RULE == 0 ? "g8 / w8_out size does not match w16"
                       : RULE == 1 ? "velocity / g8 / w8_out size does not match w16"
                                   : "m / v / g8 / w8_out size does not match w16");
    void *s = stream();
    uint16_t *w = (uint16_t *)w16.p;
    const uint8_t *g = (const uint8_t *)g8.p;
    uint8_t *o8 = (uint8_t *)w8.p;
    const uint32_t *sk = (const uint32_t *)skip.p;
    mp8_stats *st = (mp8_stats *)stats.p;
    const mp8_round r = (mp8_round)round;
    if (RULE == 0)
        check(unlocked([&] { return p_mp8_sgd_update_fp16_sr(w, g, n, lr, inv, r, seed, offset, sk, o8, st, s); }),
              "mp8_sgd_update_fp16_sr");
    else if (RULE == 1)
        check(unlocked([&] {
            return p_mp8_sgd_momentum_fp16_sr(w, (float *)s0.p, g, n, lr, inv, mu, wd, r, seed, offset, sk, o8, st, s);
        }), "mp8_sgd_momentum_fp16_sr");
    else
        check(unlocked([&] {
            return p_mp8_adam_fp16_sr(w, (float *)s0.p, (float *)s1.p, g, n, lr, inv, b1, b2, eps, wd, step, r, seed, offset,
                                      sk, o8, st, s);
        }), "mp8_adam_fp16_sr");
}

template <void (*F)(Args)>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    try {
        F(Args{args, n});
    } catch (const Raised &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    Py_RETURN_NONE;
}

// init(error class, {entry point name: address})
PyObject *init(PyObject *, PyObject *args) {
    PyObject *error, *table;
    if (!PyArg_ParseTuple(args, "OO!", &error, &PyDict_Type, &table)) return nullptr;
#define MP8_TAKE(name)                                                             \
    {                                                                              \
        PyObject *v = PyDict_GetItemString(table, #name);                          \
        void *p = v ? PyLong_AsVoidPtr(v) : nullptr;                               \
        if (!p) {                                                                  \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);          \
            return nullptr;                                                        \
        }                                                                          \
        p_##name = (decltype(&name))p;                                             \
    }
    MP8_ENTRIES(MP8_TAKE)
#undef MP8_TAKE
    Py_INCREF(error);
    Py_XSETREF(g_error, error);
    Py_RETURN_NONE;
}

#define MP8_METHOD(name, fn) {name, (PyCFunction)(void *)entry<fn>, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    {"init", init, METH_VARARGS, nullptr},
    MP8_METHOD("quantize_e5m2", quantize),
    MP8_METHOD("gemm_fp8", gemm),
    MP8_METHOD("quantize_gemm_fwd_fp8", quantize_gemm_fwd),
    MP8_METHOD("conv3x3_fp8", conv),
    MP8_METHOD("wgrad_update_fp16_sr", wgrad_update<0>),
    MP8_METHOD("wgrad_momentum_fp16_sr", wgrad_update<1>),
    MP8_METHOD("wgrad_adam_fp16_sr", wgrad_update<2>),
    MP8_METHOD("conv3x3_wgrad_update_fp16_sr", conv_wgrad_update<0>),
    MP8_METHOD("conv3x3_wgrad_momentum_fp16_sr", conv_wgrad_update<1>),
    MP8_METHOD("sgd_update_fp16_sr", update<0>),
    MP8_METHOD("sgd_momentum_fp16_sr", update<1>),
    MP8_METHOD("adam_fp16_sr", update<2>),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&kModule); }
