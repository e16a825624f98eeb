// The calls that a training step makes, from Python without ctypes: argument checks, addresses and the current stream
// are read from the tensor objects here.  A wrapper in binding.py costs the host 5.4 us a call through ctypes, half of it
// the kernel launch; through this module 2.9.
//
// Every function takes the arguments of the wrapper of the same name, the stream last, and returns None when the library
// said OK and its status otherwise.  What is not plain -- a tensor subclass or a wrapped tensor, a tensor that is not on
// the GPU or not contiguous, a number that is not a Python int or float or does not fit, shapes or types that do not
// agree -- is not judged here: NotImplemented sends the wrapper to its general path, which serves the call or raises.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cfloat>
#include <climits>
#include <cstdint>
#include <vector>

#include "slimfit.h"

namespace {

// the library's functions, as loaded by binding.py
#define SLIMFIT_CALLS(X)                                                                                               \
    X(quant_pack) X(dequant_unpack) X(gelu_quant_pack) X(gelu_backward_dequant) X(prune_scores) X(restore_scores)      \
    X(softmax_prune) X(softmax_backward_pruned) X(prune_global_standardized) X(prune_global_workspace)                 \
    X(layernorm_forward) X(layernorm_backward) X(layernorm_backward_pruned) X(layernorm_forward_quant_pack)            \
    X(layernorm_backward_dequant) X(layernorm_param_grads) X(layernorm_param_grads_workspace) X(layer_delta_run)         \
    X(split_heads) X(merge_heads) X(product)
#define X(name) decltype(&slimfit_##name) name##_fn = nullptr;
SLIMFIT_CALLS(X)
#undef X
bool bound = false;

// Positional arguments, read in order.  ok turns false at the first that is not plain; what was read then is not used.
struct Args {
    PyObject *const *at;
    Py_ssize_t left;
    bool ok;

    Args(PyObject *const *args, Py_ssize_t n, Py_ssize_t want) : at(args), left(n), ok(bound && n == want) {}
    PyObject *next()
    {
        if (left <= 0) { ok = false; return Py_None; }
        --left;
        return *at++;
    }
    const at::Tensor *tensor()
    {
        PyObject *o = next();
        if (!THPVariable_CheckExact(o)) { ok = false; return nullptr; }
        const at::Tensor &t = THPVariable_Unpack(o);
        constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                               c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Batched,
                                               c10::DispatchKey::Functionalize, c10::DispatchKey::Negative,
                                               c10::DispatchKey::Conjugate, c10::DispatchKey::ZeroTensor});
        if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || t.key_set().has_any(wrapped) || !t.has_storage() ||
            !t.is_contiguous()) {
            ok = false;
            return nullptr;
        }
        return &t;
    }
    const at::Tensor *tensor_or_none()
    {
        if (left > 0 && *at == Py_None) { next(); return nullptr; }
        return tensor();
    }
    int64_t i64()
    {
        PyObject *o = next();
        if (!PyLong_Check(o)) { ok = false; return 0; }
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow) ok = false;
        return v;
    }
    int32_t i32()
    {
        const int64_t v = i64();
        if (v < INT32_MIN || v > INT32_MAX) { ok = false; return 0; }
        return (int32_t)v;
    }
    float f32()
    {
        PyObject *o = next();
        if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
        if (!PyLong_Check(o)) { ok = false; return 0.0f; }
        const double v = PyLong_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return (float)v;
    }
    int32_t truth()                                         // what bool() makes of it
    {
        const int v = PyObject_IsTrue(next());
        if (v < 0) { PyErr_Clear(); ok = false; }
        return v > 0;
    }
    bool own_stream = false;                                // the caller named a stream
    void *stream()
    {
        PyObject *o = next();
        if (!ok) return nullptr;
        if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
        own_stream = true;
        if (!PyLong_CheckExact(o)) { ok = false; return nullptr; }
        void *s = PyLong_AsVoidPtr(o);
        if (!s && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return s;
    }
    void need(bool agrees) { ok = ok && agrees; }
};

PyObject *general() { Py_RETURN_NOTIMPLEMENTED; }
PyObject *status(int32_t rc)
{
    if (rc == SLIMFIT_OK) Py_RETURN_NONE;
    return PyLong_FromLong(rc);
}
// the call itself, without the interpreter lock; `...` reads tensors only through pointers taken before
#define SLIMFIT_RUN(...)                                    \
    int32_t rc;                                             \
    Py_BEGIN_ALLOW_THREADS rc = (__VA_ARGS__);              \
    Py_END_ALLOW_THREADS return status(rc)

bool is(const at::Tensor *t, at::ScalarType s) { return t->scalar_type() == s; }
bool f32(const at::Tensor *t) { return is(t, at::kFloat); }
bool activation(const at::Tensor *t) { return f32(t) || is(t, at::kBFloat16); }
bool same_type(const at::Tensor *a, const at::Tensor *b) { return a->scalar_type() == b->scalar_type(); }
int32_t dtype_of(const at::Tensor *t) { return f32(t) ? SLIMFIT_F32 : SLIMFIT_BF16; }
template <typename P = void> P *ptr(const at::Tensor *t) { return t ? static_cast<P *>(t->data_ptr()) : nullptr; }

// codes / scales hold what Alg. 2 writes for n elements (bad bits or block values are left to the library)
bool cache_fits(int64_t n, int32_t mode, int32_t bits, int32_t block, const at::Tensor *codes, const at::Tensor *scales)
{
    if (!is(codes, at::kByte) || (scales && !f32(scales))) return false;
    if ((bits == 4 || bits == 8) && codes->numel() < (n * bits + 7) / 8) return false;
    if (mode == SLIMFIT_Q_BLOCK && (block == 32 || block == 64 || block == 128 || block == 256) &&
        (!scales || scales->numel() < (n + block - 1) / block))
        return false;
    return true;
}
bool rows_of(const at::Tensor *t, int64_t &rows, int64_t &cols)
{
    if (t->dim() != 2) return false;
    rows = t->size(0);
    cols = t->size(1);
    return cols <= INT32_MAX;
}

PyObject *quant_pack(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 8);
    const at::Tensor *x = a.tensor();
    const int32_t mode = a.i32(), bits = a.i32(), block = a.i32(), frac = a.i32();
    const at::Tensor *codes = a.tensor(), *scales = a.tensor_or_none();
    void *st = a.stream();
    if (a.ok) a.need(activation(x) && cache_fits(x->numel(), mode, bits, block, codes, scales));
    if (!a.ok) return general();
    const void *xp = ptr(x);
    const int32_t dt = dtype_of(x);
    const int64_t n = x->numel();
    auto *cp = ptr<uint8_t>(codes);
    auto *sp = ptr<float>(scales);
    SLIMFIT_RUN(quant_pack_fn(xp, dt, n, mode, bits, block, frac, cp, sp, st));
}

PyObject *dequant_unpack(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 8);
    const at::Tensor *codes = a.tensor(), *scales = a.tensor_or_none();
    const int32_t mode = a.i32(), bits = a.i32(), block = a.i32(), frac = a.i32();
    const at::Tensor *y = a.tensor();
    void *st = a.stream();
    if (a.ok) a.need(activation(y) && cache_fits(y->numel(), mode, bits, block, codes, scales));
    if (!a.ok) return general();
    auto *cp = ptr<uint8_t>(codes);
    auto *sp = ptr<float>(scales);
    void *yp = ptr(y);
    const int32_t dt = dtype_of(y);
    const int64_t n = y->numel();
    SLIMFIT_RUN(dequant_unpack_fn(cp, sp, n, mode, bits, block, frac, yp, dt, st));
}

PyObject *gelu_quant_pack(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 9);
    const at::Tensor *x = a.tensor();
    const int32_t mode = a.i32(), bits = a.i32(), block = a.i32(), frac = a.i32();
    const at::Tensor *y = a.tensor(), *codes = a.tensor(), *scales = a.tensor_or_none();
    void *st = a.stream();
    if (a.ok)
        a.need(activation(x) && same_type(x, y) && x->numel() == y->numel() &&
               cache_fits(x->numel(), mode, bits, block, codes, scales));
    if (!a.ok) return general();
    const void *xp = ptr(x);
    void *yp = ptr(y);
    auto *cp = ptr<uint8_t>(codes);
    auto *sp = ptr<float>(scales);
    const int32_t dt = dtype_of(x);
    const int64_t n = x->numel();
    SLIMFIT_RUN(gelu_quant_pack_fn(xp, dt, n, mode, bits, block, frac, yp, cp, sp, st));
}

PyObject *gelu_backward_dequant(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 9);
    const at::Tensor *codes = a.tensor(), *scales = a.tensor_or_none();
    const int32_t mode = a.i32(), bits = a.i32(), block = a.i32(), frac = a.i32();
    const at::Tensor *dy = a.tensor(), *dx = a.tensor();
    void *st = a.stream();
    if (a.ok)
        a.need(activation(dx) && same_type(dx, dy) && dx->numel() == dy->numel() &&
               cache_fits(dx->numel(), mode, bits, block, codes, scales));
    if (!a.ok) return general();
    auto *cp = ptr<uint8_t>(codes);
    auto *sp = ptr<float>(scales);
    const void *gp = ptr(dy);
    void *xp = ptr(dx);
    const int32_t dt = dtype_of(dx);
    const int64_t n = dx->numel();
    SLIMFIT_RUN(gelu_backward_dequant_fn(cp, sp, n, mode, bits, block, frac, gp, xp, dt, st));
}

// vals / idx (/ counts) hold rows * k pairs
bool pairs_fit(int64_t rows, int64_t k, const at::Tensor *vals, const at::Tensor *idx)
{
    return k >= 0 && k <= INT32_MAX && is(idx, at::kUInt16) && vals->numel() >= rows * k && idx->numel() >= rows * k;
}
bool counts_fit(int64_t rows, const at::Tensor *counts) { return !counts || (is(counts, at::kInt) && counts->numel() >= rows); }

PyObject *prune_scores(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 8);
    const at::Tensor *p = a.tensor();
    const int32_t k = a.i32(), mode = a.i32();
    const float tau = a.f32();
    const at::Tensor *vals = a.tensor(), *idx = a.tensor(), *counts = a.tensor_or_none();
    void *st = a.stream();
    int64_t rows = 0, cols = 0;
    if (a.ok) a.need(rows_of(p, rows, cols) && activation(p) && same_type(p, vals) && pairs_fit(rows, k, vals, idx) && counts_fit(rows, counts));
    if (!a.ok) return general();
    const void *pp = ptr(p);
    void *vp = ptr(vals);
    auto *ip = ptr<uint16_t>(idx);
    auto *np = ptr<int32_t>(counts);
    const int32_t dt = dtype_of(p);
    SLIMFIT_RUN(prune_scores_fn(pp, dt, rows, (int32_t)cols, k, mode, tau, vp, ip, np, st));
}

PyObject *restore_scores(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 5);
    const at::Tensor *vals = a.tensor(), *idx = a.tensor(), *counts = a.tensor_or_none(), *out = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, cols = 0, k = 0, have = 0;
    if (a.ok)
        a.need(rows_of(out, rows, cols) && rows_of(vals, have, k) && activation(out) && same_type(out, vals) && is(idx, at::kUInt16) &&
               have >= rows && idx->numel() >= rows * k && counts_fit(rows, counts));
    if (!a.ok) return general();
    const void *vp = ptr(vals);
    auto *ip = ptr<uint16_t>(idx);
    auto *np = ptr<int32_t>(counts);
    void *op = ptr(out);
    const int32_t dt = dtype_of(out);
    SLIMFIT_RUN(restore_scores_fn(vp, ip, np, dt, rows, (int32_t)cols, (int32_t)k, op, st));
}

PyObject *softmax_prune(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 6);
    const at::Tensor *logits = a.tensor();
    const int32_t k = a.i32();
    const at::Tensor *probs = a.tensor(), *vals = a.tensor(), *idx = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, cols = 0;
    if (a.ok)
        a.need(rows_of(logits, rows, cols) && activation(logits) && probs->sizes() == logits->sizes() && same_type(logits, probs) &&
               same_type(logits, vals) && pairs_fit(rows, k, vals, idx));
    if (!a.ok) return general();
    const void *lp = ptr(logits);
    void *pp = ptr(probs), *vp = ptr(vals);
    auto *ip = ptr<uint16_t>(idx);
    const int32_t dt = dtype_of(logits);
    SLIMFIT_RUN(softmax_prune_fn(lp, dt, rows, (int32_t)cols, k, pp, vp, ip, st));
}

PyObject *softmax_backward_pruned(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 6);
    const at::Tensor *vals = a.tensor(), *idx = a.tensor(), *counts = a.tensor_or_none(), *dp = a.tensor(), *ds = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, cols = 0, k = 0, have = 0;
    if (a.ok)
        a.need(rows_of(dp, rows, cols) && rows_of(vals, have, k) && activation(dp) && ds->sizes() == dp->sizes() && same_type(dp, ds) &&
               same_type(dp, vals) && is(idx, at::kUInt16) && vals->sizes() == idx->sizes() && have >= rows && counts_fit(rows, counts));
    if (!a.ok) return general();
    const void *vp = ptr(vals), *gp = ptr(dp);
    auto *ip = ptr<uint16_t>(idx);
    auto *np = ptr<int32_t>(counts);
    void *sp = ptr(ds);
    const int32_t dt = dtype_of(dp);
    SLIMFIT_RUN(softmax_backward_pruned_fn(vp, ip, np, gp, dt, rows, (int32_t)cols, (int32_t)k, sp, st));
}

// The caller's workspace, or one from torch's allocator (given back when the wrapper returns; the allocator keeps the
// block for the current stream's later work).  Only a caller that brings one may name a stream.
struct Scratch {
    at::Tensor own;
    void *at = nullptr;
    size_t bytes = 0;
    bool take(const at::Tensor *given, bool own_stream, size_t need, const at::Tensor *like)
    {
        if (given) {
            if (!is(given, at::kByte)) return false;
            at = given->data_ptr();
            bytes = (size_t)given->numel();
            return true;
        }
        if (own_stream) return false;
        own = at::empty({(int64_t)need}, like->options().dtype(at::kByte).requires_grad(false));
        at = own.data_ptr();
        bytes = need;
        return true;
    }
};

PyObject *prune_global_standardized(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 11);
    const at::Tensor *x = a.tensor(), *mean = a.tensor(), *rstd = a.tensor();
    const int64_t k = a.i64();
    const at::Tensor *vals = a.tensor(), *idx = a.tensor();
    const int32_t by_magnitude = a.truth();
    const at::Tensor *tile_ptr = a.tensor_or_none(), *row_ptr = a.tensor_or_none(), *workspace = a.tensor_or_none();
    void *st = a.stream();
    int64_t rows = 0, H = 0, n = 0;
    size_t need = 0;
    if (a.ok) {
        n = x->numel();
        a.need(rows_of(x, rows, H) && activation(x) && f32(vals) && is(idx, at::kInt) && f32(mean) && f32(rstd) && mean->numel() >= rows &&
               rstd->numel() >= rows && vals->numel() >= k && idx->numel() >= k && n <= INT32_MAX &&
               (!tile_ptr || (is(tile_ptr, at::kInt) && tile_ptr->numel() >= (n + SLIMFIT_GLOBAL_TILE - 1) / SLIMFIT_GLOBAL_TILE + 1)) &&
               (!row_ptr || (is(row_ptr, at::kInt) && row_ptr->numel() >= rows + 1)));
    }
    if (a.ok && !workspace) a.need(prune_global_workspace_fn(n, &need) == SLIMFIT_OK);
    Scratch w;
    if (!a.ok || !w.take(workspace, a.own_stream, need, x)) return general();
    const void *xp = ptr(x);
    const float *mp = ptr<float>(mean), *rp = ptr<float>(rstd);
    void *vp = ptr(vals);
    int32_t *ip = ptr<int32_t>(idx), *tp = ptr<int32_t>(tile_ptr), *row = ptr<int32_t>(row_ptr);
    const int32_t dt = dtype_of(x);
    SLIMFIT_RUN(prune_global_standardized_fn(xp, dt, n, H, mp, rp, k, by_magnitude, vp, ip, tp, row, w.at, w.bytes, st));
}

PyObject *layernorm_forward(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 8);
    const at::Tensor *x = a.tensor(), *gamma = a.tensor(), *beta = a.tensor();
    const float eps = a.f32();
    const at::Tensor *y = a.tensor(), *mean = a.tensor(), *rstd = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, H = 0;
    if (a.ok)
        a.need(rows_of(x, rows, H) && activation(x) && y->sizes() == x->sizes() && same_type(x, y) && f32(gamma) && f32(beta) && f32(mean) &&
               f32(rstd) && gamma->numel() == H && beta->numel() == H && mean->numel() >= rows && rstd->numel() >= rows);
    if (!a.ok) return general();
    const void *xp = ptr(x);
    const float *gp = ptr<float>(gamma), *bp = ptr<float>(beta);
    void *yp = ptr(y);
    float *mp = ptr<float>(mean), *rp = ptr<float>(rstd);
    const int32_t dt = dtype_of(x);
    SLIMFIT_RUN(layernorm_forward_fn(xp, dt, gp, bp, rows, H, eps, yp, mp, rp, st));
}

PyObject *layernorm_backward(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 7);
    const at::Tensor *x = a.tensor(), *mean = a.tensor(), *rstd = a.tensor(), *gamma = a.tensor(), *dy = a.tensor(), *dx = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, H = 0;
    if (a.ok)
        a.need(rows_of(x, rows, H) && activation(x) && dy->sizes() == x->sizes() && dx->sizes() == x->sizes() && same_type(x, dy) &&
               same_type(x, dx) && f32(mean) && f32(rstd) && f32(gamma) && mean->numel() >= rows && rstd->numel() >= rows &&
               gamma->numel() == H);
    if (!a.ok) return general();
    const void *xp = ptr(x), *dyp = ptr(dy);
    const float *mp = ptr<float>(mean), *rp = ptr<float>(rstd), *gp = ptr<float>(gamma);
    void *dxp = ptr(dx);
    const int32_t dt = dtype_of(x);
    SLIMFIT_RUN(layernorm_backward_fn(xp, dt, mp, rp, gp, dyp, rows, H, dxp, st));
}

PyObject *layernorm_backward_pruned(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 9);
    const at::Tensor *vals = a.tensor(), *idx = a.tensor(), *row_ptr = a.tensor();
    const int64_t k = a.i64();
    const at::Tensor *rstd = a.tensor(), *gamma = a.tensor(), *dy = a.tensor(), *dx = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, H = 0;
    if (a.ok)
        a.need(rows_of(dy, rows, H) && activation(dy) && dx->sizes() == dy->sizes() && same_type(dx, dy) && f32(vals) && f32(rstd) &&
               f32(gamma) && is(idx, at::kInt) && is(row_ptr, at::kInt) && row_ptr->numel() >= rows + 1 && vals->numel() >= k &&
               idx->numel() >= k && rstd->numel() >= rows && gamma->numel() >= H);
    if (!a.ok) return general();
    const float *vp = ptr<float>(vals), *rp = ptr<float>(rstd), *gp = ptr<float>(gamma);
    const int32_t *ip = ptr<int32_t>(idx), *row = ptr<int32_t>(row_ptr);
    const void *dyp = ptr(dy);
    void *dxp = ptr(dx);
    const int32_t dt = dtype_of(dy);
    SLIMFIT_RUN(layernorm_backward_pruned_fn(vp, ip, row, k, rp, gp, dyp, dt, rows, H, dxp, st));
}

// codes / scales hold what the LayerNorm kernels write for rows of H elements (H is a multiple of the block)
bool row_cache_fits(int64_t rows, int64_t H, int32_t bits, int32_t block, const at::Tensor *codes, const at::Tensor *scales)
{
    return is(codes, at::kByte) && f32(scales) && bits >= 0 && bits <= 64 && codes->numel() >= rows * H * bits / 8 &&
           scales->numel() >= rows * H / (block > 1 ? block : 1);
}

PyObject *layernorm_forward_quant_pack(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 12);
    const at::Tensor *x = a.tensor(), *gamma = a.tensor(), *beta = a.tensor();
    const float eps = a.f32();
    const int32_t bits = a.i32(), block = a.i32();
    const at::Tensor *y = a.tensor(), *mean = a.tensor(), *rstd = a.tensor(), *codes = a.tensor(), *scales = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, H = 0;
    if (a.ok)
        a.need(rows_of(x, rows, H) && activation(x) && y->sizes() == x->sizes() && same_type(x, y) && f32(gamma) && f32(beta) && f32(mean) &&
               f32(rstd) && gamma->numel() == H && beta->numel() == H && mean->numel() >= rows && rstd->numel() >= rows &&
               row_cache_fits(rows, H, bits, block, codes, scales));
    if (!a.ok) return general();
    const void *xp = ptr(x);
    const float *gp = ptr<float>(gamma), *bp = ptr<float>(beta);
    void *yp = ptr(y);
    float *mp = ptr<float>(mean), *rp = ptr<float>(rstd), *sp = ptr<float>(scales);
    auto *cp = ptr<uint8_t>(codes);
    const int32_t dt = dtype_of(x);
    SLIMFIT_RUN(layernorm_forward_quant_pack_fn(xp, dt, gp, bp, rows, H, eps, bits, block, yp, mp, rp, cp, sp, st));
}

PyObject *layernorm_backward_dequant(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 10);
    const at::Tensor *codes = a.tensor(), *scales = a.tensor();
    const int32_t bits = a.i32(), block = a.i32();
    const at::Tensor *mean = a.tensor(), *rstd = a.tensor(), *gamma = a.tensor(), *dy = a.tensor(), *dx = a.tensor();
    void *st = a.stream();
    int64_t rows = 0, H = 0;
    if (a.ok)
        a.need(rows_of(dy, rows, H) && activation(dy) && dx->sizes() == dy->sizes() && same_type(dx, dy) && f32(mean) && f32(rstd) &&
               f32(gamma) && gamma->numel() == H && mean->numel() >= rows && rstd->numel() >= rows &&
               row_cache_fits(rows, H, bits, block, codes, scales));
    if (!a.ok) return general();
    const uint8_t *cp = ptr<uint8_t>(codes);
    const float *sp = ptr<float>(scales), *mp = ptr<float>(mean), *rp = ptr<float>(rstd), *gp = ptr<float>(gamma);
    const void *dyp = ptr(dy);
    void *dxp = ptr(dx);
    const int32_t dt = dtype_of(dy);
    SLIMFIT_RUN(layernorm_backward_dequant_fn(cp, sp, bits, block, mp, rp, gp, dyp, dt, rows, H, dxp, st));
}

PyObject *layernorm_param_grads(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 8);
    const at::Tensor *x = a.tensor(), *mean = a.tensor(), *rstd = a.tensor(), *dy = a.tensor(), *dgamma = a.tensor(), *dbeta = a.tensor(),
                     *workspace = a.tensor_or_none();
    void *st = a.stream();
    int64_t rows = 0, H = 0;
    size_t need = 0;
    if (a.ok)
        a.need(rows_of(x, rows, H) && activation(x) && dy->sizes() == x->sizes() && same_type(x, dy) && f32(mean) && f32(rstd) && f32(dgamma) &&
               f32(dbeta) && mean->numel() >= rows && rstd->numel() >= rows && dgamma->numel() == H && dbeta->numel() == H &&
               layernorm_param_grads_workspace_fn(rows, H, &need) == SLIMFIT_OK);
    Scratch w;
    if (!a.ok || !w.take(workspace, a.own_stream, need, x)) return general();
    const void *xp = ptr(x), *dyp = ptr(dy);
    const float *mp = ptr<float>(mean), *rp = ptr<float>(rstd);
    float *gp = ptr<float>(dgamma), *bp = ptr<float>(dbeta);
    const int32_t dt = dtype_of(x);
    SLIMFIT_RUN(layernorm_param_grads_fn(xp, dt, mp, rp, dyp, rows, H, gp, bp, w.at, w.bytes, st));
}

PyObject *layer_delta_run(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 8);
    PyObject *numel = a.next();
    const int32_t prev_dt = a.i32(), cur_dt = a.i32();
    const int32_t is_delta = a.truth();
    const float eps = a.f32();
    const at::Tensor *d = a.tensor(), *workspace = a.tensor();
    void *st = a.stream();
    a.need(PyList_CheckExact(numel) || PyTuple_CheckExact(numel));
    std::vector<int64_t> sizes;
    if (a.ok) {
        const Py_ssize_t L = PySequence_Fast_GET_SIZE(numel);
        a.need(L > 0 && L <= INT32_MAX && f32(d) && d->numel() >= L);
        Args each(PySequence_Fast_ITEMS(numel), L, L);
        sizes.reserve((size_t)L);
        for (Py_ssize_t i = 0; i < L && a.ok; ++i) sizes.push_back(each.i64());
        a.need(each.ok);
    }
    if (!a.ok) return general();
    float *dp = ptr<float>(d);
    void *wp = ptr(workspace);
    const size_t bytes = workspace->nbytes();
    SLIMFIT_RUN(layer_delta_run_fn(sizes.data(), (int32_t)sizes.size(), prev_dt, cur_dt, is_delta, eps, dp, wp, bytes, st));
}

bool heads_ok(const at::Tensor *qkv, const at::Tensor *q, const at::Tensor *kt, const at::Tensor *v)
{
    if (q->dim() != 4 || kt->dim() != 4 || qkv->dim() < 2 || qkv->numel() != 3 * q->numel()) return false;
    const int64_t batch = q->size(0), heads = q->size(1), tokens = q->size(2), dim = q->size(3);
    return heads <= INT32_MAX && tokens <= INT32_MAX && dim <= INT32_MAX && v->sizes() == q->sizes() && kt->size(0) == batch &&
           kt->size(1) == heads && kt->size(2) == dim && kt->size(3) == tokens && qkv->size(0) == batch && qkv->size(1) == tokens &&
           activation(qkv) && same_type(qkv, q) && same_type(qkv, kt) && same_type(qkv, v);
}

PyObject *split_heads(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 6);
    const at::Tensor *qkv = a.tensor();
    const float scale = a.f32();
    const at::Tensor *q = a.tensor(), *kt = a.tensor(), *v = a.tensor();
    void *st = a.stream();
    if (a.ok) a.need(heads_ok(qkv, q, kt, v));
    if (!a.ok) return general();
    const void *fp = ptr(qkv);
    void *qp = ptr(q), *kp = ptr(kt), *vp = ptr(v);
    const int64_t batch = q->size(0);
    const int32_t heads = (int32_t)q->size(1), tokens = (int32_t)q->size(2), dim = (int32_t)q->size(3), dt = dtype_of(qkv);
    SLIMFIT_RUN(split_heads_fn(fp, dt, batch, tokens, heads, dim, scale, qp, kp, vp, st));
}

PyObject *merge_heads(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 6);
    const at::Tensor *q = a.tensor(), *kt = a.tensor(), *v = a.tensor();
    const float scale = a.f32();
    const at::Tensor *qkv = a.tensor();
    void *st = a.stream();
    if (a.ok) a.need(heads_ok(qkv, q, kt, v));
    if (!a.ok) return general();
    void *fp = ptr(qkv);
    const void *qp = ptr(q), *kp = ptr(kt), *vp = ptr(v);
    const int64_t batch = q->size(0);
    const int32_t heads = (int32_t)q->size(1), tokens = (int32_t)q->size(2), dim = (int32_t)q->size(3), dt = dtype_of(qkv);
    SLIMFIT_RUN(merge_heads_fn(qp, kp, vp, dt, batch, tokens, heads, dim, scale, fp, st));
}

PyObject *product(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    Args a(args, n_args, 6);
    const at::Tensor *x = a.tensor(), *y = a.tensor();
    const int32_t y_deep = a.truth();
    const at::Tensor *out = a.tensor();
    a.tensor_or_none();                                     // a workspace, which the product does not need
    void *st = a.stream();
    int64_t M = 0, N = 0, K = 0;
    if (a.ok) {
        a.need(x->dim() == 2 && y->dim() == 2 && out->dim() == 2 && f32(x) && f32(y) && f32(out));
        if (a.ok) {
            M = x->size(0), K = x->size(1), N = y->size(y_deep ? 0 : 1);
            a.need(y->size(y_deep ? 1 : 0) == K && out->size(0) == M && out->size(1) == N);
        }
    }
    if (!a.ok) return general();
    const float *xp = ptr<float>(x), *yp = ptr<float>(y);
    float *op = ptr<float>(out);
    SLIMFIT_RUN(product_fn(xp, yp, y_deep, M, N, K, op, nullptr, 0, st));
}

// a C++ exception must not cross into the interpreter (torch's allocator raises one when memory runs out: the general
// path, which asks again, raises torch's own)
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    try {
        return F(self, args, n);
    } catch (...) {
        return general();
    }
}

// bind(addresses): the library's functions in the order of CALLS
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    void *address[32];
    Py_ssize_t want = 0;
#define X(name) ++want;
    SLIMFIT_CALLS(X)
#undef X
    if (n != want) {
        PyErr_SetString(PyExc_TypeError, "one address per function is expected");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        address[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_ssize_t i = 0;
#define X(name) name##_fn = reinterpret_cast<decltype(name##_fn)>(address[i++]);
    SLIMFIT_CALLS(X)
#undef X
    bound = true;
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&bind)), METH_FASTCALL, nullptr},
    METHOD(quant_pack), METHOD(dequant_unpack), METHOD(gelu_quant_pack), METHOD(gelu_backward_dequant), METHOD(prune_scores),
    METHOD(restore_scores), METHOD(softmax_prune), METHOD(softmax_backward_pruned), METHOD(prune_global_standardized),
    METHOD(layernorm_forward), METHOD(layernorm_backward), METHOD(layernorm_backward_pruned), METHOD(layernorm_forward_quant_pack),
    METHOD(layernorm_backward_dequant), METHOD(layernorm_param_grads), METHOD(layer_delta_run), METHOD(split_heads), METHOD(merge_heads),
    METHOD(product),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    PyObject *names = PyTuple_New(0);
#define X(name)                                                              \
    if (names) {                                                             \
        PyObject *one = Py_BuildValue("(s)", "slimfit_" #name), *all = one ? PySequence_Concat(names, one) : nullptr; \
        Py_XDECREF(one);                                                     \
        Py_DECREF(names);                                                    \
        names = all;                                                         \
    }
    SLIMFIT_CALLS(X)
#undef X
    // the torch whose headers this was compiled with: binding.py does not use it with another
    if (!names || PyModule_AddStringConstant(m, "TORCH", SLIMFIT_TORCH) < 0 || PyModule_AddObject(m, "CALLS", names) < 0) {
        Py_XDECREF(names);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
