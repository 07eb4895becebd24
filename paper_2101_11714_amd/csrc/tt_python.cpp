// Argument marshalling of the calls that a training or serving step makes, as a CPython extension: tensors are unpacked,
// checked and handed to the C ABI of libtt_emb.so here, where the same work in Python (ctypes objects, a dozen tensor
// attributes and the current stream, per call) took 6-9 us, more than most of the kernels of a step.  Host time of a pass:
// a forward of 64 lookups 8.7 -> 3.4 us, the two calls of the Kaggle-shaped step 20 -> 7 us, of which the launches are 2-3 us each.
// Every function takes its arguments by position, returns the library's return code, and raises AssertionError for a
// tensor of the wrong device, type, layout or size.  binding.py documents and wraps them.  What torch throws on the way
// (a tensor without storage, as tracing and vmap make them) becomes a RuntimeError.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/tt_emb.h"

namespace {

// What a call has collected; `ok` turns false, with the Python error set, at the first argument that does not fit.
struct Args {
    PyObject *const *a;
    bool ok = true;

    explicit Args(PyObject *const *args, Py_ssize_t n, Py_ssize_t want) : a(args)
    {
        if (n != want) {
            PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
            ok = false;
        }
    }

    bool fail(const char *what)
    {
        if (ok) PyErr_SetString(PyExc_AssertionError, what);
        return ok = false;
    }

    const at::Tensor *tensor(PyObject *o)
    {
        if (!ok) return nullptr;
        if (!THPVariable_Check(o)) {
            PyErr_SetString(PyExc_TypeError, "a tensor is expected");
            ok = false;
            return nullptr;
        }
        return &THPVariable_Unpack(o);
    }

    // a contiguous device tensor of the given type: its address, and the number of its elements in *n
    void *dev(PyObject *o, at::ScalarType type, int64_t *n = nullptr)
    {
        const at::Tensor *t = tensor(o);
        if (!t) return nullptr;
        if (!t->is_cuda() || t->scalar_type() != type || !t->is_contiguous()) {
            fail("a contiguous device tensor of the right type is expected");
            return nullptr;
        }
        if (n) *n = t->numel();
        return t->data_ptr();
    }
    float *f32(int i, int64_t *n = nullptr) { return (float *)dev(a[i], at::kFloat, n); }
    int64_t *i64(int i, int64_t *n = nullptr) { return (int64_t *)dev(a[i], at::kLong, n); }
    uint8_t *u8(int i, int64_t *n = nullptr) { return (uint8_t *)dev(a[i], at::kByte, n); }
    float *f32_or_null(int i, int64_t *n = nullptr) { return ok && a[i] != Py_None ? f32(i, n) : nullptr; }

    // a contiguous array of the device, of whatever type (or pinned host memory, which the device reads and writes as well)
    void *bytes_or_null(int i, size_t *n)
    {
        *n = 0;
        if (!ok || a[i] == Py_None) return nullptr;
        const at::Tensor *t = tensor(a[i]);
        if (!t) return nullptr;
        if (!t->is_contiguous() || !(t->is_cuda() || t->is_pinned())) {
            fail("a contiguous workspace on the device is expected");
            return nullptr;
        }
        *n = (size_t)t->numel() * t->element_size();
        return t->data_ptr();
    }

    int64_t integer(int i)
    {
        if (!ok) return 0;
        const long long v = PyLong_AsLongLong(a[i]);
        if (v == -1 && PyErr_Occurred()) ok = false;
        return v;
    }
    float real(int i)
    {
        if (!ok) return 0.f;
        const double v = PyFloat_AsDouble(a[i]);
        if (v == -1.0 && PyErr_Occurred()) ok = false;
        return (float)v;
    }
    bool truth(int i)
    {
        const int v = ok ? PyObject_IsTrue(a[i]) : 0;
        if (v < 0) ok = false;
        return v > 0;
    }

    // offsets[n_bags + 1] or None; longer: a call that takes an array with more entries as well
    const int64_t *offsets(int i, int64_t n_bags, bool longer = false)
    {
        if (!ok || a[i] == Py_None) return nullptr;
        int64_t n = 0;
        const int64_t *p = i64(i, &n);
        if (ok && (longer ? n < n_bags + 1 : n != n_bags + 1)) fail("offsets must have n_bags + 1 entries");
        return p;
    }

    // the struct behind a ctypes structure (which outlives the call)
    const void *structure(PyObject *o, size_t size)
    {
        Py_buffer v;
        if (!ok) return nullptr;
        if (PyObject_GetBuffer(o, &v, PyBUF_SIMPLE) != 0) {
            ok = false;
            return nullptr;
        }
        const void *p = v.buf;
        const bool fits = (size_t)v.len == size;
        PyBuffer_Release(&v);
        if (!fits) {
            PyErr_SetString(PyExc_TypeError, "a structure of another size is expected");
            ok = false;
        }
        return p;
    }
    const tt_shape_t *shape(int i) { return (const tt_shape_t *)structure(a[i], sizeof(tt_shape_t)); }
    const void *member(int i, const char *name, size_t size)
    {
        if (!ok || a[i] == Py_None) return nullptr;
        PyObject *c = PyObject_GetAttrString(a[i], name);
        if (!c) {
            ok = false;
            return nullptr;
        }
        const void *p = structure(c, size);
        Py_DECREF(c);                                        // (its owner still holds it)
        return p;
    }
    const tt_cache_t *cache(int i) { return (const tt_cache_t *)member(i, "c", sizeof(tt_cache_t)); }
    const tt_freq_t *freq(int i) { return (const tt_freq_t *)member(i, "_c", sizeof(tt_freq_t)); }

    // three fp32 tensors; like: the sizes they must have, or null; n: their sizes, or null
    void cores(int i, float *p[3], const int64_t *like = nullptr, int64_t *n = nullptr)
    {
        if (!ok) return;
        PyObject *seq = PySequence_Fast(a[i], "three tensors are expected");
        if (!seq) {
            ok = false;
            return;
        }
        if (PySequence_Fast_GET_SIZE(seq) < 3) fail("three tensors are expected");
        for (int k = 0; ok && k < 3; ++k) {
            int64_t m = 0;
            p[k] = (float *)dev(PySequence_Fast_GET_ITEM(seq, k), at::kFloat, &m);
            if (ok && like && m != like[k]) fail("an array has another size than its core");
            if (n) n[k] = m;
        }
        Py_DECREF(seq);
    }
};

int64_t dim(const tt_shape_t *s) { return (int64_t)s->n[0] * s->n[1] * s->n[2]; }
int64_t t0_floats(const tt_shape_t *s) { return (int64_t)s->n[0] * s->n[1] * s->r[2]; }
void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

template <typename F>
PyObject *call(F f)
{
    void *st = stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// shape, cores, indices, offsets, n_bags: the first five arguments of the lookup calls
struct Lookup {
    const tt_shape_t *shape;
    float *cores[3] = {};
    int64_t sizes[3] = {};
    const int64_t *indices, *offsets;
    int64_t L = 0, n_bags;

    explicit Lookup(Args &g, bool longer_offsets = false)
    {
        shape = g.shape(0);
        g.cores(1, cores, nullptr, sizes);
        indices = g.i64(2, &L);
        n_bags = g.integer(4);
        offsets = g.offsets(3, n_bags, longer_offsets);
    }
};

#define TT_FUNCTION(name) PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t nargs)

// no C++ exception may leave a function that Python calls
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
TT_FUNCTION(guarded)
{
    try {
        return F(nullptr, args, nargs);
    } catch (const c10::Error &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// The calling thread may allocate although a stream is captured somewhere: what is enqueued on a stream that is not captured is no
// part of the graph, and by default an allocation of any thread would end the capture.
struct CaptureElsewhere {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool on = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~CaptureElsewhere()
    {
        if (on) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

// Scratch memory of torch's allocator for the current stream (the kernels that use it are enqueued there before it is given
// back), or nothing: while the stream is captured, since a graph's scratch memory has to live as long as the graph, and where
// there is no room for it.
at::DataPtr scratch(size_t bytes, void *st)
{
    const CaptureElsewhere guard;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (!bytes || hipStreamIsCapturing((hipStream_t)st, &status) != hipSuccess || status != hipStreamCaptureStatusNone) return {};
    try {
        return c10::GetAllocator(c10::DeviceType::CUDA)->allocate(bytes);
    } catch (const c10::OutOfMemoryError &) {
        return {};
    }
}

// shape cores indices offsets n_bags output alpha cache workspace
TT_FUNCTION(emb_fwd)
{
    Args g(args, nargs, 9);
    if (!g.ok) return nullptr;
    Lookup q(g);
    int64_t no = 0;
    size_t wsb;
    float *out = g.f32(5, &no);
    const float *alpha = g.f32_or_null(6);
    const tt_cache_t *cache = g.cache(7);
    void *ws = g.bytes_or_null(8, &wsb);
    if (g.ok && no != q.n_bags * dim(q.shape)) g.fail("output has another size");
    if (!g.ok) return nullptr;
    const int64_t cached = cache ? cache->K : 0;
    if (tt_emb_fwd_rows_pays(q.shape, q.L, q.n_bags, cached)) {
        const size_t bytes = tt_emb_fwd_rows_workspace_bytes(q.shape, q.L, q.n_bags);
        const at::DataPtr mem = scratch(bytes, stream());
        if (mem)
            return call([&](void *st) { return tt_emb_fwd_rows(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, out, mem.get(), bytes, st); });
    }
    return call([&](void *st) { return tt_emb_fwd(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, cache, out, ws, wsb, st); });
}

// shape cores indices offsets n_bags output alpha workspace
TT_FUNCTION(emb_fwd_rows)
{
    Args g(args, nargs, 8);
    if (!g.ok) return nullptr;
    Lookup q(g);
    int64_t no = 0;
    size_t wsb;
    float *out = g.f32(5, &no);
    const float *alpha = g.f32_or_null(6);
    void *ws = g.bytes_or_null(7, &wsb);
    if (g.ok && no != q.n_bags * dim(q.shape)) g.fail("output has another size");
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_emb_fwd_rows(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, out, ws, wsb, st); });
}

// shape cores indices offsets n_bags output t0 alpha cache
TT_FUNCTION(emb_fwd_keep_t0)
{
    Args g(args, nargs, 9);
    if (!g.ok) return nullptr;
    Lookup q(g);
    int64_t nt = 0;
    float *out = g.f32(5), *t0 = g.f32(6, &nt);
    const float *alpha = g.f32_or_null(7);
    const tt_cache_t *cache = g.cache(8);
    if (g.ok && nt < q.L * t0_floats(q.shape)) g.fail("t0 is too small");
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_emb_fwd_keep_t0(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, cache, out, t0, st); });
}

// shape cores indices offsets n_bags output workspace t0 alpha cache
TT_FUNCTION(emb_fwd_prepared)
{
    Args g(args, nargs, 10);
    if (!g.ok) return nullptr;
    Lookup q(g);
    int64_t no = 0, nt = 0, wsb = 0;
    float *out = g.f32(5, &no);
    uint8_t *ws = g.u8(6, &wsb);
    float *t0 = g.f32_or_null(7, &nt);
    const float *alpha = g.f32_or_null(8);
    const tt_cache_t *cache = g.cache(9);
    if (g.ok && t0 && nt < q.L * t0_floats(q.shape)) g.fail("t0 is too small");
    if (g.ok && no != q.n_bags * dim(q.shape)) g.fail("output has another size");
    if (!g.ok) return nullptr;
    return call([&](void *st) {
        return tt_emb_fwd_prepared(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, cache, out, t0, ws, (size_t)wsb, st);
    });
}

// shape cores indices offsets n_bags grad_output grad_cores alpha cache grad_cache workspace t0
TT_FUNCTION(emb_bwd)
{
    Args g(args, nargs, 12);
    if (!g.ok) return nullptr;
    Lookup q(g);
    size_t wsb;
    float *grads[3] = {};
    const float *go = g.f32(5);
    g.cores(6, grads, q.sizes);
    const float *alpha = g.f32_or_null(7);
    const tt_cache_t *cache = g.cache(8);
    float *gc = g.f32_or_null(9);
    void *ws = g.bytes_or_null(10, &wsb);
    const float *t0 = g.f32_or_null(11);
    const bool with_t0 = args[11] != Py_None;
    if (!g.ok) return nullptr;
    return call([&](void *st) {
        return with_t0 ? tt_emb_bwd_t0(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, cache, go, t0, grads, gc, ws, wsb, st)
                       : tt_emb_bwd(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, cache, go, grads, gc, ws, wsb, st);
    });
}

// shape indices offsets n_bags cache workspace kept_t0
TT_FUNCTION(emb_bwd_prepare)
{
    Args g(args, nargs, 7);
    if (!g.ok) return nullptr;
    int64_t L = 0;
    size_t wsb;
    const tt_shape_t *shape = g.shape(0);
    const int64_t *indices = g.i64(1, &L);
    const int64_t n_bags = g.integer(3);
    const int64_t *offsets = g.offsets(2, n_bags, true);
    const tt_cache_t *cache = g.cache(4);
    void *ws = g.bytes_or_null(5, &wsb);
    const bool kept = g.truth(6);
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_emb_bwd_prepare(shape, indices, L, offsets, n_bags, cache, kept ? 1 : 0, ws, wsb, st); });
}

// shape cores cores_out indices offsets n_bags grad_output lr alpha cache workspace t0 prepared
TT_FUNCTION(emb_bwd_sgd)
{
    Args g(args, nargs, 13);
    if (!g.ok) return nullptr;
    int64_t L = 0, sizes[3];
    size_t wsb;
    float *cores[3] = {}, *outs[3] = {};
    const tt_shape_t *shape = g.shape(0);
    g.cores(1, cores, nullptr, sizes);
    g.cores(2, outs, sizes);
    const int64_t *indices = g.i64(3, &L);
    const int64_t n_bags = g.integer(5);
    const int64_t *offsets = g.offsets(4, n_bags);
    const float *go = g.f32(6);
    const float lr = g.real(7);
    const float *alpha = g.f32_or_null(8);
    const tt_cache_t *cache = g.cache(9);
    void *ws = g.bytes_or_null(10, &wsb);
    const float *t0 = g.f32_or_null(11);
    const bool with_t0 = args[11] != Py_None, prepared = g.truth(12);
    if (!g.ok) return nullptr;
    return call([&](void *st) {
        if (prepared) return tt_emb_bwd_sgd_prepared(shape, cores, outs, indices, L, offsets, n_bags, alpha, cache, go, t0, lr, ws, wsb, st);
        if (with_t0) return tt_emb_bwd_sgd_t0(shape, cores, outs, indices, L, offsets, n_bags, alpha, cache, go, t0, lr, ws, wsb, st);
        return tt_emb_bwd_sgd(shape, cores, outs, indices, L, offsets, n_bags, alpha, cache, go, lr, ws, wsb, st);
    });
}

// shape indices kept cache
TT_FUNCTION(emb_kept_prepare)
{
    Args g(args, nargs, 4);
    if (!g.ok) return nullptr;
    int64_t L = 0, kb = 0;
    const tt_shape_t *shape = g.shape(0);
    const int64_t *indices = g.i64(1, &L);
    uint8_t *kept = g.u8(2, &kb);
    const tt_cache_t *cache = g.cache(3);
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_emb_kept_prepare(shape, indices, L, cache, kept, (size_t)kb, st); });
}

// shape cores indices offsets n_bags output kept alpha cache lists_ready
TT_FUNCTION(emb_fwd_keep)
{
    Args g(args, nargs, 10);
    if (!g.ok) return nullptr;
    Lookup q(g);
    int64_t kb = 0;
    float *out = g.f32(5);
    uint8_t *kept = g.u8(6, &kb);
    const float *alpha = g.f32_or_null(7);
    const tt_cache_t *cache = g.cache(8);
    const bool ready = g.truth(9);
    if (!g.ok) return nullptr;
    return call([&](void *st) {
        return tt_emb_fwd_keep(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, cache, out, kept, (size_t)kb, ready ? 1 : 0, st);
    });
}

// the (indices, kept) pair of the next batch, or None
const tt_next_batch_t *next_batch(Args &g, int i, tt_next_batch_t *nb)
{
    if (!g.ok || g.a[i] == Py_None) return nullptr;
    PyObject *seq = PySequence_Fast(g.a[i], "next_batch is a pair (indices, kept)");
    if (!seq) {
        g.ok = false;
        return nullptr;
    }
    if (PySequence_Fast_GET_SIZE(seq) != 2) {
        g.fail("next_batch is a pair (indices, kept)");
    } else {
        int64_t kb = 0;
        nb->indices = (const int64_t *)g.dev(PySequence_Fast_GET_ITEM(seq, 0), at::kLong, &nb->L);
        nb->kept = g.dev(PySequence_Fast_GET_ITEM(seq, 1), at::kByte, &kb);
        nb->kept_bytes = (size_t)kb;
    }
    Py_DECREF(seq);
    return g.ok ? nb : nullptr;
}

// shape cores indices offsets n_bags grad_output kept grad_cores alpha cache grad_cache workspace next_batch
TT_FUNCTION(emb_bwd_kept)
{
    Args g(args, nargs, 13);
    if (!g.ok) return nullptr;
    Lookup q(g, true);
    int64_t kb = 0;
    size_t wsb;
    float *grads[3] = {};
    tt_next_batch_t nb{};
    const float *go = g.f32(5);
    const uint8_t *kept = g.u8(6, &kb);
    g.cores(7, grads);
    const float *alpha = g.f32_or_null(8);
    const tt_cache_t *cache = g.cache(9);
    float *gc = g.f32_or_null(10);
    void *ws = g.bytes_or_null(11, &wsb);
    const tt_next_batch_t *next = next_batch(g, 12, &nb);
    if (!g.ok) return nullptr;
    return call([&](void *st) {
        return tt_emb_bwd_kept(q.shape, q.cores, q.indices, q.L, q.offsets, q.n_bags, alpha, cache, go, kept, (size_t)kb, grads, gc, next, ws, wsb, st);
    });
}

// shape cores cores_out indices offsets n_bags grad_output kept lr alpha cache workspace next_batch
TT_FUNCTION(emb_bwd_sgd_kept)
{
    Args g(args, nargs, 13);
    if (!g.ok) return nullptr;
    int64_t L = 0, kb = 0, sizes[3];
    size_t wsb;
    float *cores[3] = {}, *outs[3] = {};
    tt_next_batch_t nb{};
    const tt_shape_t *shape = g.shape(0);
    g.cores(1, cores, nullptr, sizes);
    g.cores(2, outs, sizes);
    const int64_t *indices = g.i64(3, &L);
    const int64_t n_bags = g.integer(5);
    const int64_t *offsets = g.offsets(4, n_bags, true);
    const float *go = g.f32(6);
    const uint8_t *kept = g.u8(7, &kb);
    const float lr = g.real(8);
    const float *alpha = g.f32_or_null(9);
    const tt_cache_t *cache = g.cache(10);
    void *ws = g.bytes_or_null(11, &wsb);
    const tt_next_batch_t *next = next_batch(g, 12, &nb);
    if (!g.ok) return nullptr;
    return call([&](void *st) {
        return tt_emb_bwd_sgd_kept(shape, cores, outs, indices, L, offsets, n_bags, alpha, cache, go, kept, (size_t)kb, lr, next, ws, wsb, st);
    });
}

// shape cores cores_out indices offsets n_bags grad_output lr alpha cache
TT_FUNCTION(emb_bwd_sgd_static)
{
    Args g(args, nargs, 10);
    if (!g.ok) return nullptr;
    int64_t L = 0, sizes[3];
    float *cores[3] = {}, *outs[3] = {};
    const tt_shape_t *shape = g.shape(0);
    g.cores(1, cores, nullptr, sizes);
    g.cores(2, outs, sizes);
    const int64_t *indices = g.i64(3, &L);
    const int64_t n_bags = g.integer(5);
    const int64_t *offsets = g.offsets(4, n_bags);
    const float *go = g.f32(6);
    const float lr = g.real(7);
    const float *alpha = g.f32_or_null(8);
    const tt_cache_t *cache = g.cache(9);
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_emb_bwd_sgd_static(shape, cores, outs, indices, L, offsets, n_bags, alpha, cache, go, lr, st); });
}

// shape cores grad_cores lr cache grad_cache zero_grad
TT_FUNCTION(emb_sgd_update)
{
    Args g(args, nargs, 7);
    if (!g.ok) return nullptr;
    float *cores[3] = {}, *grads[3] = {};
    const tt_shape_t *shape = g.shape(0);
    g.cores(1, cores);
    g.cores(2, grads);
    const float lr = g.real(3);
    const tt_cache_t *cache = g.cache(4);
    float *gc = g.f32_or_null(5);
    const bool zero = g.truth(6);
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_emb_sgd_update(shape, cores, grads, lr, cache, gc, zero ? 1 : 0, st); });
}

// shape cores cand_rows cand_counts cache workspace
template <int (*F)(const tt_shape_t *, const float *const *, const int64_t *, const int64_t *, int64_t, const tt_cache_t *, void *, size_t, void *)>
TT_FUNCTION(cache_fill)
{
    Args g(args, nargs, 6);
    if (!g.ok) return nullptr;
    float *cores[3] = {};
    int64_t n = 0, m = 0;
    size_t wsb;
    const tt_shape_t *shape = g.shape(0);
    g.cores(1, cores);
    const int64_t *rows = g.i64(2, &n), *counts = g.i64(3, &m);
    const tt_cache_t *cache = g.cache(4);
    void *ws = g.bytes_or_null(5, &wsb);
    if (g.ok && n != m) g.fail("as many counts as rows are expected");
    if (!g.ok) return nullptr;
    return call([&](void *st) { return F(shape, cores, rows, counts, n, cache, ws, wsb, st); });
}

// tracker indices
TT_FUNCTION(freq_update)
{
    Args g(args, nargs, 2);
    if (!g.ok) return nullptr;
    int64_t L = 0;
    const tt_freq_t *f = g.freq(0);
    const int64_t *indices = g.i64(1, &L);
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_freq_update(f, indices, L, st); });
}

// tracker rows counts n_out
TT_FUNCTION(freq_export)
{
    Args g(args, nargs, 4);
    if (!g.ok) return nullptr;
    int64_t nr = 0, nc = 0;
    const tt_freq_t *f = g.freq(0);
    int64_t *rows = g.i64(1, &nr), *counts = g.i64(2, &nc), *n_out = g.i64(3);
    if (g.ok && (nr < f->capacity || nc < f->capacity)) g.fail("rows and counts need room for the whole table");
    if (!g.ok) return nullptr;
    return call([&](void *st) { return tt_freq_export(f, rows, counts, n_out, st); });
}

#define TT_METHOD(name, function) {name, (PyCFunction)(void (*)(void))guarded<function>, METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    TT_METHOD("emb_fwd", emb_fwd),
    TT_METHOD("emb_fwd_rows", emb_fwd_rows),
    TT_METHOD("emb_fwd_keep_t0", emb_fwd_keep_t0),
    TT_METHOD("emb_fwd_prepared", emb_fwd_prepared),
    TT_METHOD("emb_bwd", emb_bwd),
    TT_METHOD("emb_bwd_prepare", emb_bwd_prepare),
    TT_METHOD("emb_bwd_sgd", emb_bwd_sgd),
    TT_METHOD("emb_kept_prepare", emb_kept_prepare),
    TT_METHOD("emb_fwd_keep", emb_fwd_keep),
    TT_METHOD("emb_bwd_kept", emb_bwd_kept),
    TT_METHOD("emb_bwd_sgd_kept", emb_bwd_sgd_kept),
    TT_METHOD("emb_bwd_sgd_static", emb_bwd_sgd_static),
    TT_METHOD("emb_sgd_update", emb_sgd_update),
    TT_METHOD("freq_update", freq_update),
    TT_METHOD("freq_export", freq_export),
    TT_METHOD("cache_build", cache_fill<tt_cache_build>),
    TT_METHOD("cache_refill", cache_fill<tt_cache_refill>),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tt_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tt_call(void) { return PyModule_Create(&module); }
