// The Python binding's marshalling in native code: torch tensors in and out of the C entry points.
// Small layers are bound by the host: a launch costs 2.7 us in the HIP runtime whatever is launched, and
// shape checks, output allocation, the stream lookup and argument conversion in Python cost another 6
// to 20 us per call (a single-precision reducing layer of 1024 tokens: 63 us of host time for 35 us of
// kernels).  Here a call adds about 1 us to its launches.  Nothing is cached between calls: workspaces come from
// torch's caching allocator on the call's stream and go back to it when the kernels are enqueued, which
// is what dropping a workspace tensor does.
// Host code only; the functions take their arguments by position and are wrapped, with their defaults
// and documentation, by binding.py.
#define __HIP_PLATFORM_AMD__ 1
#include <Python.h>
// (torch's headers need Python.h first)
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cmath>
#include <string>

#include "strd.h"

namespace {

using at::Tensor;
using Args = PyObject *const *;

PyObject *g_error = nullptr;  // binding.StrdError

struct Fail {
    std::string what;
};
[[noreturn]] void fail(std::string what) { throw Fail{std::move(what)}; }

void check(int rc, const char *what) {
    if (rc != STRD_OK) fail(std::string(what) + " failed: " + strd_status_string(rc));
}

// Every function body runs inside this: library errors become StrdError, torch's (out of memory) what
// torch makes of them.
template <PyObject *(*BODY)(Args)>
PyObject *entry(PyObject *, Args a, Py_ssize_t) {
    HANDLE_TH_ERRORS
    try {
        return BODY(a);
    } catch (const Fail &f) {
        PyErr_SetString(g_error, f.what.c_str());
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

const Tensor &tensor(PyObject *o) {
    if (!THPVariable_Check(o)) fail("a torch tensor is needed");
    return THPVariable_Unpack(o);
}
void on_device(const Tensor &t) {
    if (!t.is_cuda()) fail("tensors must live on the GPU");
    if (!t.is_contiguous()) fail("tensors must be contiguous");
}
const Tensor &dev(PyObject *o) {
    const Tensor &t = tensor(o);
    on_device(t);
    return t;
}
// An optional tensor: nullptr for None.
const Tensor *opt(PyObject *o) { return o == Py_None ? nullptr : &dev(o); }
void *ptr(const Tensor *t) { return t ? t->data_ptr() : nullptr; }
float *f32(const Tensor *t) { return static_cast<float *>(ptr(t)); }
const float *f32(const Tensor &t) { return static_cast<const float *>(t.data_ptr()); }

strd_dtype io_of(const Tensor &t) {
    if (t.scalar_type() == at::kFloat) return STRD_F32;
    if (t.scalar_type() == at::kBFloat16) return STRD_BF16;
    fail(std::string("unsupported tensor dtype ") + c10::toString(t.scalar_type()) + " (fp32 or bf16)");
}
bool is_f32(const Tensor &t) { return t.scalar_type() == at::kFloat; }

// Values that the library takes as int: one that does not fit is refused, not cut.
int narrow(long long v, const char *what) {
    if (v < INT_MIN || v > INT_MAX) fail(std::string(what) + " does not fit 32 bits: " + std::to_string(v));
    return (int)v;
}
int whole(PyObject *v, const char *what) {  // takes over v
    if (!v) throw python_error();
    int over = 0;
    const long long n = PyLong_AsLongLongAndOverflow(v, &over);
    Py_DECREF(v);
    if (over) fail(std::string(what) + " does not fit 32 bits");
    return narrow(n, what);
}
int integer(PyObject *o, const char *what = "a number") { return whole(PyNumber_Index(o), what); }
// Fields of a sequence descriptor: whatever Python's int() takes.
int integer_of(PyObject *o, const char *what) { return whole(PyNumber_Long(o), what); }
int size(const Tensor &t, int dim) { return narrow(t.size(dim), "a tensor's size"); }
bool truth(PyObject *o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw python_error();
    return v;
}
double number(PyObject *o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw python_error();
    return v;
}
float scale_or_default(PyObject *o, int64_t d) { return (float)(o == Py_None ? std::pow((double)d, -0.5) : number(o)); }

Tensor empty(at::IntArrayRef sizes, at::ScalarType type, const Tensor &like) {
    return Tensor(at::detail::empty_cuda(sizes, type, like.device(), std::nullopt));
}
Tensor out_or(PyObject *o, at::IntArrayRef sizes, at::ScalarType type, const Tensor &like) {
    return o == Py_None ? empty(sizes, type, like) : dev(o);
}
hipStream_t stream() { return c10::hip::getCurrentHIPStream().stream(); }
PyObject *wrap(Tensor t) { return THPVariable_Wrap(std::move(t)); }
PyObject *none() { Py_RETURN_NONE; }
PyObject *pair(PyObject *a, PyObject *b) {
    PyObject *t = PyTuple_New(2);
    PyTuple_SET_ITEM(t, 0, a);
    PyTuple_SET_ITEM(t, 1, b);
    return t;
}

// A workspace for one call: the caller's tensor, or a block of torch's allocator that goes back to its
// stream's pool when this goes out of scope, after the kernels have been enqueued.
struct Workspace {
    void *p = nullptr;
    size_t bytes = 0;
    bool mine = false;
    Tensor held;
    Workspace(PyObject *given, size_t need, const Tensor &like, hipStream_t st) {
        if (given != Py_None) {
            const Tensor &t = dev(given);
            p = t.data_ptr();
            bytes = t.numel();
        } else if (need) {
            bytes = need;
            if (like.device().index() == c10::hip::current_device()) {
                p = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(need, st);
                mine = true;
            } else {
                held = empty({(int64_t)need}, at::kByte, like);
                p = held.data_ptr();
            }
        }
    }
    ~Workspace() {
        if (mine) c10::hip::HIPCachingAllocator::raw_delete(p);
    }
    Workspace(const Workspace &) = delete;
};

// The C entry points run without the interpreter lock, as they do through ctypes.
struct NoLock {
    PyThreadState *s = PyEval_SaveThread();
    ~NoLock() { PyEval_RestoreThread(s); }
};
template <typename F>
int call(F &&f) {
    NoLock unlocked;
    return f();
}

// ------------------------------------------------------------------ scores -----------------
PyObject *score_attn(Args a) {  // q_txt, k_vis, scale, out, ws
    const Tensor &q = dev(a[0]), &k = dev(a[1]);
    if (q.dim() != 3 || k.dim() != 3 || q.size(2) != k.size(2) || q.scalar_type() != k.scalar_type()) fail("q/k mismatch");
    const strd_dtype io = io_of(q);
    const int M = size(q, 0), Hq = size(q, 1), d = size(q, 2), N = size(k, 0), Hkv = size(k, 1);
    const float scale = scale_or_default(a[2], d);
    Tensor s = out_or(a[3], {N}, at::kFloat, q);
    const hipStream_t st = stream();
    Workspace ws(a[4], a[4] == Py_None ? strd_score_attn_workspace(M, N, Hq, Hkv, d, io) : 0, q, st);
    check(call([&] {
              return strd_score_attn(q.data_ptr(), k.data_ptr(), f32(&s), M, N, Hq, Hkv, d, scale, io, ws.p, ws.bytes, st);
          }),
          "score_attn");
    return wrap(std::move(s));
}

PyObject *score_mamba(Args a) {  // B_vis, C_txt, dt_vis, out, ws
    const Tensor &B = dev(a[0]), &C = dev(a[1]), &dt = dev(a[2]);
    if (B.dim() != 3 || C.dim() != 3 || dt.dim() != 2 || C.size(1) != B.size(1) || C.size(2) != B.size(2) ||
        dt.size(0) != B.size(0) || !is_f32(dt) || B.scalar_type() != C.scalar_type())
        fail("B/C/dt mismatch");
    const strd_dtype io = io_of(B);
    const int N = size(B, 0), G = size(B, 1), n = size(B, 2), M = size(C, 0), H = size(dt, 1);
    Tensor s = out_or(a[3], {N}, at::kFloat, B);
    const hipStream_t st = stream();
    Workspace ws(a[4], a[4] == Py_None ? strd_score_mamba_workspace(M, N, H, G, n, io) : 0, B, st);
    check(call([&] {
              return strd_score_mamba(B.data_ptr(), C.data_ptr(), f32(dt), f32(&s), M, N, H, G, n, io, ws.p, ws.bytes, st);
          }),
          "score_mamba");
    return wrap(std::move(s));
}

// ------------------------------------------------------------------ selection, compaction --
PyObject *select_topk(Args a) {  // scores, K, out, ws
    const Tensor &s = dev(a[0]);
    if (!is_f32(s) || s.dim() != 1) fail("scores must be a 1-D fp32 tensor");
    const int N = size(s, 0), K = integer(a[1]);
    if (a[2] == Py_None && K < 0) fail("select_topk failed: K is negative");
    Tensor idx = out_or(a[2], {K}, at::kInt, s);
    const hipStream_t st = stream();
    Workspace ws(a[3], a[3] == Py_None ? strd_select_topk_workspace(N, K) : 0, s, st);
    check(call([&] { return strd_select_topk(f32(s), N, K, (int32_t *)idx.data_ptr(), ws.p, ws.bytes, st); }), "select_topk");
    return wrap(std::move(idx));
}

// Sizes of `t`, of any number of dimensions, with `rows` in place of the first one.
struct Sizes {
    at::DimVector v;
    Sizes(int64_t rows, const Tensor &t) : v(t.sizes().begin(), t.sizes().end()) {
        if (v.empty()) fail("a tensor with rows is needed");
        v[0] = rows;
    }
    operator at::IntArrayRef() const { return v; }
    int64_t row() const {
        int64_t r = 1;
        for (size_t i = 1; i < v.size(); ++i) r *= v[i];
        return r;
    }
};
const int32_t *i32(const Tensor *t) { return t ? (const int32_t *)t->data_ptr() : nullptr; }

struct Sequence {
    PyObject *fast;
    explicit Sequence(PyObject *o) : fast(PySequence_Fast(o, "a sequence is needed")) {
        if (!fast) throw python_error();
    }
    ~Sequence() { Py_DECREF(fast); }
    Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(fast); }
    PyObject *operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(fast, i); }
    Sequence(const Sequence &) = delete;
};

PyObject *compact_batch(Args a) {  // srcs, idx, N, M, pos_in, want_pos, outs
    Sequence srcs(a[0]);
    const Tensor &idx = dev(a[1]);
    const int N = integer(a[2]), M = integer(a[3]);
    const Tensor *pos_in = opt(a[4]);
    if (idx.scalar_type() != at::kInt || idx.dim() < 1) fail("idx must be int32");
    const int K = size(idx, 0), n = (int)srcs.size();
    if (n > STRD_COMPACT_MAX) fail("compact_batch failed: " + std::string(strd_status_string(STRD_EINVAL)));
    strd_compact_item items[STRD_COMPACT_MAX];
    Tensor dst[STRD_COMPACT_MAX];
    if (a[6] != Py_None) {
        Sequence outs(a[6]);
        if (outs.size() < n) fail("compact_batch: one output per tensor");
        for (int i = 0; i < n; ++i) dst[i] = dev(outs[i]);
    }
    for (int i = 0; i < n; ++i) {
        const Tensor &t = dev(srcs[i]);
        const Sizes sz((int64_t)K + M, t);
        if (a[6] == Py_None) dst[i] = empty(sz, t.scalar_type(), t);
        if (t.size(0) != (int64_t)N + M || dst[i].scalar_type() != t.scalar_type() || dst[i].sizes() != at::IntArrayRef(sz))
            fail("compact_batch: tensor " + std::to_string(i) + " has the wrong shape");
        items[i] = {t.data_ptr(), dst[i].data_ptr(), sz.row() * (int64_t)t.element_size()};
    }
    Tensor pos;
    if (truth(a[5]) || pos_in) pos = empty({(int64_t)K + M}, at::kInt, idx);
    const hipStream_t st = stream();
    check(call([&] {
              return strd_compact_batch(items, n, i32(&idx), N, M, K, i32(pos_in),
                                        pos.defined() ? (int32_t *)pos.data_ptr() : nullptr, st);
          }),
          "compact_batch");
    PyObject *list = a[6] == Py_None ? PyList_New(n) : PySequence_List(a[6]);  // the caller's outputs, all of them
    if (!list) throw python_error();
    if (a[6] == Py_None)
        for (int i = 0; i < n; ++i) PyList_SET_ITEM(list, i, wrap(std::move(dst[i])));
    return pair(list, pos.defined() ? wrap(std::move(pos)) : none());
}

// ------------------------------------------------------------------ packed batches ---------
struct Seqs {
    strd_seq s[STRD_VARLEN_MAX];
    int n;
    int64_t rows = 0, kept = 0, out_rows = 0;
    int max_n = 0;
    explicit Seqs(PyObject *o) {
        Sequence list(o);
        n = (int)list.size();
        if (n > STRD_VARLEN_MAX) fail(std::string("too many sequences: ") + strd_status_string(STRD_EINVAL));
        for (int i = 0; i < n; ++i) {
            Sequence t(list[i]);
            if (t.size() != 3) fail("a sequence is described by (N, M, K)");
            s[i].N = integer_of(t[0], "N");
            s[i].M = integer_of(t[1], "M");
            s[i].K = integer_of(t[2], "K");
            rows += (int64_t)s[i].N + s[i].M;
            kept += s[i].K;
            out_rows += (int64_t)s[i].K + s[i].M;
            max_n = std::max(max_n, s[i].N);
        }
    }
    int ld(PyObject *o) const { return o == Py_None ? narrow(((int64_t)max_n + 3) / 4 * 4, "ld") : integer_of(o, "ld"); }
};

PyObject *score_attn_varlen(Args a) {  // q_all, k_all, seqs, scale, ld, out
    const Tensor &q = dev(a[0]), &k = dev(a[1]);
    const Seqs sq(a[2]);
    if (q.dim() != 3 || k.dim() != 3 || k.size(0) != q.size(0) || k.size(2) != q.size(2) ||
        q.scalar_type() != k.scalar_type() || q.size(0) != sq.rows)
        fail("score_attn_varlen: q/k/seqs mismatch");
    const strd_dtype io = io_of(q);
    const int Hq = size(q, 1), d = size(q, 2), Hkv = size(k, 1), ld = sq.ld(a[4]);
    const float scale = scale_or_default(a[3], d);
    const bool mine = a[5] == Py_None;  // a matrix made here has zeros behind the scores
    Tensor s = out_or(a[5], {sq.n, ld}, at::kFloat, q);
    const hipStream_t st = stream();
    Workspace ws(Py_None, strd_score_attn_varlen_workspace(sq.s, sq.n, Hq, Hkv, d, io), q, st);
    check(call([&] {
              return (mine ? strd_score_attn_varlen_padded : strd_score_attn_varlen)(q.data_ptr(), k.data_ptr(), f32(&s), ld, sq.s, sq.n, Hq, Hkv, d, scale, io, ws.p,
                                            ws.bytes, st);
          }),
          "score_attn_varlen");
    return wrap(std::move(s));
}

PyObject *score_mamba_varlen(Args a) {  // B_all, C_all, dt_all, seqs, ld, out
    const Tensor &B = dev(a[0]), &C = dev(a[1]), &dt = dev(a[2]);
    const Seqs sq(a[3]);
    if (B.dim() != 3 || dt.dim() != 2 || C.sizes() != B.sizes() || dt.size(0) != B.size(0) || !is_f32(dt) ||
        B.scalar_type() != C.scalar_type() || B.size(0) != sq.rows)
        fail("score_mamba_varlen: B/C/dt/seqs mismatch");
    const strd_dtype io = io_of(B);
    const int G = size(B, 1), n = size(B, 2), H = size(dt, 1), ld = sq.ld(a[4]);
    const bool mine = a[5] == Py_None;
    Tensor s = out_or(a[5], {sq.n, ld}, at::kFloat, B);
    const hipStream_t st = stream();
    Workspace ws(Py_None, strd_score_mamba_varlen_workspace(sq.s, sq.n, H, G, n, io), B, st);
    check(call([&] {
              return (mine ? strd_score_mamba_varlen_padded : strd_score_mamba_varlen)(B.data_ptr(), C.data_ptr(), f32(dt), f32(&s), ld, sq.s, sq.n, H, G, n, io, ws.p,
                                             ws.bytes, st);
          }),
          "score_mamba_varlen");
    return wrap(std::move(s));
}

PyObject *select_topk_varlen(Args a) {  // scores, seqs, out
    const Tensor &s = dev(a[0]);
    const Seqs sq(a[1]);
    if (!is_f32(s) || s.dim() != 2 || s.size(0) != sq.n) fail("select_topk_varlen: scores must be fp32 [nseq, ld]");
    Tensor idx = out_or(a[2], {sq.kept}, at::kInt, s);
    const int ld = size(s, 1);
    const hipStream_t st = stream();
    check(call([&] { return strd_select_topk_varlen(f32(s), ld, sq.s, sq.n, (int32_t *)idx.data_ptr(), st); }),
          "select_topk_varlen");
    return wrap(std::move(idx));
}

PyObject *compact_varlen(Args a) {  // srcs, idx, seqs, pos_in, want_pos
    Sequence srcs(a[0]);
    const Tensor &idx = dev(a[1]);
    const Seqs sq(a[2]);
    const Tensor *pos_in = opt(a[3]);
    if (idx.scalar_type() != at::kInt || idx.dim() < 1 || idx.size(0) != sq.kept)
        fail("compact_varlen: idx must be int32 [sum K]");
    const int n = (int)srcs.size();
    if (n > STRD_COMPACT_MAX) fail("compact_varlen failed: " + std::string(strd_status_string(STRD_EINVAL)));
    strd_compact_item items[STRD_COMPACT_MAX];
    Tensor dst[STRD_COMPACT_MAX];
    for (int i = 0; i < n; ++i) {
        const Tensor &t = dev(srcs[i]);
        const Sizes sz(sq.out_rows, t);
        if (t.size(0) != sq.rows) fail("compact_varlen: tensor " + std::to_string(i) + " has the wrong number of rows");
        dst[i] = empty(sz, t.scalar_type(), t);
        items[i] = {t.data_ptr(), dst[i].data_ptr(), sz.row() * (int64_t)t.element_size()};
    }
    Tensor pos;
    if (truth(a[4]) || pos_in) pos = empty({sq.out_rows}, at::kInt, idx);
    const hipStream_t st = stream();
    check(call([&] {
              return strd_compact_varlen(items, n, i32(&idx), sq.s, sq.n, i32(pos_in),
                                         pos.defined() ? (int32_t *)pos.data_ptr() : nullptr, st);
          }),
          "compact_varlen");
    PyObject *list = PyList_New(n);
    for (int i = 0; i < n; ++i) PyList_SET_ITEM(list, i, wrap(std::move(dst[i])));
    return pair(list, pos.defined() ? wrap(std::move(pos)) : none());
}

// ------------------------------------------------------------------ mixers -----------------
struct Scan {
    const Tensor &x, &dt, &A, &B, &C;
    int rows, H, P, G, n;
    strd_dtype io;
    Scan(Args a, const char *what) : x(dev(a[0])), dt(dev(a[1])), A(dev(a[2])), B(dev(a[3])), C(dev(a[4])) {
        bool ok = x.dim() == 3 && B.dim() == 3 && dt.dim() == 2 && A.dim() == 1;
        if (ok) {
            rows = size(x, 0), H = size(x, 1), P = size(x, 2), G = size(B, 1), n = size(B, 2);
            ok = dt.size(0) == rows && dt.size(1) == H && A.size(0) == H && B.size(0) == rows && C.sizes() == B.sizes() &&
                 is_f32(dt) && is_f32(A) && B.scalar_type() == x.scalar_type() && C.scalar_type() == x.scalar_type();
        }
        if (!ok) fail(std::string(what) + ": inconsistent shapes or dtypes");
        io = io_of(x);
    }
    void optional(const Tensor *D, const Tensor *S, const char *what) const {
        if (D && (D->dim() != 1 || D->size(0) != H || !is_f32(*D)))
            fail(std::string(what) + ": D must be fp32 [H]");
        if (S && (S->dim() != 3 || S->size(0) != H || S->size(1) != P || S->size(2) != n || !is_f32(*S)))
            fail(std::string(what) + ": S_in must be fp32 [H, P, n]");
    }
};

PyObject *ssd_prefill(Args a) {  // x, dt, A, B, C, D, S_in, chunk, want_state, out, ws
    const Scan t(a, "ssd_prefill");
    const Tensor *D = opt(a[5]), *S_in = opt(a[6]);
    t.optional(D, S_in, "ssd_prefill");
    const int chunk = integer(a[7]), T = t.rows;
    Tensor y = out_or(a[9], t.x.sizes(), t.x.scalar_type(), t.x), S;
    if (truth(a[8])) S = empty({t.H, t.P, t.n}, at::kFloat, t.x);
    const hipStream_t st = stream();
    Workspace ws(a[10], a[10] == Py_None ? strd_ssd_prefill_workspace(T, t.H, t.P, t.G, t.n, chunk, t.io) : 0, t.x, st);
    check(call([&] {
              return strd_ssd_prefill(t.x.data_ptr(), f32(t.dt), f32(t.A), t.B.data_ptr(), t.C.data_ptr(), f32(D), f32(S_in),
                                      y.data_ptr(), S.defined() ? f32(&S) : nullptr, T, t.H, t.P, t.G, t.n, chunk, t.io, ws.p,
                                      ws.bytes, st);
          }),
          "ssd_prefill");
    return pair(wrap(std::move(y)), S.defined() ? wrap(std::move(S)) : none());
}

PyObject *ssd_prefill_gather(Args a) {  // x, dt, A, B, C, idx, N, M, D, S_in, chunk, want_state, out, ws
    const Scan t(a, "ssd_prefill_gather");
    const Tensor &idx = dev(a[5]);
    const int N = integer(a[6]), M = integer(a[7]), chunk = integer(a[10]);
    const Tensor *D = opt(a[8]), *S_in = opt(a[9]);
    if (t.rows != (int64_t)N + M || idx.scalar_type() != at::kInt || idx.dim() < 1)
        fail("ssd_prefill_gather: inconsistent shapes or dtypes");
    const int K = size(idx, 0);
    Tensor y = out_or(a[12], {(int64_t)K + M, t.H, t.P}, t.x.scalar_type(), t.x), S;
    if (truth(a[11])) S = empty({t.H, t.P, t.n}, at::kFloat, t.x);
    const hipStream_t st = stream();
    Workspace ws(a[13], a[13] == Py_None ? strd_ssd_prefill_workspace(narrow((int64_t)K + M, "K + M"), t.H, t.P, t.G, t.n, chunk, t.io) : 0, t.x, st);
    check(call([&] {
              return strd_ssd_prefill_gather(t.x.data_ptr(), f32(t.dt), f32(t.A), t.B.data_ptr(), t.C.data_ptr(), f32(D),
                                             f32(S_in), i32(&idx), y.data_ptr(), S.defined() ? f32(&S) : nullptr, N, M, K,
                                             t.H, t.P, t.G, t.n, chunk, t.io, ws.p, ws.bytes, st);
          }),
          "ssd_prefill_gather");
    return pair(wrap(std::move(y)), S.defined() ? wrap(std::move(S)) : none());
}

PyObject *attn_prefill(Args a) {  // q, k, v, scale, out, ws
    const Tensor &q = dev(a[0]), &k = dev(a[1]), &v = dev(a[2]);
    if (q.dim() != 3 || k.dim() != 3 || k.size(0) != q.size(0) || k.size(2) != q.size(2) || v.sizes() != k.sizes() ||
        k.scalar_type() != q.scalar_type() || v.scalar_type() != q.scalar_type())
        fail("attn_prefill: inconsistent shapes or dtypes");
    const strd_dtype io = io_of(q);
    const int T = size(q, 0), Hq = size(q, 1), d = size(q, 2), Hkv = size(k, 1);
    const float scale = scale_or_default(a[3], d);
    Tensor o = out_or(a[4], q.sizes(), q.scalar_type(), q);
    const hipStream_t st = stream();
    Workspace ws(a[5], a[5] == Py_None ? strd_attn_prefill_workspace(T, Hq, Hkv, d, io) : 0, q, st);
    check(call([&] {
              return strd_attn_prefill(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), T, Hq, Hkv, d, scale, io, ws.p,
                                       ws.bytes, st);
          }),
          "attn_prefill");
    return wrap(std::move(o));
}

PyObject *ssd_decode_step(Args a) {  // x, dt, A, B, C, D, S
    const Tensor &x = dev(a[0]), &dt = dev(a[1]), &A = dev(a[2]), &B = dev(a[3]), &C = dev(a[4]), &S = dev(a[6]);
    const Tensor *D = opt(a[5]);
    bool ok = x.dim() == 2 && B.dim() == 2 && dt.dim() == 1 && A.dim() == 1 && S.dim() == 3;
    if (ok) {
        const int64_t H = x.size(0);
        ok = dt.size(0) == H && A.size(0) == H && C.sizes() == B.sizes() && S.size(0) == H && S.size(1) == x.size(1) &&
             S.size(2) == B.size(1) && is_f32(S) && is_f32(dt) && is_f32(A) && B.scalar_type() == x.scalar_type() &&
             C.scalar_type() == x.scalar_type() && (!D || (D->dim() == 1 && D->size(0) == H && is_f32(*D)));
    }
    if (!ok) fail("ssd_decode_step: inconsistent shapes or dtypes");
    const strd_dtype io = io_of(x);
    const int H = size(x, 0), P = size(x, 1), G = size(B, 0), n = size(B, 1);
    Tensor y = empty(x.sizes(), x.scalar_type(), x);
    const hipStream_t st = stream();
    check(call([&] {
              return strd_ssd_decode_step(x.data_ptr(), f32(dt), f32(A), B.data_ptr(), C.data_ptr(), f32(D), f32(&S),
                                          y.data_ptr(), H, P, G, n, io, st);
          }),
          "ssd_decode_step");
    return wrap(std::move(y));
}

PyObject *attn_decode_step(Args a) {  // q, k_cache, v_cache, scale, ws
    const Tensor &q = dev(a[0]), &k = dev(a[1]), &v = dev(a[2]);
    if (q.dim() != 2 || k.dim() != 3 || k.size(2) != q.size(1) || v.sizes() != k.sizes() ||
        k.scalar_type() != q.scalar_type() || v.scalar_type() != q.scalar_type())
        fail("attn_decode_step: inconsistent shapes or dtypes");
    const strd_dtype io = io_of(q);
    const int Hq = size(q, 0), d = size(q, 1), T = size(k, 0), Hkv = size(k, 1);
    const float scale = scale_or_default(a[3], d);
    Tensor o = empty(q.sizes(), q.scalar_type(), q);
    const hipStream_t st = stream();
    Workspace ws(a[4], a[4] == Py_None ? strd_attn_decode_step_workspace(T, Hq, Hkv, d, io) : 0, q, st);
    check(call([&] {
              return strd_attn_decode_step(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), T, Hq, Hkv, d, scale, io,
                                           ws.p, ws.bytes, st);
          }),
          "attn_decode_step");
    return wrap(std::move(o));
}

// ------------------------------------------------------------------ block glue -------------
// Row pitch in elements of a 2-D GPU tensor whose rows are contiguous (a column slice is fine).
int pitch(const Tensor &t, const char *what) {
    if (!t.is_cuda()) fail("tensors must live on the GPU");
    if (t.dim() != 2 || t.stride(1) != 1) fail(std::string(what) + ": rows must be contiguous");
    return narrow(t.stride(0), "a row pitch");
}

PyObject *linear(Args a) {  // x, w, residual, out
    const Tensor &x = dev(a[0]), &w = dev(a[1]);
    const Tensor *res = opt(a[2]);
    if (x.dim() != 2 || w.dim() != 2 || w.size(0) != x.size(1) || w.scalar_type() != x.scalar_type() ||
        (res && (res->dim() != 2 || res->size(0) != x.size(0) || res->size(1) != w.size(1) ||
                 res->scalar_type() != x.scalar_type())))
        fail("linear: x [T,Kd], w [Kd,Nd], residual [T,Nd], one dtype");
    const strd_dtype io = io_of(x);
    const int T = size(x, 0), Kd = size(x, 1), Nd = size(w, 1);
    Tensor out = out_or(a[3], {T, Nd}, x.scalar_type(), x);
    const hipStream_t st = stream();
    check(call([&] { return strd_linear(x.data_ptr(), w.data_ptr(), ptr(res), out.data_ptr(), T, Kd, Nd, io, st); }), "linear");
    return wrap(std::move(out));
}

PyObject *rmsnorm(Args a) {  // x, w, eps, out
    const Tensor &x = dev(a[0]), &w = dev(a[1]);
    if (x.dim() != 2 || w.dim() != 1 || w.size(0) != x.size(1) || w.scalar_type() != x.scalar_type())
        fail("rmsnorm: x [T,d] contiguous, w [d] of the same dtype");
    const strd_dtype io = io_of(x);
    const int T = size(x, 0), d = size(x, 1);
    const float eps = (float)number(a[2]);
    Tensor out = out_or(a[3], x.sizes(), x.scalar_type(), x);
    const hipStream_t st = stream();
    check(call([&] { return strd_rmsnorm(x.data_ptr(), w.data_ptr(), out.data_ptr(), T, d, eps, io, st); }), "rmsnorm");
    return wrap(std::move(out));
}

PyObject *gated_rmsnorm(Args a) {  // y, z, w, groups, eps, out
    const Tensor &y = dev(a[0]), &z = tensor(a[1]), &w = dev(a[2]);
    if (y.dim() != 2 || z.sizes() != y.sizes() || w.dim() != 1 || w.size(0) != y.size(1) ||
        z.scalar_type() != y.scalar_type() || w.scalar_type() != y.scalar_type())
        fail("gated_rmsnorm: y, z [T,D], w [D], one dtype");
    const strd_dtype io = io_of(y);
    const int T = size(y, 0), D = size(y, 1), groups = integer(a[3]), ldz = pitch(z, "z");
    const float eps = (float)number(a[4]);
    Tensor out = out_or(a[5], y.sizes(), y.scalar_type(), y);
    const hipStream_t st = stream();
    check(call([&] {
              return strd_gated_rmsnorm(y.data_ptr(), z.data_ptr(), ldz, w.data_ptr(), out.data_ptr(), T, D, groups, eps, io, st);
          }),
          "gated_rmsnorm");
    return wrap(std::move(out));
}

PyObject *conv1d_silu(Args a) {  // xbc, w, b, Cx, Cb
    const Tensor &in = tensor(a[0]), &w = dev(a[1]);
    const Tensor *b = opt(a[2]);
    const int Cx = integer(a[3]), Cb = integer(a[4]), Ct = narrow((int64_t)Cx + 2 * (int64_t)Cb, "Cx + 2 Cb");
    if (in.dim() != 2 || in.size(1) < Ct || w.dim() != 2 || w.size(0) != Ct || w.scalar_type() != in.scalar_type() ||
        (b && (b->dim() != 1 || b->size(0) != Ct || b->scalar_type() != in.scalar_type())))
        fail("conv1d_silu: xbc [T, >=Cx+2Cb], w [Cx+2Cb, W], b [Cx+2Cb], one dtype");
    const strd_dtype io = io_of(in);
    const int T = size(in, 0), W = size(w, 1), ld = pitch(in, "xbc");
    Tensor x = empty({T, Cx}, in.scalar_type(), in), B = empty({T, Cb}, in.scalar_type(), in),
           C = empty({T, Cb}, in.scalar_type(), in);
    const hipStream_t st = stream();
    check(call([&] {
              return strd_conv1d_silu(in.data_ptr(), ld, w.data_ptr(), ptr(b), x.data_ptr(), B.data_ptr(), C.data_ptr(), T, Cx,
                                      Cb, W, io, st);
          }),
          "conv1d_silu");
    PyObject *t = PyTuple_New(3);
    PyTuple_SET_ITEM(t, 0, wrap(std::move(x)));
    PyTuple_SET_ITEM(t, 1, wrap(std::move(B)));
    PyTuple_SET_ITEM(t, 2, wrap(std::move(C)));
    return t;
}

PyObject *softplus_dt(Args a) {  // raw, bias
    const Tensor &raw = tensor(a[0]);
    const Tensor *bias = opt(a[1]);
    if (raw.dim() != 2) fail("softplus_dt: raw [T,H]");
    const int T = size(raw, 0), H = size(raw, 1);
    if (bias && (bias->dim() != 1 || bias->size(0) != H || !is_f32(*bias))) fail("softplus_dt: bias [H] fp32");
    const strd_dtype io = io_of(raw);
    const int ld = pitch(raw, "raw");
    Tensor dt = empty({T, H}, at::kFloat, raw);
    const hipStream_t st = stream();
    check(call([&] { return strd_softplus_dt(raw.data_ptr(), ld, 0, f32(bias), f32(&dt), T, H, io, st); }), "softplus_dt");
    return wrap(std::move(dt));
}

PyObject *set_error(PyObject *, PyObject *cls) {
    Py_XINCREF(cls);
    Py_XSETREF(g_error, cls);
    Py_RETURN_NONE;
}

#define STRD_ENTRY(name) {#name, (PyCFunction)(void (*)(void))&entry<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"set_error", set_error, METH_O, nullptr},
    STRD_ENTRY(score_attn), STRD_ENTRY(score_mamba), STRD_ENTRY(select_topk), STRD_ENTRY(compact_batch),
    STRD_ENTRY(score_attn_varlen), STRD_ENTRY(score_mamba_varlen), STRD_ENTRY(select_topk_varlen), STRD_ENTRY(compact_varlen),
    STRD_ENTRY(ssd_prefill), STRD_ENTRY(ssd_prefill_gather), STRD_ENTRY(attn_prefill), STRD_ENTRY(ssd_decode_step),
    STRD_ENTRY(attn_decode_step), STRD_ENTRY(linear), STRD_ENTRY(rmsnorm), STRD_ENTRY(gated_rmsnorm), STRD_ENTRY(conv1d_silu),
    STRD_ENTRY(softplus_dt), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "strd_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_strd_host() { return PyModule_Create(&module); }
