// The per-call side of binding.py in native code: torch tensors in, a descriptor of include/lvlm.h filled, the
// workspace grown where it has to be, the library called on the current stream, the outputs handed back.
//
// What bounds the short calls is the host: a decode step is one lvlm_decode_attn per layer, whose two kernels take some
// 9.5 us, and filling the same descriptors through ctypes took 12 us of Python per call.  Measured, eager calls: one token
// through 48 layers (budget 2048) 631 -> 450 us, one small fp32 layer 19.7 -> 14.0 us, one sequence's scores 22.4 -> 19.7 us;
// what is left of a call on the host is mostly its kernel launches.
//
// The functions of the library are passed in as addresses (setup), so this module works with whichever build of
// liblvlm.so binding.py has loaded.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/lvlm.h"

namespace {

// ---- the library's entry points and binding.py's exception ----
struct Lib {
    decltype(&lvlm_last_error) last_error;
    decltype(&lvlm_workspace_bytes) workspace_bytes;
    decltype(&lvlm_set_workspace) set_workspace;
    decltype(&lvlm_score_tokens) score_tokens;
    decltype(&lvlm_score_from_probs) score_from_probs;
    decltype(&lvlm_prefill_attn) prefill_attn;
    decltype(&lvlm_merge_compact) merge_compact;
    decltype(&lvlm_merge_similar) merge_similar;
    decltype(&lvlm_kv_compress) kv_compress;
    decltype(&lvlm_decode_attn) decode_attn;
    decltype(&lvlm_decode_attn_static) decode_attn_static;
} lib;
PyObject *lvlm_error = nullptr;

struct Core {
    PyObject_HEAD
    lvlm_ctx *h;
    int device;
    PyObject *ws;      // the workspace tensor the context holds, or null
};

// A Python exception is set: unwinds to the entry point.
struct PyErr {};
[[noreturn]] void raise(PyObject *type, const char *msg) {
    PyErr_SetString(type, msg);
    throw PyErr{};
}
void require(bool ok, const char *msg) {
    if (!ok) raise(PyExc_AssertionError, msg);
}

void check(Core *c, lvlm_status st) {
    if (st == LVLM_OK) return;
    PyObject *e = PyObject_CallFunction(lvlm_error, "is", (int)st, lib.last_error(c->h));
    if (e) {
        PyErr_SetObject(lvlm_error, e);
        Py_DECREF(e);
    }
    throw PyErr{};
}

// ---- arguments ----
// Positional-or-keyword names first (n_pos of them), keyword-only names after; `need`: bit per required name.
constexpr int kMaxArgs = 24;
struct Signature {
    const char *fn;
    int n_pos, n;
    unsigned need;
    const char *name[kMaxArgs];
    PyObject *key[kMaxArgs];
    void intern() {
        for (int i = 0; i < n; ++i) key[i] = PyUnicode_InternFromString(name[i]);
    }
    void parse(PyObject *const *args, Py_ssize_t n_args, PyObject *kwnames, PyObject **out) const {
        if (n_args > n_pos) {
            PyErr_Format(PyExc_TypeError, "%s() takes %d positional arguments but %zd were given", fn, n_pos + 1, n_args + 1);
            throw PyErr{};
        }
        for (int i = 0; i < n; ++i) out[i] = i < n_args ? args[i] : nullptr;
        const Py_ssize_t n_kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
        for (Py_ssize_t x = 0; x < n_kw; ++x) {
            PyObject *k = PyTuple_GET_ITEM(kwnames, x);
            int i = 0;
            while (i < n && key[i] != k) ++i;
            if (i == n)
                for (i = 0; i < n && PyUnicode_Compare(key[i], k) != 0; ++i) {}
            if (i == n || out[i]) {
                PyErr_Format(PyExc_TypeError, i == n ? "%s() got an unexpected keyword argument '%U'"
                                                     : "%s() got multiple values for argument '%U'", fn, k);
                throw PyErr{};
            }
            out[i] = args[n_args + x];
        }
        for (int i = 0; i < n; ++i)
            if ((need >> i & 1) && !out[i]) {
                PyErr_Format(PyExc_TypeError, "%s() missing a required argument: '%s'", fn, name[i]);
                throw PyErr{};
            }
    }
};

bool given(PyObject *o) { return o && o != Py_None; }

const at::Tensor &tensor(PyObject *o, const char *what) {
    if (!o || !THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch.Tensor", what);
        throw PyErr{};
    }
    return THPVariable_Unpack(o);
}
// the device pointer of an optional tensor
void *ptr(PyObject *o, const char *what) { return given(o) ? tensor(o, what).data_ptr() : nullptr; }

// an integer field of a descriptor (32 bits are kept, as a C structure's field would)
int32_t integer(PyObject *o, int32_t otherwise) {
    if (!o) return otherwise;
    if (PyFloat_Check(o)) raise(PyExc_TypeError, "int expected instead of float instance");
    const unsigned long v = PyLong_AsUnsignedLongMask(o);
    if (v == (unsigned long)-1 && PyErr_Occurred()) throw PyErr{};
    return (int32_t)v;
}
double real(PyObject *o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PyErr{};
    return v;
}
bool truth(PyObject *o, bool otherwise) {
    if (!o) return otherwise;
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyErr{};
    return v != 0;
}

int32_t dtype_code(const at::Tensor &t) {
    switch (t.scalar_type()) {
        case at::kBFloat16: return LVLM_BF16;
        case at::kFloat: return LVLM_F32;
        case at::kInt: return LVLM_I32;
        default: raise(PyExc_KeyError, c10::toString(t.scalar_type()));
    }
}
void dims(const at::Tensor &t, int n, const char *msg) {
    if (t.dim() != n) raise(PyExc_ValueError, msg);
}

// ---- outputs ----
at::Tensor empty(at::IntArrayRef sizes, const at::Tensor &like, at::ScalarType dt) {
    return at::empty(sizes, at::TensorOptions().dtype(dt).device(like.device()));
}
// An output argument: the caller's tensor (a new reference), or a new one.
struct Out {
    PyObject *o = nullptr;
    ~Out() { Py_XDECREF(o); }
    Out() = default;
    Out(const Out &) = delete;
    Out &operator=(const Out &) = delete;
    bool set(PyObject *arg) {
        if (!given(arg)) return false;
        Py_INCREF(arg);
        o = arg;
        return true;
    }
    void set(at::Tensor &&t) {
        o = THPVariable_Wrap(std::move(t));
        if (!o) throw PyErr{};
    }
    PyObject *take() {
        PyObject *r = o ? o : (Py_INCREF(Py_None), Py_None);
        o = nullptr;
        return r;
    }
};
template <class... O>
PyObject *tuple_of(O &...outs) {
    PyObject *t = PyTuple_New(sizeof...(outs));
    if (!t) throw PyErr{};
    Py_ssize_t i = 0;
    (PyTuple_SET_ITEM(t, i++, outs.take()), ...);
    return t;
}

void *stream() { return static_cast<void *>(c10::hip::getCurrentHIPStream().stream()); }

// ---- workspace ----
void reserve_bytes(Core *c, size_t nbytes) {
    if (c->ws && (size_t)THPVariable_Unpack(c->ws).numel() >= nbytes) return;
    at::Tensor t = at::empty({(int64_t)(nbytes < 256 ? 256 : nbytes)},
                             at::TensorOptions().dtype(at::kByte).device(at::Device(at::kCUDA, (c10::DeviceIndex)c->device)));
    void *p = t.data_ptr();
    const size_t n = (size_t)t.numel();
    PyObject *o = THPVariable_Wrap(std::move(t));
    if (!o) throw PyErr{};
    Py_XSETREF(c->ws, o);
    check(c, lib.set_workspace(c->h, p, n));
}
void reserve_for(Core *c, lvlm_op op, const void *desc) {
    size_t n = 0;
    check(c, lib.workspace_bytes(c->h, op, desc, &n));
    reserve_bytes(c, n);
}

// Runs a launch without the interpreter lock (it can wait for room in the stream's queue).
template <class F>
void launch(Core *c, F f) {
    lvlm_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    check(c, st);
}

// ---- step 1 ----
Signature sig_score{"score_tokens", 2, 11, 0x1fu,
                    {"q", "k", "q_pos0", "img_begin", "n_img", "scale", "causal", "row_lse", "score_head", "score_mean", "reserve"}, {}};
PyObject *score_tokens(Core *c, PyObject *const *a) {
    const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[1], "k");
    dims(q, 4, "q must be [B, T, Hq, d]");
    dims(k, 4, "k must be [B, N, Hkv, d]");
    require(q.stride(3) == 1 && k.stride(3) == 1, "head dimension must be contiguous");
    lvlm_score_desc d{};
    d.dtype = dtype_code(q);
    d.B = (int32_t)q.size(0); d.T = (int32_t)q.size(1); d.Hq = (int32_t)q.size(2); d.hd = (int32_t)q.size(3);
    d.N = (int32_t)k.size(1); d.Hkv = (int32_t)k.size(2);
    d.q_pos0 = integer(a[2], 0);
    d.img_begin = integer(a[3], 0);
    d.n_img = integer(a[4], 0);
    d.scale = (float)(given(a[5]) ? real(a[5]) : 1.0 / std::sqrt((double)d.hd));
    d.causal = truth(a[6], true);
    d.q_stride_b = q.stride(0); d.q_stride_t = q.stride(1); d.q_stride_h = q.stride(2);
    d.k_stride_b = k.stride(0); d.k_stride_n = k.stride(1); d.k_stride_h = k.stride(2);
    Out sh, sm;
    if (sh.set(a[8])) {
        const at::Tensor &t = tensor(a[8], "score_head");
        d.sh_stride_b = t.stride(0);
        d.sh_stride_h = t.stride(1);
    } else {
        sh.set(empty({d.B, d.Hkv, d.n_img}, q, at::kFloat));
    }
    if (!sm.set(a[9])) sm.set(empty({d.B, d.n_img}, q, at::kFloat));
    if (truth(a[10], true)) reserve_for(c, LVLM_OP_SCORE, &d);
    void *s = stream(), *pq = q.data_ptr(), *pk = k.data_ptr();
    float *lse = (float *)ptr(a[7], "row_lse"), *psh = (float *)ptr(sh.o, "score_head"), *psm = (float *)ptr(sm.o, "score_mean");
    launch(c, [&] { return lib.score_tokens(c->h, s, &d, pq, pk, lse, psh, psm); });
    return tuple_of(sh, sm);
}

Signature sig_probs{"score_from_probs", 1, 7, 0xfu,
                    {"probs", "n_kv_heads", "img_begin", "n_img", "score_head", "score_mean", "reserve"}, {}};
PyObject *score_from_probs(Core *c, PyObject *const *a) {
    const at::Tensor &p = tensor(a[0], "probs");
    dims(p, 4, "probs must be [B, Hq, T, N]");
    require(p.stride(3) == 1, "the key axis must be contiguous");
    lvlm_probs_desc d{};
    d.dtype = dtype_code(p);
    d.B = (int32_t)p.size(0); d.Hq = (int32_t)p.size(1); d.T = (int32_t)p.size(2); d.N = (int32_t)p.size(3);
    d.Hkv = integer(a[1], 0);
    d.img_begin = integer(a[2], 0);
    d.n_img = integer(a[3], 0);
    d.p_stride_b = p.stride(0); d.p_stride_h = p.stride(1); d.p_stride_t = p.stride(2);
    Out sh, sm;
    if (sh.set(a[4])) {
        const at::Tensor &t = tensor(a[4], "score_head");
        d.sh_stride_b = t.stride(0);
        d.sh_stride_h = t.stride(1);
    } else {
        sh.set(empty({d.B, d.Hkv, d.n_img}, p, at::kFloat));
    }
    if (!sm.set(a[5])) sm.set(empty({d.B, d.n_img}, p, at::kFloat));
    if (truth(a[6], true)) reserve_for(c, LVLM_OP_SCORE_PROBS, &d);
    void *s = stream(), *pp = p.data_ptr();
    float *psh = (float *)ptr(sh.o, "score_head"), *psm = (float *)ptr(sm.o, "score_mean");
    launch(c, [&] { return lib.score_from_probs(c->h, s, &d, pp, psh, psm); });
    return tuple_of(sh, sm);
}

Signature sig_prefill{"prefill_attn", 3, 13, 0x7u,
                      {"q", "k", "v", "scale", "causal", "n_text", "img_begin", "n_img", "out", "row_lse", "score_head",
                       "score_mean", "reserve"}, {}};
PyObject *prefill_attn(Core *c, PyObject *const *a) {
    const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[1], "k"), &v = tensor(a[2], "v");
    dims(q, 4, "q must be [B, N, Hq, d]");
    lvlm_prefill_desc d{};
    d.B = (int32_t)q.size(0); d.N = (int32_t)q.size(1); d.Hq = (int32_t)q.size(2); d.hd = (int32_t)q.size(3);
    require(k.dim() == 4 && v.dim() == 4 && k.size(0) == d.B && k.size(1) == d.N && k.size(3) == d.hd && v.sizes() == k.sizes(),
            "k and v must be [B, N, Hkv, d]");
    require(q.stride(3) == 1 && k.stride(3) == 1 && v.stride(3) == 1, "head dimension must be contiguous");
    d.dtype = dtype_code(q);
    d.Hkv = (int32_t)k.size(2);
    d.scale = (float)(given(a[3]) ? real(a[3]) : 1.0 / std::sqrt((double)d.hd));
    d.causal = truth(a[4], true);
    d.T = integer(a[5], 0);
    d.img_begin = integer(a[6], 0);
    d.n_img = integer(a[7], 0);
    Out out, lse, sh, sm;
    if (!out.set(a[8])) out.set(empty({d.B, d.N, d.Hq, d.hd}, q, q.scalar_type()));
    if (!lse.set(a[9])) lse.set(empty({d.B, d.Hq, d.N}, q, at::kFloat));
    const at::Tensor &o = tensor(out.o, "out");
    dims(o, 4, "out must be [B, N, Hq, d]");
    require(o.stride(3) == 1 && tensor(lse.o, "row_lse").is_contiguous(), "out needs contiguous head vectors, row_lse must be contiguous");
    if (!sh.set(a[10]) && d.T > 0) sh.set(empty({d.B, d.Hkv, d.n_img}, q, at::kFloat));
    if (!sm.set(a[11]) && d.T > 0) sm.set(empty({d.B, d.n_img}, q, at::kFloat));
    d.q_stride_b = q.stride(0); d.q_stride_n = q.stride(1); d.q_stride_h = q.stride(2);
    d.k_stride_b = k.stride(0); d.k_stride_n = k.stride(1); d.k_stride_h = k.stride(2);
    d.v_stride_b = v.stride(0); d.v_stride_n = v.stride(1); d.v_stride_h = v.stride(2);
    d.o_stride_b = o.stride(0); d.o_stride_n = o.stride(1); d.o_stride_h = o.stride(2);
    if (sh.o && !tensor(sh.o, "score_head").is_contiguous()) {
        d.sh_stride_b = tensor(sh.o, "score_head").stride(0);
        d.sh_stride_h = tensor(sh.o, "score_head").stride(1);
    }
    if (truth(a[12], true)) reserve_for(c, LVLM_OP_PREFILL_ATTN, &d);
    void *s = stream(), *pq = q.data_ptr(), *pk = k.data_ptr(), *pv = v.data_ptr(), *po = o.data_ptr();
    float *pl = (float *)ptr(lse.o, "row_lse"), *psh = (float *)ptr(sh.o, "score_head"), *psm = (float *)ptr(sm.o, "score_mean");
    launch(c, [&] { return lib.prefill_attn(c->h, s, &d, pq, pk, pv, po, pl, psh, psm); });
    return tuple_of(out, lse, sh, sm);
}

// ---- steps 2-4 ----
// The plane table of a merge: planes, their outputs (made where none were passed) and rules.
struct Planes {
    lvlm_plane tab[LVLM_MAX_PLANES + 1] = {};
    int n = 0;
    PyObject *planes = nullptr, *outs = nullptr, *rules = nullptr, *result = nullptr;   // result: what the call returns
    ~Planes() {
        Py_XDECREF(planes);
        Py_XDECREF(outs);
        Py_XDECREF(rules);
        Py_XDECREF(result);
    }
    static PyObject *fast(PyObject *o, const char *msg) {
        PyObject *f = PySequence_Fast(o, msg);
        if (!f) throw PyErr{};
        return f;
    }
    const at::Tensor &first(PyObject *arg) {
        planes = fast(arg, "planes must be a sequence of tensors");
        n = (int)PySequence_Fast_GET_SIZE(planes);
        if (n < 1) raise(PyExc_IndexError, "planes is empty");
        const at::Tensor &t = tensor(PySequence_Fast_GET_ITEM(planes, 0), "planes[0]");
        if (t.dim() < 2) raise(PyExc_IndexError, "a plane is [B, N, row]");
        return t;
    }
    void fill(PyObject *rules_arg, PyObject *outs_arg, int64_t B, int64_t rows) {
        if (given(rules_arg)) rules = fast(rules_arg, "rules must be a sequence");
        if (given(outs_arg)) {
            outs = fast(outs_arg, "outs must be a sequence of tensors");
            Py_INCREF(outs_arg);
            result = outs_arg;
        } else {
            outs = PyList_New(n);
            if (!outs) throw PyErr{};
            for (int i = 0; i < n; ++i) {
                const at::Tensor &p = tensor(PySequence_Fast_GET_ITEM(planes, i), "a plane");
                dims(p, 3, "a plane is [B, N, row]");
                PyObject *o = THPVariable_Wrap(empty({B, rows, p.size(2)}, p, p.scalar_type()));
                if (!o) throw PyErr{};
                PyList_SET_ITEM(outs, i, o);
            }
            Py_INCREF(outs);
            result = outs;
        }
        // (a table with more planes than the library takes is refused there, before it is read)
        for (int i = 0; i < n && i < LVLM_MAX_PLANES + 1; ++i) {
            if (i >= PySequence_Fast_GET_SIZE(outs) || (rules && i >= PySequence_Fast_GET_SIZE(rules))) break;
            const at::Tensor &src = tensor(PySequence_Fast_GET_ITEM(planes, i), "a plane");
            const at::Tensor &dst = tensor(PySequence_Fast_GET_ITEM(outs, i), "an output plane");
            require(src.dim() == 3 && src.stride(2) == 1 && src.stride(1) == src.size(2), "a plane is [B, N, row] with contiguous sequences");
            require(dst.dim() == 3 && dst.stride(2) == 1 && dst.stride(1) == dst.size(2), "an output plane is [B, N - r, row] with contiguous sequences");
            lvlm_plane &p = tab[i];
            p.src = src.data_ptr();
            p.dst = dst.data_ptr();
            p.src_stride_b = src.stride(0);
            p.dst_stride_b = dst.stride(0);
            p.row_elems = (int32_t)src.size(2);
            p.dtype = dtype_code(src);
            p.merge_rule = rules ? integer(PySequence_Fast_GET_ITEM(rules, i), 0) : LVLM_RULE_WEIGHTED;
        }
    }
};
void *ptr_unless_empty(PyObject *o, const char *what) {
    const at::Tensor &t = tensor(o, what);
    return t.numel() ? t.data_ptr() : nullptr;
}

Signature sig_merge{"merge_compact", 2, 11, 0x1fu,
                    {"planes", "score_mean", "img_begin", "n_img", "n_keep", "w", "rules", "outs", "keep_idx", "merged_idx", "reserve"}, {}};
PyObject *merge_compact(Core *c, PyObject *const *a) {
    Planes p;
    const at::Tensor &first = p.first(a[0]);
    lvlm_merge_desc d{};
    d.B = (int32_t)first.size(0); d.N = (int32_t)first.size(1);
    d.img_begin = integer(a[2], 0);
    d.n_img = integer(a[3], 0);
    d.n_keep = integer(a[4], 0);
    d.n_planes = p.n;
    const int64_t r = (int64_t)d.n_img - d.n_keep;
    p.fill(a[6], a[7], d.B, d.N - r);
    Out keep, merged;
    if (!keep.set(a[8])) keep.set(empty({d.B, r > 0 ? (d.n_keep > 1 ? d.n_keep - 1 : 0) : d.n_img}, first, at::kInt));
    if (!merged.set(a[9])) merged.set(empty({d.B, r > 0 ? r + 1 : 0}, first, at::kInt));
    if (truth(a[10], true)) {
        const lvlm_merge_query query{&d, p.tab};
        reserve_for(c, LVLM_OP_MERGE, &query);
    }
    void *s = stream();
    const float *score = (const float *)ptr(a[1], "score_mean"), *w = (const float *)ptr(a[5], "w");
    int32_t *pk = (int32_t *)ptr_unless_empty(keep.o, "keep_idx"), *pm = (int32_t *)ptr_unless_empty(merged.o, "merged_idx");
    launch(c, [&] { return lib.merge_compact(c->h, s, &d, score, w, p.tab, pk, pm); });
    Out outs;
    outs.set(p.result);
    return tuple_of(outs, keep, merged);
}

Signature sig_similar{"merge_similar", 2, 12, 0x1fu,
                      {"planes", "score_mean", "img_begin", "n_img", "n_keep", "size", "rules", "outs", "size_out", "keep_idx",
                       "assign", "reserve"}, {}};
PyObject *merge_similar(Core *c, PyObject *const *a) {
    Planes p;
    const at::Tensor &first = p.first(a[0]);
    lvlm_merge_desc d{};
    d.B = (int32_t)first.size(0); d.N = (int32_t)first.size(1);
    d.img_begin = integer(a[2], 0);
    d.n_img = integer(a[3], 0);
    d.n_keep = integer(a[4], 0);
    d.n_planes = p.n;
    p.fill(a[6], a[7], d.B, d.N - ((int64_t)d.n_img - d.n_keep));
    Out keep, assign, size_out;
    if (!keep.set(a[9])) keep.set(empty({d.B, d.n_keep}, first, at::kInt));
    if (!assign.set(a[10])) assign.set(empty({d.B, d.n_img}, first, at::kInt));
    if (!size_out.set(a[8])) size_out.set(empty({d.B, d.n_keep}, first, at::kFloat));
    if (truth(a[11], true)) {
        const lvlm_merge_query query{&d, p.tab};
        reserve_for(c, LVLM_OP_MERGE_SIMILAR, &query);
    }
    void *s = stream();
    const float *score = (const float *)ptr(a[1], "score_mean"), *size = (const float *)ptr(a[5], "size");
    float *so = (float *)ptr(size_out.o, "size_out");
    int32_t *pk = (int32_t *)ptr(keep.o, "keep_idx"), *pa = (int32_t *)ptr(assign.o, "assign");
    launch(c, [&] { return lib.merge_similar(c->h, s, &d, score, p.tab, size, so, pk, pa); });
    Out outs;
    outs.set(p.result);
    return tuple_of(outs, keep, assign, size_out);
}

// ---- step 5 ----
Signature sig_kv{"kv_compress", 6, 15, 0x7fu,
                 {"k_cache", "v_cache", "score", "kind", "orig_pos", "length", "mode", "order", "beta", "budget", "n_recent",
                  "len_bound", "n_evicted", "reserve", "want_evicted"}, {}};
PyObject *kv_compress(Core *c, PyObject *const *a) {
    const at::Tensor &k = tensor(a[0], "k_cache"), &v = tensor(a[1], "v_cache"), &score = tensor(a[2], "score");
    dims(k, 4, "k_cache must be [B, Hkv, Lmax, d]");
    require(k.is_contiguous() && v.is_contiguous() && score.is_contiguous(), "the caches and scores must be contiguous");
    lvlm_kv_desc d{};
    d.dtype = dtype_code(k);
    d.B = (int32_t)k.size(0); d.Hkv = (int32_t)k.size(1); d.Lmax = (int32_t)k.size(2); d.hd = (int32_t)k.size(3);
    d.mode = integer(a[6], 0);
    d.order = integer(a[7], LVLM_ORDER_STABLE);
    d.beta = a[8] ? real(a[8]) : 0.995;
    d.budget = integer(a[9], 0);
    d.n_recent = integer(a[10], 0);
    d.len_bound = integer(a[11], 0);
    Out ev;
    if (!ev.set(a[12]) && truth(a[14], true)) ev.set(empty({d.B, d.Hkv}, k, at::kInt));
    if (truth(a[13], true)) reserve_for(c, LVLM_OP_KV_COMPRESS, &d);
    void *s = stream(), *pk = k.data_ptr(), *pv = v.data_ptr();
    float *ps = (float *)score.data_ptr();
    uint8_t *kind = (uint8_t *)ptr(a[3], "kind");
    int32_t *pos = (int32_t *)ptr(a[4], "orig_pos"), *len = (int32_t *)ptr(a[5], "length"), *pe = (int32_t *)ptr(ev.o, "n_evicted");
    launch(c, [&] { return lib.kv_compress(c->h, s, &d, pk, pv, ps, kind, pos, len, pe); });
    return ev.take();
}

// ---- step 6 ----
Signature sig_decode{"decode_attn", 9, 19, 0x1ffu,
                     {"q", "k_new", "v_new", "k_cache", "v_cache", "score", "kind", "orig_pos", "length", "scale", "score_decay",
                      "new_kind", "new_pos", "len_bound", "evict_budget", "evict_recent", "out", "reserve", "static_scratch"}, {}};
PyObject *decode_attn(Core *c, PyObject *const *a) {
    const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[3], "k_cache"), &v = tensor(a[4], "v_cache");
    dims(q, 3, "q must be [B, Hq, d]");
    dims(k, 4, "k_cache must be [B, Hkv, Lmax, d]");
    require(q.is_contiguous() && k.is_contiguous() && v.is_contiguous(), "q and the caches must be contiguous");
    lvlm_attn_desc d{};
    d.dtype = dtype_code(q);
    d.B = (int32_t)q.size(0); d.Hq = (int32_t)q.size(1); d.hd = (int32_t)q.size(2);
    d.Hkv = (int32_t)k.size(1); d.Lmax = (int32_t)k.size(2);
    d.scale = (float)(given(a[9]) ? real(a[9]) : 1.0 / std::sqrt((double)d.hd));
    d.score_decay = a[10] ? (float)real(a[10]) : 1.0f;
    d.new_kind = integer(a[11], LVLM_KIND_GENERATED);
    d.new_pos = integer(a[12], 0);
    d.len_bound = integer(a[13], 0);
    d.evict_budget = integer(a[14], 0);
    d.evict_recent = integer(a[15], 0);
    Out out;
    if (!out.set(a[16])) out.set(empty(q.sizes(), q, q.scalar_type()));
    const bool fixed = truth(a[18], false);
    if (truth(a[17], true) && !fixed) reserve_for(c, LVLM_OP_DECODE_ATTN, &d);
    void *s = stream(), *pq = q.data_ptr(), *pk = k.data_ptr(), *pv = v.data_ptr();
    void *kn = ptr(a[1], "k_new"), *vn = ptr(a[2], "v_new"), *po = ptr(out.o, "out");
    float *score = (float *)ptr(a[5], "score");
    uint8_t *kind = (uint8_t *)ptr(a[6], "kind");
    int32_t *pos = (int32_t *)ptr(a[7], "orig_pos"), *len = (int32_t *)ptr(a[8], "length");
    const auto call = fixed ? lib.decode_attn_static : lib.decode_attn;
    launch(c, [&] { return call(c->h, s, &d, pq, kn, vn, pk, pv, score, kind, pos, len, po); });
    return out.take();
}

// ---- the type ----
template <Signature &SIG, PyObject *(*IMPL)(Core *, PyObject *const *)>
PyObject *entry(PyObject *self, PyObject *const *args, Py_ssize_t n_args, PyObject *kwnames) {
    HANDLE_TH_ERRORS
    try {
        PyObject *a[kMaxArgs];
        SIG.parse(args, n_args, kwnames, a);
        return IMPL(reinterpret_cast<Core *>(self), a);
    } catch (const PyErr &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
#define LVLM_METHOD(name, sig, doc) \
    {#name, (PyCFunction)(void (*)(void))entry<sig, name>, METH_FASTCALL | METH_KEYWORDS, doc}

PyObject *attach(PyObject *self, PyObject *args) {
    unsigned long long h;
    int device;
    if (!PyArg_ParseTuple(args, "Ki", &h, &device)) return nullptr;
    reinterpret_cast<Core *>(self)->h = reinterpret_cast<lvlm_ctx *>(h);
    reinterpret_cast<Core *>(self)->device = device;
    Py_RETURN_NONE;
}
PyObject *reserve(PyObject *self, PyObject *n) {
    HANDLE_TH_ERRORS
    try {
        const size_t bytes = PyLong_AsSize_t(n);
        if (bytes == (size_t)-1 && PyErr_Occurred()) return nullptr;
        reserve_bytes(reinterpret_cast<Core *>(self), bytes);
        Py_RETURN_NONE;
    } catch (const PyErr &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
PyObject *get_ws(PyObject *self, void *) {
    PyObject *o = reinterpret_cast<Core *>(self)->ws;
    if (!o) o = Py_None;
    Py_INCREF(o);
    return o;
}
int set_ws(PyObject *self, PyObject *v, void *) {
    if (v == Py_None) v = nullptr;
    if (v && !THPVariable_Check(v)) {
        PyErr_SetString(PyExc_TypeError, "the workspace must be a torch.Tensor or None");
        return -1;
    }
    Py_XINCREF(v);
    Py_XSETREF(reinterpret_cast<Core *>(self)->ws, v);
    return 0;
}
void dealloc(PyObject *self) {
    Py_CLEAR(reinterpret_cast<Core *>(self)->ws);
    Py_TYPE(self)->tp_free(self);
}

PyMethodDef methods[] = {
    LVLM_METHOD(score_tokens, sig_score,
                "score_tokens($self, q, k, *, q_pos0, img_begin, n_img, scale=None, causal=True, row_lse=None, score_head=None, "
                "score_mean=None, reserve=True)\n--\n\n"
                "lvlm_score_tokens.  q [B,T,Hq,d], k [B,N,Hkv,d] -> (score_head [B,Hkv,n_img], score_mean [B,n_img])."),
    LVLM_METHOD(score_from_probs, sig_probs,
                "score_from_probs($self, probs, *, n_kv_heads, img_begin, n_img, score_head=None, score_mean=None, reserve=True)\n--\n\n"
                "lvlm_score_from_probs.  probs [B,Hq,T,N] (softmax rows of the query rows to be summed) ->\n"
                "(score_head [B,Hkv,n_img], score_mean [B,n_img])."),
    LVLM_METHOD(prefill_attn, sig_prefill,
                "prefill_attn($self, q, k, v, *, scale=None, causal=True, n_text=0, img_begin=0, n_img=0, out=None, row_lse=None, "
                "score_head=None, score_mean=None, reserve=True)\n--\n\n"
                "lvlm_prefill_attn.  q [B,N,Hq,d], k, v [B,N,Hkv,d] (any strides with a contiguous head vector) ->\n"
                "(out [B,N,Hq,d], row_lse [B,Hq,N], score_head, score_mean); the scores (of the last n_text rows over\n"
                "the image keys) only when n_text > 0, else None."),
    LVLM_METHOD(merge_compact, sig_merge,
                "merge_compact($self, planes, score_mean, *, img_begin, n_img, n_keep, w=None, rules=None, outs=None, "
                "keep_idx=None, merged_idx=None, reserve=True)\n--\n\n"
                "lvlm_merge_compact.  planes: list of [B,N,row] tensors -> (outs, keep_idx, merged_idx)."),
    LVLM_METHOD(merge_similar, sig_similar,
                "merge_similar($self, planes, score_mean, *, img_begin, n_img, n_keep, size=None, rules=None, outs=None, "
                "size_out=None, keep_idx=None, assign=None, reserve=True)\n--\n\n"
                "lvlm_merge_similar.  planes: list of [B,N,row] tensors -> (outs, keep_idx, assign, size_out)."),
    LVLM_METHOD(kv_compress, sig_kv,
                "kv_compress($self, k_cache, v_cache, score, kind, orig_pos, length, *, mode, order=0, beta=0.995, budget=0, "
                "n_recent=0, len_bound=0, n_evicted=None, reserve=True, want_evicted=True)\n--\n\n"
                "lvlm_kv_compress (in place).  Caches [B,Hkv,Lmax,d]; returns n_evicted [B,Hkv] (None if not wanted)."),
    LVLM_METHOD(decode_attn, sig_decode,
                "decode_attn($self, q, k_new, v_new, k_cache, v_cache, score, kind, orig_pos, length, *, scale=None, "
                "score_decay=1.0, new_kind=2, new_pos=0, len_bound=0, evict_budget=0, evict_recent=0, out=None, reserve=True, "
                "static_scratch=False)\n--\n\n"
                "lvlm_decode_attn.  q [B,Hq,d], k_new/v_new [B,Hkv,d] or None -> out [B,Hq,d].\n"
                "static_scratch: lvlm_decode_attn_static instead (the library's own fixed scratch array, no workspace)."),
    {"reserve", reserve, METH_O, "reserve($self, nbytes, /)\n--\n\nGrows the attached workspace (never shrinks); call outside graph capture."},
    {"_attach", attach, METH_VARARGS, "The lvlm_ctx handle (an address, 0: none) and device the calls go to."},
    {nullptr, nullptr, 0, nullptr}};
PyGetSetDef getset[] = {{"_ws", get_ws, set_ws, "the workspace tensor", nullptr}, {nullptr, nullptr, nullptr, nullptr, nullptr}};

PyTypeObject core_type = {PyVarObject_HEAD_INIT(nullptr, 0) "paper_2509_00419_amd._torch_binding.ContextCalls"};

// setup(error class, address of lvlm_last_error, ... in the order of Lib)
PyObject *setup(PyObject *, PyObject *args) {
    PyObject *err;
    unsigned long long p[11];
    if (!PyArg_ParseTuple(args, "OKKKKKKKKKKK", &err, &p[0], &p[1], &p[2], &p[3], &p[4], &p[5], &p[6], &p[7], &p[8], &p[9], &p[10]))
        return nullptr;
    Py_INCREF(err);
    Py_XSETREF(lvlm_error, err);
    static_assert(sizeof(Lib) == sizeof(p), "one address per entry point");
    memcpy(&lib, p, sizeof(lib));
    Py_RETURN_NONE;
}
PyMethodDef functions[] = {{"setup", setup, METH_VARARGS, "The exception class and the addresses of the library's entry points."},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_binding", "Native calls of binding.Context.", -1, functions,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_binding(void) {
    for (Signature *s : {&sig_score, &sig_probs, &sig_prefill, &sig_merge, &sig_similar, &sig_kv, &sig_decode}) s->intern();
    core_type.tp_basicsize = sizeof(Core);
    core_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE;
    core_type.tp_doc = "The per-call methods of binding.Context.";
    core_type.tp_methods = methods;
    core_type.tp_getset = getset;
    core_type.tp_new = PyType_GenericNew;
    core_type.tp_dealloc = dealloc;
    if (PyType_Ready(&core_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&core_type);
    if (PyModule_AddObject(m, "ContextCalls", reinterpret_cast<PyObject *>(&core_type)) < 0) {
        Py_DECREF(&core_type);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
