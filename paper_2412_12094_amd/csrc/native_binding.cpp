// The binding's host path in native code: what happens between a Python call and the C entry point.
//
// The functions of binding.py that enqueue work take torch tensors and pass device pointers, sizes
// and the current stream to libsepattn.  At the small end of the range (one conversation, one decode
// step) the kernels last a few microseconds, so what a call costs on the host decides how fast a
// generation loop runs: in Python (ctypes argument objects, current_stream(), torch.empty) it was
// about 5.5 us per call on top of the kernel launches, here it is well under 1 us.  Nothing is
// computed here: checks on the tensors, allocation of outputs and workspaces that the caller did not
// pass (through torch's allocator), one call into the library.
//
// The module does not link libsepattn: bind(path) opens the library the binding uses and looks the
// entry points up, so that SEPATTN_LIB selects another build for this path as well.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "sepattn.h"

namespace {

#define LIB_FUNCTIONS(X)                                                                                               \
    X(sepattn_mark_separators) X(sepattn_compact_workspace_bytes) X(sepattn_compact_indices)  \
    X(sepattn_mark_compact) X(sepattn_forward_workspace_bytes) X(sepattn_forward) X(sepattn_forward_headwise)          \
    X(sepattn_backward_headwise_workspace_bytes) X(sepattn_backward_headwise) X(sepattn_doc_bounds)                    \
    X(sepattn_forward_packed) X(sepattn_backward_packed) X(sepattn_backward_workspace_bytes) X(sepattn_backward)       \
    X(sepattn_decode_workspace_bytes) X(sepattn_decode) X(sepattn_decode_noalloc) X(sepkv_evict_window)                \
    X(sepkv_fill_from_prefill) X(sepattn_decode_rope) X(sepkv_append)
// what some of them call where the outputs are their own, fresh ones
#define LIB_FRESH_FUNCTIONS(F) F(sepattn_compact_indices_filled) F(sepattn_mark_compact_filled) F(sepkv_fill_from_prefill_zeroed)
struct Lib {
#define X(name) decltype(&::name) name;
    LIB_FUNCTIONS(X)
    LIB_FRESH_FUNCTIONS(X)
#undef X
} lib;
PyObject *g_raise = nullptr;  // Python callable: raises SepattnError(function, status)

// A failed check: the Python error is set, the caller returns nullptr.
struct Failed {};
[[noreturn]] void fail(PyObject *type, const char *msg) {
    PyErr_SetString(type, msg);
    throw Failed{};
}
void require(bool ok, const char *msg) {
    if (!ok) fail(PyExc_AssertionError, msg);
}

// a tensor argument (borrowed from the caller for the duration of the call)
const at::Tensor &tensor(PyObject *o) {
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a torch tensor is expected");
    return THPVariable_Unpack(o);
}
// ... that must live on the GPU and be contiguous
const at::Tensor &dev(PyObject *o) {
    const at::Tensor &t = tensor(o);
    if (!t.is_cuda()) fail(PyExc_ValueError, "libsepattn works on GPU tensors only");
    if (!t.is_contiguous()) fail(PyExc_ValueError, "tensors must be contiguous");
    return t;
}
void *ptr(const at::Tensor &t) { return t.data_ptr(); }
void *ptr(PyObject *o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }
const int32_t *i32(const at::Tensor &t) { return static_cast<const int32_t *>(t.data_ptr()); }

void *stream_of(const at::Tensor &t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

int dtype_code(const at::Tensor &t) {
    const auto s = t.scalar_type();
    if (s == at::kBFloat16) return SEPATTN_BF16;
    if (s == at::kFloat) return SEPATTN_FP32;
    fail(PyExc_TypeError, "unsupported dtype: bf16 or fp32 expected");
}
at::Tensor empty(c10::IntArrayRef shape, at::ScalarType type, const at::Device &device) {
    return at::detail::empty_cuda(shape, type, device, std::nullopt);
}
at::Tensor fresh_like(const at::Tensor &t) { return empty(t.sizes(), t.scalar_type(), t.device()); }

long as_long(PyObject *o) {
    if (PyLong_CheckExact(o)) {
        const long v = PyLong_AsLong(o);
        if (v == -1 && PyErr_Occurred()) throw Failed{};
        return v;
    }
    PyObject *n = PyNumber_Long(o);  // what int(o) gives
    if (!n) throw Failed{};
    const long v = PyLong_AsLong(n);
    Py_DECREF(n);
    if (v == -1 && PyErr_Occurred()) throw Failed{};
    return v;
}
int as_int(PyObject *o) {
    const long v = as_long(o);
    if (v < INT32_MIN || v > INT32_MAX) fail(PyExc_OverflowError, "argument does not fit 32 bits");
    return (int)v;
}
float as_float(PyObject *o) {
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    PyObject *n = PyNumber_Float(o);  // what float(o) gives
    if (!n) throw Failed{};
    const double v = PyFloat_AS_DOUBLE(n);
    Py_DECREF(n);
    return (float)v;
}
bool as_bool(PyObject *o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Failed{};
    return v != 0;
}
// a reference that this call owns
struct Owned {
    PyObject *o;
    explicit Owned(PyObject *x) : o(x) {
        if (!o) throw Failed{};
    }
    ~Owned() { Py_DECREF(o); }
    Owned(const Owned &) = delete;
    Owned &operator=(const Owned &) = delete;
};
std::vector<int32_t> int_list(PyObject *o) {
    if (PyObject_Size(o) < 0) throw Failed{};    // an iterator is refused
    const Owned items(PySequence_Tuple(o));      // items of its own: int() of one may run code that changes the list
    const Py_ssize_t n = PyTuple_GET_SIZE(items.o);
    std::vector<int32_t> v((size_t)n);
    for (Py_ssize_t k = 0; k < n; ++k) v[(size_t)k] = (int32_t)as_long(PyTuple_GET_ITEM(items.o, k));
    return v;
}
// The N tensors of an `out` argument, which may be any iterable; None: the call allocates its own.  The items
// are held until the call has returned: an iterator that made them is no longer their owner.
template <int N>
struct Out {
    PyObject *items = nullptr;  // a tuple
    explicit Out(PyObject *o) {
        if (o == Py_None) return;
        items = PySequence_Tuple(o);
        if (!items) throw Failed{};
        if (PyTuple_GET_SIZE(items) == N) return;
        Py_DECREF(items);
        fail(PyExc_ValueError, "out: wrong number of tensors");
    }
    ~Out() { Py_XDECREF(items); }
    Out(const Out &) = delete;
    Out &operator=(const Out &) = delete;
    bool given() const { return items != nullptr; }
    PyObject *operator[](int k) const { return PyTuple_GET_ITEM(items, k); }
};
void check(const char *fn, int rc) {
    if (rc == SEPATTN_OK) return;
    PyObject *r = PyObject_CallFunction(g_raise, "si", fn, rc);
    Py_XDECREF(r);
    throw Failed{};
}
// What a call allocates and enqueues runs without the interpreter lock: the allocator may wait for the device, a
// launch for a place in a full queue, and other Python threads go on meanwhile.  Arguments are taken apart before
// (no Python object is touched inside), results wrapped afterwards.
template <typename F>
auto unlocked(F f) {
    struct Lock {
        PyThreadState *state = PyEval_SaveThread();
        ~Lock() { PyEval_RestoreThread(state); }
    } lock;
    return f();
}
// the caller's workspace, or one from torch's allocator that goes back when the call returns (the
// allocator hands it out again in stream order)
struct Workspace {
    at::Tensor own;
    void *p = nullptr;
    size_t bytes = 0;
    bool given;
    explicit Workspace(PyObject *ws) : given(ws != Py_None) {
        if (!given) return;
        const at::Tensor &t = tensor(ws);
        p = t.data_ptr();
        bytes = (size_t)t.numel();
    }
    void allocate(size_t need, const at::Device &device) {
        bytes = need < 256 ? 256 : need;
        own = empty({(int64_t)bytes}, at::kByte, device);
        p = own.data_ptr();
    }
};
PyObject *wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }
PyObject *keep(PyObject *o) {
    Py_INCREF(o);
    return o;
}
template <typename... P>
PyObject *tuple_of(P *...items) {  // takes over the references
    PyObject *t = PyTuple_New(sizeof...(items));
    Py_ssize_t k = 0;
    (PyTuple_SET_ITEM(t, k++, items), ...);
    return t;
}

sepattn_params attn_params(const at::Tensor &Q, const at::Tensor &K, int a, int n, float scale, const at::Tensor &idx) {
    if (Q.dim() != 4 || K.dim() < 2) fail(PyExc_ValueError, "Q [B,Hq,L,d] and K [B,Hkv,L,d] are expected");
    sepattn_params p;
    p.B = (int)Q.size(0);
    p.Hq = (int)Q.size(1);
    p.Hkv = (int)K.size(1);
    p.L = (int)Q.size(2);
    p.d = (int)Q.size(3);
    p.a = a;
    p.n = n;
    p.scale = scale;
    p.dtype = dtype_code(Q);
    p.cap = (int)idx.size(1);
    return p;
}

// ---- marking and compaction ----------------------------------------------------------------------
// mark_separators(token_ids, sep_ids, out)
PyObject *mark_separators(PyObject *const *a) {
    const at::Tensor &tok = dev(a[0]);
    if (a[2] != Py_None) dev(a[2]);
    require(tok.scalar_type() == at::kInt && tok.dim() == 2, "token_ids: int32 [B, L]");
    const int B = (int)tok.size(0), L = (int)tok.size(1);
    const std::vector<int32_t> ids = int_list(a[1]);
    at::Tensor out;
    if (a[2] != Py_None) out = tensor(a[2]);
    check("sepattn_mark_separators", unlocked([&] {
              if (!out.defined()) out = empty({B, L}, at::kByte, tok.device());
              return lib.sepattn_mark_separators(i32(tok), B, L, ids.data(), (int)ids.size(), (uint8_t *)ptr(out), stream_of(tok));
          }));
    return a[2] == Py_None ? wrap(std::move(out)) : keep(a[2]);
}

// Index arrays, the caller's or (`allocate`) the call's own, where every entry of the list behind the last separator is
// `fill` (the _filled entry points write it).  Arguments: the last three of `out`, cap, want_prefix, fill.
struct IndexOut {
    at::Tensor idx, cnt, pre;
    int cap = 0, fill = 0;
    bool want_prefix = false;
    int32_t *idx_p = nullptr, *cnt_p = nullptr, *pre_p = nullptr;
    template <int N>
    IndexOut(const Out<N> &out, int L, PyObject *cap_o, PyObject *want_prefix_o, PyObject *fill_o) {
        if (out.given()) {
            const at::Tensor &i = dev(out[N - 3]);
            cap = (int)i.size(1);
            idx_p = (int32_t *)ptr(i);
            cnt_p = (int32_t *)ptr(dev(out[N - 2]));
            pre_p = out[N - 1] == Py_None ? nullptr : (int32_t *)ptr(dev(out[N - 1]));
        } else {
            cap = cap_o == Py_None ? L : as_int(cap_o);
            want_prefix = as_bool(want_prefix_o);
            fill = as_int(fill_o);
        }
    }
    void allocate(int B, int L, const at::Device &device) {
        idx = empty({B, cap > 1 ? cap : 1}, at::kInt, device);
        cnt = empty({B}, at::kInt, device);
        idx_p = (int32_t *)ptr(idx), cnt_p = (int32_t *)ptr(cnt);
        if (!want_prefix) return;
        pre = empty({B, L + 1}, at::kInt, device);
        pre_p = (int32_t *)ptr(pre);
    }
    PyObject *prefix_object() const { return pre.defined() ? wrap(pre) : keep(Py_None); }
};

// compact_indices(is_sep, cap, want_prefix, fill, out, ws)
PyObject *compact_indices(PyObject *const *a) {
    const at::Tensor &sep = dev(a[0]);
    require(sep.scalar_type() == at::kByte && sep.dim() == 2, "is_sep: uint8 [B, L]");
    const int B = (int)sep.size(0), L = (int)sep.size(1);
    const Out<3> out(a[4]);
    IndexOut o(out, L, a[1], a[2], a[3]);
    Workspace ws(a[5]);
    check("sepattn_compact_indices", unlocked([&] {
              if (!ws.given) ws.allocate(lib.sepattn_compact_workspace_bytes(B, L), sep.device());
              if (!out.given()) o.allocate(B, L, sep.device());
              if (!out.given())
                  return lib.sepattn_compact_indices_filled((const uint8_t *)ptr(sep), B, L, o.idx_p, o.cap, o.cnt_p, o.pre_p, o.fill,
                                                            ws.p, ws.bytes, stream_of(sep));
              return lib.sepattn_compact_indices((const uint8_t *)ptr(sep), B, L, o.idx_p, o.cap, o.cnt_p, o.pre_p, ws.p, ws.bytes,
                                                 stream_of(sep));
          }));
    if (out.given()) return tuple_of(keep(out[0]), keep(out[1]), keep(out[2]));
    return tuple_of(wrap(o.idx), wrap(o.cnt), o.prefix_object());
}

// mark_compact(token_ids, sep_ids, cap, want_prefix, fill, out, ws)
PyObject *mark_compact(PyObject *const *a) {
    const at::Tensor &tok = dev(a[0]);
    require(tok.scalar_type() == at::kInt && tok.dim() == 2, "token_ids: int32 [B, L]");
    const int B = (int)tok.size(0), L = (int)tok.size(1);
    const std::vector<int32_t> ids = int_list(a[1]);
    const Out<4> out(a[5]);
    at::Tensor sep;
    if (out.given()) sep = dev(out[0]);
    IndexOut o(out, L, a[2], a[3], a[4]);
    Workspace ws(a[6]);
    check("sepattn_mark_compact", unlocked([&] {
              if (!ws.given) ws.allocate(lib.sepattn_compact_workspace_bytes(B, L), tok.device());
              if (!out.given()) {
                  sep = empty({B, L}, at::kByte, tok.device());
                  o.allocate(B, L, tok.device());
                  return lib.sepattn_mark_compact_filled(i32(tok), B, L, ids.data(), (int)ids.size(), (uint8_t *)ptr(sep), o.idx_p,
                                                         o.cap, o.cnt_p, o.pre_p, o.fill, ws.p, ws.bytes, stream_of(tok));
              }
              return lib.sepattn_mark_compact(i32(tok), B, L, ids.data(), (int)ids.size(), (uint8_t *)ptr(sep), o.idx_p, o.cap,
                                              o.cnt_p, o.pre_p, ws.p, ws.bytes, stream_of(tok));
          }));
    if (out.given()) return tuple_of(keep(out[0]), keep(out[1]), keep(out[2]), keep(out[3]));
    return tuple_of(wrap(std::move(sep)), wrap(o.idx), wrap(o.cnt), o.prefix_object());
}

// doc_bounds(cu_seqlens, L, a, is_sep_row, out)
PyObject *doc_bounds(PyObject *const *a) {
    const at::Tensor &cu = dev(a[0]);
    if (a[3] != Py_None) dev(a[3]);
    require(cu.scalar_type() == at::kInt && cu.dim() == 1, "cu_seqlens: int32 [n_docs + 1]");
    const int L = as_int(a[1]);
    const int n_docs = (int)cu.numel() - 1, init = as_int(a[2]);
    // `out` itself is returned, so it has to be a sequence; items beyond the two are left alone
    const Out<2> out(Owned(a[4] == Py_None ? keep(Py_None) : PySequence_GetSlice(a[4], 0, 2)).o);
    at::Tensor s, e;
    if (out.given()) {
        s = dev(out[0]);
        e = dev(out[1]);
    }
    uint8_t *row = (uint8_t *)ptr(a[3]);
    check("sepattn_doc_bounds", unlocked([&] {
              if (!out.given()) {
                  s = empty({L}, at::kInt, cu.device());
                  e = empty({L}, at::kInt, cu.device());
              }
              return lib.sepattn_doc_bounds(i32(cu), n_docs, L, init, (int32_t *)ptr(s), (int32_t *)ptr(e), row, stream_of(cu));
          }));
    if (out.given()) return keep(a[4]);
    return tuple_of(wrap(std::move(s)), wrap(std::move(e)));
}

// ---- attention -------------------------------------------------------------------------------------
// The three forms of a call differ in what stands between the sizes and the tensors: nothing, the
// heads' windows, or the documents' bounds (nh / ds, de).
enum Form { kPlain, kHeadwise, kPacked };

// the documents' bounds of a packed call: the kernels read a row of L entries for every row of the batch
struct DocBounds {
    const int32_t *start, *end;
    DocBounds(PyObject *so, PyObject *eo, const sepattn_params &p) {
        const at::Tensor &s = dev(so), &e = dev(eo);
        require(s.scalar_type() == at::kInt && e.scalar_type() == at::kInt && s.dim() == 2 && s.size(0) == p.B &&
                    s.size(1) == p.L && e.sizes() == s.sizes(), "doc_start, doc_end: int32 [B, L]");
        start = i32(s);
        end = i32(e);
    }
};

// forward(Q, K, V, sep_idx, sep_count, sep_prefix, a, n | n_per_head, scale, out, ws [, doc_start, doc_end])
template <Form F>
PyObject *forward(PyObject *const *a) {
    const at::Tensor &Q = dev(a[0]), &K = dev(a[1]), &V = dev(a[2]), &idx = dev(a[3]), &cnt = dev(a[4]), &pre = dev(a[5]);
    require(K.sizes() == V.sizes() && Q.scalar_type() == K.scalar_type() && K.scalar_type() == V.scalar_type(),
            "K and V of one shape, Q, K, V of one dtype");
    const sepattn_params p = attn_params(Q, K, as_int(a[6]), F == kHeadwise ? 1 : as_int(a[7]), as_float(a[8]), idx);
    std::vector<int32_t> nh;
    const int32_t *ds = nullptr, *de = nullptr;
    if constexpr (F == kHeadwise) {
        nh = int_list(a[7]);
        require((int)nh.size() == p.Hq, "n_per_head: one window per query head");
    }
    if constexpr (F == kPacked) {
        const DocBounds d(a[11], a[12], p);
        ds = d.start, de = d.end;
    }
    const Out<2> out(a[9]);
    at::Tensor O, LSE;
    void *optr = nullptr, *lptr = nullptr;
    if (out.given()) optr = ptr(out[0]), lptr = ptr(out[1]);
    Workspace ws(a[10]);
    constexpr const char *name = F == kPlain ? "sepattn_forward" : (F == kHeadwise ? "sepattn_forward_headwise" : "sepattn_forward_packed");
    check(name, unlocked([&] {
              if (!out.given()) {
                  O = fresh_like(Q);
                  LSE = empty({p.B, p.Hq, p.L}, at::kFloat, Q.device());
                  optr = ptr(O), lptr = ptr(LSE);
              }
              // (the forward needs no workspace; the query keeps this right if that changes)
              const size_t need = lib.sepattn_forward_workspace_bytes(&p);
              if (!ws.given && need > 0) ws.allocate(need, Q.device());
              float *lse = (float *)lptr;
              void *st = stream_of(Q);
              if constexpr (F == kPlain)
                  return lib.sepattn_forward(&p, ptr(Q), ptr(K), ptr(V), i32(idx), i32(cnt), i32(pre), optr, lse, ws.p, ws.bytes, st);
              else if constexpr (F == kHeadwise)
                  return lib.sepattn_forward_headwise(&p, nh.data(), ptr(Q), ptr(K), ptr(V), i32(idx), i32(cnt), i32(pre), optr, lse,
                                                      ws.p, ws.bytes, st);
              else
                  return lib.sepattn_forward_packed(&p, ds, de, ptr(Q), ptr(K), ptr(V), i32(idx), i32(cnt), i32(pre), optr, lse, ws.p,
                                                    ws.bytes, st);
          }));
    if (out.given()) return tuple_of(keep(out[0]), keep(out[1]));
    return tuple_of(wrap(std::move(O)), wrap(std::move(LSE)));
}

// backward(Q, K, V, O, LSE, dO, sep_idx, sep_count, sep_prefix, a, n | n_per_head, scale, out, ws [, doc_start, doc_end])
template <Form F>
PyObject *backward(PyObject *const *a) {
    const at::Tensor &Q = dev(a[0]), &K = dev(a[1]), &V = dev(a[2]), &O = dev(a[3]), &LSE = dev(a[4]), &dO = dev(a[5]),
                     &idx = dev(a[6]), &cnt = dev(a[7]), &pre = dev(a[8]);
    const sepattn_params p = attn_params(Q, K, as_int(a[9]), F == kHeadwise ? 1 : as_int(a[10]), as_float(a[11]), idx);
    std::vector<int32_t> nh;
    const int32_t *ds = nullptr, *de = nullptr;
    if constexpr (F == kHeadwise) {
        nh = int_list(a[10]);
        require((int)nh.size() == p.Hq, "n_per_head: one window per query head");
    }
    if constexpr (F == kPacked) {
        const DocBounds d(a[14], a[15], p);
        ds = d.start, de = d.end;
    }
    const Out<3> out(a[12]);
    at::Tensor g[3];
    void *gp[3];
    for (int k = 0; out.given() && k < 3; ++k) gp[k] = ptr(out[k]);
    Workspace ws(a[13]);
    constexpr const char *name = F == kPlain ? "sepattn_backward" : (F == kHeadwise ? "sepattn_backward_headwise" : "sepattn_backward_packed");
    check(name, unlocked([&] {
              if (!out.given()) {
                  g[0] = fresh_like(Q);
                  g[1] = fresh_like(K);
                  g[2] = fresh_like(V);
                  for (int k = 0; k < 3; ++k) gp[k] = ptr(g[k]);
              }
              if (!ws.given)
                  ws.allocate(F == kHeadwise ? lib.sepattn_backward_headwise_workspace_bytes(&p, nh.data())
                                             : lib.sepattn_backward_workspace_bytes(&p), Q.device());
              const float *lse = (const float *)ptr(LSE);
              void *st = stream_of(Q);
              if constexpr (F == kPlain)
                  return lib.sepattn_backward(&p, ptr(Q), ptr(K), ptr(V), ptr(O), lse, ptr(dO), i32(idx), i32(cnt), i32(pre), gp[0],
                                              gp[1], gp[2], ws.p, ws.bytes, st);
              else if constexpr (F == kHeadwise)
                  return lib.sepattn_backward_headwise(&p, nh.data(), ptr(Q), ptr(K), ptr(V), ptr(O), lse, ptr(dO), i32(idx), i32(cnt),
                                                       i32(pre), gp[0], gp[1], gp[2], ws.p, ws.bytes, st);
              else
                  return lib.sepattn_backward_packed(&p, ds, de, ptr(Q), ptr(K), ptr(V), ptr(O), lse, ptr(dO), i32(idx), i32(cnt),
                                                     i32(pre), gp[0], gp[1], gp[2], ws.p, ws.bytes, st);
          }));
    if (out.given()) return tuple_of(keep(out[0]), keep(out[1]), keep(out[2]));
    return tuple_of(wrap(std::move(g[0])), wrap(std::move(g[1])), wrap(std::move(g[2])));
}

// ---- the streaming cache ---------------------------------------------------------------------------
const at::Tensor &sizes_arg(PyObject *o) {
    const at::Tensor &t = dev(o);
    require(t.scalar_type() == at::kInt && t.dim() == 2 && t.size(1) == SEPKV_SIZES_COLS, "sizes: int32 [S, 6]");
    return t;
}
sepkv_params kv_params(const at::Tensor &Kc, int S, int Hq, int a, int s, int w, float scale) {
    if (Kc.dim() != 4) fail(PyExc_ValueError, "Kc [S,Hkv,c,d] is expected");
    sepkv_params p;
    p.S = S;
    p.Hq = Hq;
    p.Hkv = (int)Kc.size(1);
    p.d = (int)Kc.size(3);
    p.a = a;
    p.s = s;
    p.w = w;
    p.c = (int)Kc.size(2);
    p.scale = scale;
    p.dtype = dtype_code(Kc);
    return p;
}

enum Decode { kKept, kRope, kNoAlloc };  // positions as the keys hold them, by place in the cache; no allocation

// decode(q, Kc, Vc, sizes, rope_table, a, s, w, scale, out, ws): the table is looked at with kRope only; kNoAlloc: out is
// required, ws unused
template <Decode F>
PyObject *decode(PyObject *const *a) {
    const at::Tensor &q = dev(a[0]), &Kc = dev(a[1]), &Vc = dev(a[2]);
    const at::Tensor *table = F == kRope ? &dev(a[4]) : nullptr;
    const at::Tensor &sizes = sizes_arg(a[3]);
    if (q.dim() != 3) fail(PyExc_ValueError, "q [S,Hq,d] is expected");
    if (F == kRope)
        require(table->scalar_type() == at::kFloat && table->dim() == 3 && table->size(1) == 2 && table->size(2) * 2 == q.size(2),
                "rope_table: fp32 [n_pos, 2, d/2]");
    sepkv_params p = kv_params(Kc, (int)q.size(0), (int)q.size(1), as_int(a[5]), as_int(a[6]), as_int(a[7]), as_float(a[8]));
    p.d = (int)q.size(2);
    const Out<2> out(a[9]);
    if (F == kNoAlloc && !out.given()) fail(PyExc_TypeError, "out is required");
    at::Tensor o, lse;
    void *optr = nullptr, *lptr = nullptr;
    if (out.given()) optr = ptr(out[0]), lptr = ptr(out[1]);  // an item None: no LSE wanted
    Workspace ws(F == kNoAlloc ? Py_None : a[10]);
    check(F == kNoAlloc ? "sepattn_decode_noalloc" : (F == kRope ? "sepattn_decode_rope" : "sepattn_decode"), unlocked([&] {
              if (!out.given()) {
                  o = fresh_like(q);
                  lse = empty({p.S, p.Hq}, at::kFloat, q.device());
                  optr = ptr(o), lptr = ptr(lse);
              }
              if (F != kNoAlloc && !ws.given) ws.allocate(lib.sepattn_decode_workspace_bytes(&p), q.device());
              void *st = stream_of(q);
              if constexpr (F == kNoAlloc)
                  return lib.sepattn_decode_noalloc(&p, ptr(q), ptr(Kc), ptr(Vc), i32(sizes), optr, (float *)lptr, st);
              else if constexpr (F == kRope)
                  return lib.sepattn_decode_rope(&p, ptr(q), ptr(Kc), ptr(Vc), i32(sizes), (const float *)ptr(*table),
                                                 (int)table->size(0), optr, (float *)lptr, ws.p, ws.bytes, st);
              else
                  return lib.sepattn_decode(&p, ptr(q), ptr(Kc), ptr(Vc), i32(sizes), optr, (float *)lptr, ws.p, ws.bytes, st);
          }));
    if (out.given()) return tuple_of(keep(out[0]), keep(out[1]));
    return tuple_of(wrap(std::move(o)), wrap(std::move(lse)));
}

// append(k_new, v_new, is_sep_new, Kc, Vc, win_is_sep, sizes, Hq, a, s, w)
PyObject *append(PyObject *const *a) {
    const at::Tensor &k = dev(a[0]), &v = dev(a[1]), &sep = dev(a[2]), &Kc = dev(a[3]), &Vc = dev(a[4]), &flags = dev(a[5]);
    const at::Tensor &sizes = sizes_arg(a[6]);
    require(sep.scalar_type() == at::kByte && flags.scalar_type() == at::kByte, "is_sep_new, win_is_sep: uint8");
    const sepkv_params p = kv_params(Kc, (int)Kc.size(0), as_int(a[7]), as_int(a[8]), as_int(a[9]), as_int(a[10]), 1.0f);
    const int64_t want[3] = {p.S, p.Hkv, p.d};
    require(k.sizes() == c10::IntArrayRef(want, 3) && v.sizes() == k.sizes() && k.scalar_type() == Kc.scalar_type(),
            "k_new, v_new: [S, Hkv, d] in the cache's dtype");
    check("sepkv_append", unlocked([&] {
              return lib.sepkv_append(&p, ptr(k), ptr(v), (const uint8_t *)ptr(sep), ptr(Kc), ptr(Vc), (uint8_t *)ptr(flags),
                                      (int32_t *)ptr(sizes), stream_of(Kc));
          }));
    return keep(Py_None);
}

// evict_window(Kc, Vc, win_is_sep, sizes, Hq, a, s, w, ws)
PyObject *evict_window(PyObject *const *a) {
    const at::Tensor &Kc = dev(a[0]), &Vc = dev(a[1]), &flags = dev(a[2]);
    const at::Tensor &sizes = sizes_arg(a[3]);
    const sepkv_params p = kv_params(Kc, (int)Kc.size(0), as_int(a[4]), as_int(a[5]), as_int(a[6]), as_int(a[7]), 1.0f);
    // the step needs no scratch memory: a workspace is passed on if the caller has one, NULL otherwise
    const Workspace ws(a[8]);
    check("sepkv_evict_window", unlocked([&] {
              return lib.sepkv_evict_window(&p, ptr(Kc), ptr(Vc), (const uint8_t *)ptr(flags), (int32_t *)ptr(sizes), ws.p, ws.bytes,
                                            stream_of(Kc));
          }));
    return keep(Py_None);
}

// fill_from_prefill(K, V, is_sep, sep_idx, sep_prefix, Hq, a, s, w, c, nw, out)
PyObject *fill_from_prefill(PyObject *const *a) {
    const at::Tensor &K = dev(a[0]), &V = dev(a[1]), &sep = dev(a[2]), &idx = dev(a[3]), &pre = dev(a[4]);
    const int L = K.dim() == 4 ? (int)K.size(2) : 0, nw = as_int(a[10]);
    sepkv_params p = kv_params(K, (int)K.size(0), as_int(a[5]), as_int(a[6]), as_int(a[7]), as_int(a[8]), 1.0f);
    p.c = as_int(a[9]);
    const Out<4> out(a[11]);
    at::Tensor Kc, Vc, flags, sizes;
    if (out.given()) {
        Kc = dev(out[0]);
        Vc = dev(out[1]);
        flags = dev(out[2]);
        sizes = dev(out[3]);
        require(sizes.scalar_type() == at::kInt && sizes.dim() == 2 && sizes.size(0) == p.S && sizes.size(1) == SEPKV_SIZES_COLS,
                "sizes: int32 [S, 6]");
    }
    check("sepkv_fill_from_prefill", unlocked([&] {
              if (!out.given()) {
                  Kc = empty({p.S, p.Hkv, p.c, p.d}, K.scalar_type(), K.device());
                  Vc = empty({p.S, p.Hkv, p.c, p.d}, K.scalar_type(), K.device());
                  flags = empty({p.S, p.c - p.a - p.s}, at::kByte, K.device());
                  sizes = empty({p.S, SEPKV_SIZES_COLS}, at::kInt, K.device());
              }
              const auto fill = out.given() ? lib.sepkv_fill_from_prefill : lib.sepkv_fill_from_prefill_zeroed;
              return fill(&p, L, nw, ptr(K), ptr(V), (const uint8_t *)ptr(sep), i32(idx), (int)idx.size(1),
                          i32(pre), ptr(Kc), ptr(Vc), (uint8_t *)ptr(flags), (int32_t *)ptr(sizes), stream_of(K));
          }));
    if (out.given()) return tuple_of(keep(out[0]), keep(out[1]), keep(out[2]), keep(out[3]));
    return tuple_of(wrap(std::move(Kc)), wrap(std::move(Vc)), wrap(std::move(flags)), wrap(std::move(sizes)));
}

// ---- module ------------------------------------------------------------------------------------------
typedef PyObject *(*Body)(PyObject *const *);
template <Body F, int N>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Failed &) {
        return nullptr;
    } catch (...) {  // torch's own errors as the Python classes it gives them (OutOfMemoryError, IndexError, ...)
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

// bind(path, raise_error): open the library and look its entry points up
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "bind(path, raise_error)");
        return nullptr;
    }
    const char *path = PyUnicode_AsUTF8(args[0]);
    if (!path) return nullptr;
    void *h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!h) {
        PyErr_SetString(PyExc_OSError, dlerror());
        return nullptr;
    }
#define X(name)                                                            \
    lib.name = reinterpret_cast<decltype(lib.name)>(dlsym(h, #name));      \
    if (!lib.name) {                                                       \
        PyErr_SetString(PyExc_OSError, #name " is missing in the library"); \
        return nullptr;                                                    \
    }
    LIB_FUNCTIONS(X)
    LIB_FRESH_FUNCTIONS(X)
#undef X
    Py_INCREF(args[1]);
    Py_XSETREF(g_raise, args[1]);
    Py_RETURN_NONE;
}

#define METHOD(name, body, count) \
    {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&entry<body, count>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&bind)), METH_FASTCALL, nullptr},
    METHOD("mark_separators", mark_separators, 3),
    METHOD("compact_indices", compact_indices, 6),
    METHOD("mark_compact", mark_compact, 7),
    METHOD("doc_bounds", doc_bounds, 5),
    METHOD("forward", forward<kPlain>, 11),
    METHOD("forward_headwise", forward<kHeadwise>, 11),
    METHOD("forward_packed", forward<kPacked>, 13),
    METHOD("backward", backward<kPlain>, 14),
    METHOD("backward_headwise", backward<kHeadwise>, 14),
    METHOD("backward_packed", backward<kPacked>, 16),
    METHOD("decode", decode<kKept>, 11),
    METHOD("decode_rope", decode<kRope>, 11),
    METHOD("decode_noalloc", decode<kNoAlloc>, 11),
    METHOD("append", append, 11),
    METHOD("evict_window", evict_window, 9),
    METHOD("fill_from_prefill", fill_from_prefill, 12),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
