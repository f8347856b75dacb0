// The way of an ordinary call from Python to the C ABI in native code: the checks and the argument marshalling of
// rekv.py's methods on torch tensors without a Python attribute access or a ctypes conversion each.
//
// A method takes only what needs no second look: plain torch tensors (no subclass, no dispatch or function
// mode, not traced), plain ints and floats, the usual number of dimensions, everything valid.  Anything else makes it return None and
// leaves the call to the Python method, which names what is wrong or serves the unusual form.  So the methods
// here never refuse a call and never differ in what they launch.
//
// Host time with the launches, as Python methods over ctypes and so (us): a decode step 9.0 -> 3.6, a live frame's two calls
// 11.8 -> 6.6, a question's retrieval, reload and attention 24.5 -> 15.5, 28 layers of them 68 -> 26.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <initializer_list>

#include "rekv.h"

namespace {

using at::Tensor;

PyObject* g_raise = nullptr;                 // raise(status, context address): throws RekvError

struct Context {
    PyObject_HEAD
    rekv_ctx* h;
    int64_t hq, hkv, d, nf;
    at::ScalarType dtype;
};

// One call's arguments: every getter clears `ok` where the argument is not of the ordinary form.
struct Args {
    Context* c;
    bool ok = true;

    explicit Args(PyObject* self) : c(reinterpret_cast<Context*>(self)) {
        ok = c->h && !at::impl::torch_function_mode_enabled() && !c10::impl::dispatch_mode_enabled() && !torch::jit::tracer::isTracing();
    }
    bool no() { return ok = false; }
    void need(bool cond) { ok = ok && cond; }

    const Tensor* tensor(PyObject* o) {
        if (!ok || !THPVariable_CheckExact(o)) return no(), nullptr;
        const Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || at::isTensorSubclassLike(t) || t.layout() != at::kStrided) return no(), nullptr;
        return &t;
    }
    // a contiguous device tensor of so many dimensions, of a type, with the given last sizes
    const Tensor* device(PyObject* o, int64_t dims, at::ScalarType type, std::initializer_list<int64_t> last = {}) {
        const Tensor* t = tensor(o);
        if (!t) return nullptr;
        need(t->is_cuda() && t->scalar_type() == type && (dims < 0 || t->dim() == dims) && t->is_contiguous());
        if (ok) {
            int64_t i = t->dim() - (int64_t)last.size();
            need(i >= 0);
            for (int64_t n : last) need(ok && t->size(i++) == n);
        }
        return ok ? t : nullptr;
    }
    const Tensor* queries(PyObject* o, int64_t dims) { return device(o, dims, c->dtype, {c->hq, c->d}); }
    const Tensor* keys(PyObject* o, int64_t dims) { return device(o, dims, c->dtype, {c->hkv, c->d}); }
    int64_t i64(PyObject* o) {
        if (!ok || !PyLong_CheckExact(o)) return no(), 0;
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &over);
        if (over || v > (1ll << 61) || v < -(1ll << 61)) return no(), 0;
        return v;
    }
    int32_t i32(PyObject* o) {
        const int64_t v = i64(o);
        if (v != (int32_t)v) return no(), 0;
        return (int32_t)v;
    }
    double f64(PyObject* o) {
        if (!ok || !PyFloat_CheckExact(o)) return no(), 0.0;
        return PyFloat_AS_DOUBLE(o);
    }
    bool flag(PyObject* o) {
        if (!ok || !PyBool_Check(o)) return no(), false;
        return o == Py_True;
    }
    // one of two words: 0 or 1
    int32_t word(PyObject* o, const char* zero, const char* one) {
        if (!ok || !PyUnicode_CheckExact(o)) return no(), 0;
        if (PyUnicode_CompareWithASCIIString(o, zero) == 0) return 0;
        if (PyUnicode_CompareWithASCIIString(o, one) == 0) return 1;
        return no(), 0;
    }
    // frames in an arena: given, or as many as it holds; the arena's K and V hold them
    int32_t frames(PyObject* o, const Tensor* k, const Tensor* v) {
        if (!ok) return 0;
        const int64_t n = o == Py_None ? k->size(0) / c->nf : i32(o);
        need(n == (int32_t)n && k->size(0) >= n * c->nf && v->sizes() == k->sizes());
        return (int32_t)n;
    }
    const int32_t* n_sel(PyObject* o, int64_t nq) {
        if (!ok || o == Py_None) return nullptr;
        const Tensor* t = device(o, -1, at::kInt);
        need(t && t->numel() == nq);
        return ok ? static_cast<const int32_t*>(t->data_ptr()) : nullptr;
    }
    static bool fits(int64_t v) { return v == (int32_t)v; }
};

void* ptr(const Tensor& t) { return t.data_ptr(); }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// An output: the caller's tensor (a reference of its own), or a new one.
struct Out {
    PyObject* given;
    Tensor made;
    explicit Out(PyObject* o) : given(o == Py_None ? nullptr : o) {}
    const Tensor& get() const { return given ? THPVariable_Unpack(given) : made; }
    PyObject* take() const {
        if (!given) return THPVariable_Wrap(made);
        Py_INCREF(given);
        return given;
    }
};

PyObject* raise_status(Context* c, rekv_status st) {
    Py_XDECREF(PyObject_CallFunction(g_raise, "iK", (int)st, (unsigned long long)(uintptr_t)c->h));
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "a rekv call failed");
    return nullptr;
}

// Runs the C call without the interpreter lock (a growing workspace waits for the device).  The call's arguments are worked
// out before the lock is given up: a tensor's address can throw (no storage behind it, a lazy copy that finds no memory), and
// another thread may give the tensor other storage.
template <class... P, class... A>
rekv_status outside(rekv_status (*call)(P...), A... args) {
    PyThreadState* s = PyEval_SaveThread();
    const rekv_status st = call(args...);
    PyEval_RestoreThread(s);
    return st;
}

// Body of every method: exceptions of torch (an allocation that fails) leave the call to the Python method, which meets them again.
template <class Body>
PyObject* guarded(Body body) {
    try {
        PyObject* r = body();
        if (r || PyErr_Occurred()) return r;
    } catch (...) {
        PyErr_Clear();
    }
    Py_RETURN_NONE;
}

#define METHOD(name, count)                                                              \
    PyObject* name##_body(PyObject* self, PyObject* const* a);                           \
    PyObject* name(PyObject* self, PyObject* const* a, Py_ssize_t n) {                   \
        if (n != (count)) Py_RETURN_NONE;                                                \
        return guarded([&] { return name##_body(self, a); });                            \
    }                                                                                    \
    PyObject* name##_body(PyObject* self, PyObject* const* a)

at::TensorOptions on(const Tensor& t, at::ScalarType type) { return at::TensorOptions().device(t.device()).dtype(type); }

METHOD(encode_chunk, 8) {        // q, k_cache, v_cache, first_token, l_x, n_chunks, l_l, out
    Args g(self);
    const Tensor *q = g.queries(a[0], 3), *k = g.keys(a[1], 3), *v = g.keys(a[2], 3);
    const int64_t first = g.i64(a[3]);
    const int32_t l_x = g.i32(a[4]), n_chunks = g.i32(a[5]), l_l = g.i32(a[6]);
    if (!g.ok) return nullptr;
    const int64_t n = (int64_t)n_chunks * l_x;
    g.need(q->size(0) == n && k->size(0) >= first + n && v->size(0) == k->size(0));
    Out out(a[7]);
    if (g.ok && !out.given) out.made = at::empty_like(*q);
    else g.need(g.ok && g.queries(a[7], 3) && out.get().sizes() == q->sizes());
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(rekv_encode_chunk, g.c->h, ptr(*q), ptr(*k), ptr(*v), first, l_x, n_chunks, l_l, ptr(out.get()), s);
    return st ? raise_status(g.c, st) : out.take();
}

METHOD(frame_keys, 3) {          // k, n_frames, out
    Args g(self);
    const Tensor* k = g.keys(a[0], 3);
    const int32_t n = g.i32(a[1]);
    if (!g.ok) return nullptr;
    const int64_t dp = g.c->hkv * g.c->d;
    g.need(n >= 0 && k->size(0) >= n * g.c->nf);
    Out out(a[2]);
    if (g.ok && !out.given) out.made = at::empty({n, dp}, on(*k, at::kFloat));
    else g.need(g.ok && g.device(a[2], 2, at::kFloat, {dp}) && out.get().size(0) >= n);
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(rekv_frame_keys, g.c->h, ptr(*k), n, static_cast<float*>(ptr(out.get())), s);
    return st ? raise_status(g.c, st) : out.take();
}

PyObject* selection(const Tensor& idx, const Tensor& n_sel, const Tensor* scores) {
    PyObject* r = PyTuple_New(3);
    PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(idx));
    PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(n_sel));
    if (!scores) Py_INCREF(Py_None);
    PyTuple_SET_ITEM(r, 2, scores ? THPVariable_Wrap(*scores) : Py_None);
    return r;
}

METHOD(retrieve_topk, 6) {       // frame_keys, n_frames, q_question, k, frame_keys_stride, want_scores
    Args g(self);
    const Tensor *fk = g.device(a[0], -1, at::kFloat), *q = g.queries(a[2], 4);
    const int32_t n_frames = g.i32(a[1]), k = g.i32(a[3]);
    const int64_t stride = g.i64(a[4]);
    const bool want = g.flag(a[5]);
    if (!g.ok) return nullptr;
    const int64_t nq = q->size(0), nt = q->size(1), dp = g.c->hkv * g.c->d;
    g.need(n_frames >= 0 && k >= 0 && Args::fits(nq) && Args::fits(nt) && stride >= 0 && stride < (1ll << 40) &&
           fk->numel() >= (stride ? nq - 1 : 0) * stride + n_frames * dp);
    if (!g.ok) return nullptr;
    const Tensor idx = at::empty({nq, k}, on(*q, at::kInt)), n_sel = at::empty({nq}, on(*q, at::kInt));
    Tensor scores;
    if (want) scores = at::empty({nq, n_frames}, on(*q, at::kFloat));
    void* s = stream();
    const rekv_status st = outside(rekv_retrieve_topk, g.c->h, static_cast<const float*>(ptr(*fk)), stride, n_frames, ptr(*q), (int32_t)nq,
                                   (int32_t)nt, k, static_cast<int32_t*>(ptr(idx)), static_cast<int32_t*>(ptr(n_sel)),
                                   want ? static_cast<float*>(ptr(scores)) : nullptr, s);
    return st ? raise_status(g.c, st) : selection(idx, n_sel, want ? &scores : nullptr);
}

METHOD(retrieve_external, 5) {   // frame_emb, q_emb, k, tau, want_scores
    Args g(self);
    const Tensor *fe = g.device(a[0], 2, at::kFloat), *qe = g.device(a[1], 2, at::kFloat);
    const int32_t k = g.i32(a[2]);
    const double tau = g.f64(a[3]);
    const bool want = g.flag(a[4]);
    if (!g.ok) return nullptr;
    const int64_t n_frames = fe->size(0), dim = fe->size(1), nq = qe->size(0);
    g.need(qe->size(1) == dim && k >= 0 && Args::fits(n_frames) && Args::fits(dim) && Args::fits(nq));
    if (!g.ok) return nullptr;
    const Tensor idx = at::empty({nq, k}, on(*qe, at::kInt)), n_sel = at::empty({nq}, on(*qe, at::kInt));
    Tensor scores;
    if (want) scores = at::empty({nq, n_frames}, on(*qe, at::kFloat));
    void* s = stream();
    const rekv_status st = outside(rekv_retrieve_external, g.c->h, static_cast<const float*>(ptr(*fe)), (int32_t)n_frames, (int32_t)dim,
                                   static_cast<const float*>(ptr(*qe)), (int32_t)nq, (float)tau, k, static_cast<int32_t*>(ptr(idx)),
                                   static_cast<int32_t*>(ptr(n_sel)), want ? static_cast<float*>(ptr(scores)) : nullptr, s);
    return st ? raise_status(g.c, st) : selection(idx, n_sel, want ? &scores : nullptr);
}

METHOD(block_keys, 4) {          // frame_keys, n_frames, b, out
    Args g(self);
    const Tensor* fk = g.device(a[0], -1, at::kFloat);
    const int32_t n_frames = g.i32(a[1]), b = g.i32(a[2]);
    if (!g.ok) return nullptr;
    const int64_t dp = g.c->hkv * g.c->d;
    g.need(n_frames >= 0 && b > 0 && fk->numel() >= n_frames * dp);
    if (!g.ok) return nullptr;
    const int64_t n_blocks = ((int64_t)n_frames + b - 1) / b;
    Out out(a[3]);
    if (!out.given) out.made = at::empty({n_blocks > 1 ? n_blocks : 1, dp}, on(*fk, at::kFloat));
    else g.need(g.device(a[3], -1, at::kFloat) && out.get().numel() >= n_blocks * dp);
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(rekv_block_keys, g.c->h, static_cast<const float*>(ptr(*fk)), n_frames, b, static_cast<float*>(ptr(out.get())), s);
    return st ? raise_status(g.c, st) : out.take();
}

PyObject* pair(const Out& x, const Out& y) {
    PyObject* r = PyTuple_New(2);
    PyTuple_SET_ITEM(r, 0, x.take());
    PyTuple_SET_ITEM(r, 1, y.take());
    return r;
}

METHOD(expand_blocks, 3) {       // block_idx, b, n_frames
    Args g(self);
    const Tensor* blk = g.device(a[0], 2, at::kInt);
    const int32_t b = g.i32(a[1]), n_frames = g.i32(a[2]);
    if (!g.ok) return nullptr;
    const int64_t nq = blk->size(0), kb = blk->size(1);
    g.need(b >= 0 && Args::fits(nq) && Args::fits(kb));
    if (!g.ok) return nullptr;
    Out idx(Py_None), n_sel(Py_None);
    idx.made = at::empty({nq, kb * b}, on(*blk, at::kInt));
    n_sel.made = at::empty({nq}, on(*blk, at::kInt));
    void* s = stream();
    const rekv_status st = outside(rekv_expand_blocks, g.c->h, static_cast<const int32_t*>(ptr(*blk)), (int32_t)nq, (int32_t)kb, b, n_frames,
                                   static_cast<int32_t*>(ptr(idx.made)), static_cast<int32_t*>(ptr(n_sel.made)), s);
    return st ? raise_status(g.c, st) : pair(idx, n_sel);
}

METHOD(gather_kv, 6) {           // src_k, src_v, idx, n_src_frames, dst_k, dst_v; device sources
    Args g(self);
    const Tensor *k = g.keys(a[0], 3), *v = g.keys(a[1], 3), *idx = g.device(a[2], 2, at::kInt);
    const int32_t n_src = g.frames(a[3], k, v);
    if (!g.ok) return nullptr;
    const int64_t nq = idx->size(0), slots = idx->size(1);
    const int64_t shape[4] = {nq, slots * g.c->nf, g.c->hkv, g.c->d};
    g.need(Args::fits(nq) && Args::fits(slots));
    Out dk(a[4]), dv(a[5]);
    for (Out* o : {&dk, &dv}) {
        if (!g.ok) return nullptr;
        if (!o->given) o->made = at::empty(shape, on(*idx, g.c->dtype));
        else g.need(g.device(o->given, 4, g.c->dtype) && o->get().sizes() == at::IntArrayRef(shape));
    }
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(rekv_gather_kv, g.c->h, ptr(*k), ptr(*v), 0, n_src, static_cast<const int32_t*>(ptr(*idx)), (int32_t)nq,
                                   (int32_t)slots, ptr(dk.get()), ptr(dv.get()), s);
    return st ? raise_status(g.c, st) : pair(dk, dv);
}

METHOD(gather_kv_layers, 6) {    // src_k, src_v (lists), idx, n_src_frames, dst_k, dst_v
    constexpr int MOST = 256;
    Args g(self);
    const Tensor* idx = g.device(a[2], 3, at::kInt);
    g.need(PyList_CheckExact(a[0]) && PyList_CheckExact(a[1]));
    if (!g.ok) return nullptr;
    const int64_t layers = PyList_GET_SIZE(a[0]), nq = idx->size(1), slots = idx->size(2);
    g.need(layers >= 1 && layers <= MOST && PyList_GET_SIZE(a[1]) == layers && idx->size(0) == layers && Args::fits(nq) && Args::fits(slots));
    if (!g.ok) return nullptr;
    const Tensor* first = g.keys(PyList_GET_ITEM(a[0], 0), 3);
    if (!g.ok) return nullptr;
    const int64_t n_src = a[3] == Py_None ? first->size(0) / g.c->nf : g.i32(a[3]);
    g.need(Args::fits(n_src));
    const void *pk[MOST], *pv[MOST];
    for (int64_t i = 0; i < layers; ++i) {
        const Tensor *k = g.keys(PyList_GET_ITEM(a[0], i), 3), *v = g.keys(PyList_GET_ITEM(a[1], i), 3);
        g.need(g.ok && k->size(0) >= n_src * g.c->nf && v->size(0) >= n_src * g.c->nf);
        if (!g.ok) return nullptr;
        pk[i] = ptr(*k);
        pv[i] = ptr(*v);
    }
    const int64_t shape[5] = {layers, nq, slots * g.c->nf, g.c->hkv, g.c->d};
    Out dk(a[4]), dv(a[5]);
    for (Out* o : {&dk, &dv}) {
        if (!o->given) o->made = at::empty(shape, on(*idx, g.c->dtype));
        else g.need(g.device(o->given, -1, g.c->dtype) && o->get().numel() == layers * nq * shape[2] * shape[3] * shape[4]);
        if (!g.ok) return nullptr;
    }
    void* s = stream();
    const rekv_status st = outside(rekv_gather_kv_layers, g.c->h, pk, pv, (int32_t)layers, (int32_t)n_src, static_cast<const int32_t*>(ptr(*idx)),
                                   (int32_t)nq, (int32_t)slots, ptr(dk.get()), ptr(dv.get()), s);
    return st ? raise_status(g.c, st) : pair(dk, dv);
}

// mode, pos_offset, src_rotated, src_pos_offset, base, layout: six arguments in a row
struct Rope {
    int32_t mode, rotated, layout;
    int64_t pos, src_pos;
    double base;
    Rope(Args& g, PyObject* const* a)
        : mode(g.word(a[0], "consecutive", "static")), rotated(g.flag(a[2])), layout(g.word(a[5], "half", "interleaved")),
          pos(g.i64(a[1])), src_pos(g.i64(a[3])), base(g.f64(a[4])) {}
};

METHOD(gather_kv_rope, 10) {     // src_k, src_v, idx, n_src_frames, then Rope's; device sources
    Args g(self);
    const Tensor *k = g.keys(a[0], 3), *v = g.keys(a[1], 3), *idx = g.device(a[2], 2, at::kInt);
    const int32_t n_src = g.frames(a[3], k, v);
    const Rope r(g, a + 4);
    if (!g.ok) return nullptr;
    const int64_t nq = idx->size(0), slots = idx->size(1);
    g.need(Args::fits(nq) && Args::fits(slots));
    if (!g.ok) return nullptr;
    Out dk(Py_None), dv(Py_None);
    dk.made = at::empty({nq, slots * g.c->nf, g.c->hkv, g.c->d}, on(*idx, g.c->dtype));
    dv.made = at::empty({nq, slots * g.c->nf, g.c->hkv, g.c->d}, on(*idx, g.c->dtype));
    void* s = stream();
    const rekv_status st = outside(rekv_gather_kv_rope, g.c->h, ptr(*k), ptr(*v), 0, n_src, static_cast<const int32_t*>(ptr(*idx)), (int32_t)nq,
                                   (int32_t)slots, ptr(dk.made), ptr(dv.made), r.base, r.layout, r.mode, r.pos, r.rotated, r.src_pos, s);
    return st ? raise_status(g.c, st) : pair(dk, dv);
}

// What the attention calls on an arena share.
struct InPlace {
    const Tensor *q, *k, *v, *idx, *kt, *vt;
    int32_t n_src = 0;
    int64_t nq = 0, n_new = 0;
    InPlace(Args& g, PyObject* q_, PyObject* k_, PyObject* v_, PyObject* idx_, PyObject* kt_, PyObject* vt_, PyObject* n_src_)
        : q(g.queries(q_, 4)), k(g.keys(k_, 3)), v(g.keys(v_, 3)), idx(g.device(idx_, 2, at::kInt)), kt(g.keys(kt_, 4)), vt(g.keys(vt_, 4)) {
        n_src = g.frames(n_src_, k, v);
        if (!g.ok) return;
        nq = q->size(0);
        n_new = q->size(1);
        g.need(idx->size(0) == nq && kt->size(0) == nq && vt->sizes() == kt->sizes() && Args::fits(nq) && Args::fits(n_new) &&
               Args::fits(idx->size(1)));
    }
};

METHOD(attention_indexed, 11) {  // q, k_src, v_src, idx, n_ret_frames, k_text, v_text, n_text_tokens, n_src_frames, out, n_sel
    Args g(self);
    const InPlace p(g, a[0], a[1], a[2], a[3], a[5], a[6], a[8]);
    const int32_t n_ret = g.i32(a[4]), n_text = g.i32(a[7]);
    const int32_t* n_sel = g.n_sel(a[10], p.nq);
    if (!g.ok) return nullptr;
    Out out(a[9]);
    if (!out.given) out.made = at::empty_like(*p.q);
    else g.need(g.queries(a[9], 4) && out.get().sizes() == p.q->sizes());
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(rekv_attention_indexed, g.c->h, ptr(*p.q), ptr(*p.k), ptr(*p.v), p.n_src,
                                   static_cast<const int32_t*>(ptr(*p.idx)), p.idx->size(1), n_ret, n_sel, ptr(*p.kt), ptr(*p.vt), p.kt->size(1),
                                   n_text, (int32_t)p.nq, (int32_t)p.n_new, ptr(out.get()), s);
    return st ? raise_status(g.c, st) : out.take();
}

METHOD(attention_indexed_rope, 17) {   // q, k_src, v_src, idx, k_text, v_text, n_text_tokens, n_src_frames, n_sel, then Rope's, k_pos, out
    Args g(self);
    const InPlace p(g, a[0], a[1], a[2], a[3], a[4], a[5], a[7]);
    const int32_t n_text = g.i32(a[6]);
    const int32_t* n_sel = g.n_sel(a[8], p.nq);
    const Rope r(g, a + 9);
    if (!g.ok) return nullptr;
    const int64_t n_ret = p.idx->size(1), shape[4] = {p.nq, n_ret * g.c->nf, g.c->hkv, g.c->d};
    Out k_pos(a[15]), out(a[16]);
    if (!k_pos.given) k_pos.made = at::empty(shape, on(*p.q, g.c->dtype));
    else g.need(g.keys(a[15], 4) && k_pos.get().sizes() == at::IntArrayRef(shape));
    if (!g.ok) return nullptr;
    if (!out.given) out.made = at::empty_like(*p.q);
    else g.need(g.queries(a[16], 4) && out.get().sizes() == p.q->sizes());
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(rekv_attention_indexed_rope, g.c->h, ptr(*p.q), ptr(*p.k), ptr(*p.v), p.n_src,
                                   static_cast<const int32_t*>(ptr(*p.idx)), n_ret, (int32_t)n_ret, n_sel, ptr(k_pos.get()), r.base, r.layout,
                                   r.mode, r.pos, r.rotated, r.src_pos, ptr(*p.kt), ptr(*p.vt), p.kt->size(1), n_text, (int32_t)p.nq,
                                   (int32_t)p.n_new, ptr(out.get()), s);
    return st ? raise_status(g.c, st) : pair(out, k_pos);
}

METHOD(qa_attention, 7) {        // q, k_ret, v_ret, k_self, v_self, out, n_sel
    Args g(self);
    const Tensor *q = g.queries(a[0], 4), *kr = g.keys(a[1], 4), *vr = g.keys(a[2], 4), *ks = g.keys(a[3], 4), *vs = g.keys(a[4], 4);
    if (!g.ok) return nullptr;
    const int64_t nq = q->size(0), nt = q->size(1), n_ret = kr->size(1);
    const int32_t* n_sel = g.n_sel(a[6], nq);
    g.need(kr->size(0) == nq && n_ret > 0 && vr->sizes() == kr->sizes() && ks->size(0) == nq && ks->size(1) == nt && vs->sizes() == ks->sizes() &&
           Args::fits(nq) && Args::fits(nt) && Args::fits(n_ret));
    if (!g.ok) return nullptr;
    Out out(a[5]);
    if (!out.given) out.made = at::empty_like(*q);
    else g.need(g.queries(a[5], 4) && out.get().sizes() == q->sizes());
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(rekv_qa_attention, g.c->h, ptr(*q), ptr(*kr), ptr(*vr), (int32_t)n_ret, n_sel, ptr(*ks), ptr(*vs), (int32_t)nq,
                                   (int32_t)nt, ptr(out.get()), s);
    return st ? raise_status(g.c, st) : out.take();
}

METHOD(decode_attention, 9) {    // q, k_ret, v_ret, k_text, v_text, n_text_tokens, out, n_sel, no_alloc
    Args g(self);
    const Tensor *q = g.queries(a[0], 4), *kr = g.keys(a[1], 4), *vr = g.keys(a[2], 4), *kt = g.keys(a[3], 4), *vt = g.keys(a[4], 4);
    const int32_t n_text = g.i32(a[5]);
    const bool no_alloc = g.flag(a[8]);
    if (!g.ok) return nullptr;
    const int64_t nq = q->size(0), n_new = q->size(1), n_ret = kr->size(1);
    const int32_t* n_sel = g.n_sel(a[7], nq);
    g.need(kr->size(0) == nq && n_ret > 0 && vr->sizes() == kr->sizes() && kt->size(0) == nq && vt->sizes() == kt->sizes() &&
           Args::fits(nq) && Args::fits(n_new) && Args::fits(n_ret));
    if (!g.ok) return nullptr;
    Out out(a[6]);
    if (!out.given) out.made = at::empty_like(*q);
    else g.need(g.queries(a[6], 4) && out.get().sizes() == q->sizes());
    if (!g.ok) return nullptr;
    void* s = stream();
    const rekv_status st = outside(no_alloc ? rekv_decode_attention_noalloc : rekv_decode_attention, g.c->h, ptr(*q), ptr(*kr), ptr(*vr),
                                   (int32_t)n_ret, n_sel, ptr(*kt), ptr(*vt), kt->size(1), n_text, (int32_t)nq, (int32_t)n_new, ptr(out.get()), s);
    return st ? raise_status(g.c, st) : out.take();
}

// The context is gone: every later call is the Python method's.
PyObject* close_context(PyObject* self, PyObject*) {
    reinterpret_cast<Context*>(self)->h = nullptr;
    Py_RETURN_NONE;
}

int init_context(PyObject* self, PyObject* args, PyObject*) {
    Context* c = reinterpret_cast<Context*>(self);
    unsigned long long h;
    long long hq, hkv, d, nf;
    int bf16;
    if (!PyArg_ParseTuple(args, "KLLLLi", &h, &hq, &hkv, &d, &nf, &bf16)) return -1;
    c->h = reinterpret_cast<rekv_ctx*>((uintptr_t)h);
    c->hq = hq;
    c->hkv = hkv;
    c->d = d;
    c->nf = nf;
    c->dtype = bf16 ? at::kBFloat16 : at::kFloat;
    return 0;
}

#define ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ENTRY(encode_chunk), ENTRY(frame_keys), ENTRY(retrieve_topk), ENTRY(retrieve_external), ENTRY(block_keys), ENTRY(expand_blocks),
    ENTRY(gather_kv), ENTRY(gather_kv_layers), ENTRY(gather_kv_rope), ENTRY(attention_indexed), ENTRY(attention_indexed_rope),
    ENTRY(qa_attention), ENTRY(decode_attention), {"close", close_context, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};

PyTypeObject context_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* set_raise(PyObject*, PyObject* fn) {
    Py_INCREF(fn);
    Py_XDECREF(g_raise);
    g_raise = fn;
    Py_RETURN_NONE;
}
PyMethodDef functions[] = {{"set_raise", set_raise, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, functions};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    context_type.tp_name = "paper_2503_00540_amd._binding.Context";
    context_type.tp_basicsize = sizeof(Context);
    context_type.tp_flags = Py_TPFLAGS_DEFAULT;
    context_type.tp_new = PyType_GenericNew;
    context_type.tp_init = init_context;
    context_type.tp_methods = methods;
    if (PyType_Ready(&context_type) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&context_type);
    if (PyModule_AddObject(m, "Context", reinterpret_cast<PyObject*>(&context_type)) < 0) return nullptr;
    return m;
}
