// Native half of the Python binding: takes the arguments of a call as they come (tensors, sizes),
// checks them, fills the descriptor and makes the one library call.
//
// What it replaces is host time: marshalling a call through ctypes took 9-11 us of interpreter work
// (a dozen checked pointers, a descriptor, a foreign call with seventeen arguments) around the
// 2.5-3 us of the launch itself, and kept the GPU waiting wherever a call's kernels run for less than
// that: small layers and small vocabularies altogether, and the ten-microsecond draft calls of one
// sequence.  Here the same work is 1-2 us.
//
// Every function returns None whenever something is not as it expects (a tensor on another device or
// of another type, a shape that does not fit, an error status), also where torch reports it by a C++
// exception: no memory for an output, a tensor without storage, no device to take a stream from.
// Nothing has been launched then, and the caller goes on with its own, slower path, which raises the
// exact error.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <cxxabi.h>
#include <dlfcn.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/radar.h"

namespace {

struct Library {
    decltype(&radar_tree_attention) tree_attention;
    decltype(&radar_draft_expand) draft_expand;
    decltype(&radar_draft_expand_policy) draft_expand_policy;
    decltype(&radar_draft_expand_cycle) draft_expand_cycle;
    decltype(&radar_draft_expand_batch) draft_expand_batch;
    decltype(&radar_draft_rerank) draft_rerank;
    decltype(&radar_draft_rerank_cycle) draft_rerank_cycle;
    decltype(&radar_draft_rerank_batch) draft_rerank_batch;
    decltype(&radar_verify_accept) verify_accept;
    decltype(&radar_verify_accept_q) verify_accept_q;
    decltype(&radar_accept_length_distribution) accept_length_distribution;
    decltype(&radar_policy_step) policy_step;
} lib;

// Reads a call's arguments in order; `ok` turns false at the first one that does not fit.
class Reader {
public:
    Reader(PyObject *const *args, Py_ssize_t n) : at_(args), end_(args + n) {}
    bool ok = true;

    // a tensor on the GPU, of this type and densely packed; null where None is allowed and given
    const at::Tensor *tensor(at::ScalarType type, bool dense = true, bool optional = false) {
        PyObject *o = next();
        if (o == nullptr || (o == Py_None && optional)) return nullptr;
        if (!THPVariable_Check(o)) return fail();
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || t.scalar_type() != type || (dense && !t.is_contiguous())) return fail();
        return &t;
    }
    const at::Tensor *f32(bool optional = false) { return tensor(at::kFloat, true, optional); }
    const at::Tensor *i32(bool optional = false) { return tensor(at::kInt, true, optional); }
    float *fp(bool optional = false) { return pointer<float>(f32(optional)); }
    int32_t *ip(bool optional = false) { return pointer<int32_t>(i32(optional)); }
    template <typename T>
    static T *pointer(const at::Tensor *t) { return t ? static_cast<T *>(t->data_ptr()) : nullptr; }

    // a workspace: any tensor, or None
    void workspace(void **p, size_t *bytes) {
        *p = nullptr; *bytes = 0;
        PyObject *o = next();
        if (!ok || o == Py_None) return;
        if (!THPVariable_Check(o)) { fail(); return; }
        const at::Tensor &t = THPVariable_Unpack(o);
        *p = t.data_ptr();
        *bytes = t.nbytes();
    }
    int32_t integer() {
        PyObject *o = next();
        if (o == nullptr) return 0;
        const long v = PyLong_AsLong(o);
        if ((v == -1 && PyErr_Occurred()) || v < INT32_MIN || v > INT32_MAX) { PyErr_Clear(); fail(); return 0; }
        return (int32_t)v;
    }
    float real() {
        PyObject *o = next();
        if (o == nullptr) return 0.f;
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); fail(); return 0.f; }
        return (float)v;
    }
    // address of a host struct the caller keeps (0: none)
    template <typename T>
    const T *address() {
        PyObject *o = next();
        if (o == nullptr) return nullptr;
        void *p = PyLong_AsVoidPtr(o);
        if (p == nullptr && PyErr_Occurred()) { PyErr_Clear(); fail(); }
        return static_cast<const T *>(p);
    }
    PyObject *peek() const { return at_ < end_ ? *at_ : nullptr; }
    void skip() { (void)next(); }
    std::nullptr_t fail() { ok = false; return nullptr; }

private:
    PyObject *next() {
        if (at_ == end_) { ok = false; return nullptr; }
        return *at_++;
    }
    PyObject *const *at_, *const *end_;
};

// the current stream of the current device, as the slower path passes it
void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// The library call itself, with the interpreter lock released (a full queue can hold a launch up).
// (The lock is taken back outside of any handler or destructor: a thread that the interpreter ends at
// shutdown is unwound from there.)
template <typename Fn, typename... A>
radar_status call(Fn fn, A... a) {
    PyThreadState *const held = PyEval_SaveThread();
    radar_status rc;
    try {
        rc = fn(a...);
    } catch (...) {
        rc = RADAR_HIP_ERROR;
    }
    PyEval_RestoreThread(held);
    return rc;
}

// An entry point as Python calls it: no C++ exception leaves it, one becomes None.
using Entry = PyObject *(PyObject *, PyObject *const *, Py_ssize_t);
template <Entry *entry>
PyObject *guarded(PyObject *self, PyObject *const *args, Py_ssize_t n) {
    try {
        return entry(self, args, n);
    } catch (abi::__forced_unwind &) {           // the thread is being ended: not an error, and not to be swallowed
        throw;
    } catch (...) {
        PyErr_Clear();                           // a tensor subclass may have raised in Python on the way
        Py_RETURN_NONE;
    }
}

PyObject *done(radar_status rc, PyObject *result = Py_True) {
    if (rc != RADAR_OK) Py_RETURN_NONE;
    Py_INCREF(result);
    return result;
}

// q, k_cache, v_cache, parents, ctx_lens, n_nodes, out (None: allocated here), lse_out, keys_per_split,
// softmax_scale, workspace -> out
PyObject *tree_attention(PyObject *, PyObject *const *args, Py_ssize_t n) {
    Reader r(args, n);
    const at::Tensor *q = r.tensor(at::kBFloat16, false), *k = r.tensor(at::kBFloat16, false), *v = r.tensor(at::kBFloat16, false);
    const int32_t *parents = r.ip(), *ctx = r.ip(), *nodes = r.ip(true);
    PyObject *out_obj = r.peek();
    const at::Tensor *out = r.tensor(at::kBFloat16, true, true);
    const at::Tensor *lse = r.tensor(at::kFloat, false, true);
    radar_attn_desc d{};
    d.keys_per_split = r.integer();
    d.softmax_scale = r.real();
    void *ws; size_t ws_bytes;
    r.workspace(&ws, &ws_bytes);
    if (!r.ok || q->dim() != 4 || k->dim() != 4 || q->stride(3) != 1 || k->stride(3) != 1 || v->strides() != k->strides()) Py_RETURN_NONE;
    d.B = (int32_t)q->size(0); d.T_max = (int32_t)q->size(1); d.Hq = (int32_t)q->size(2); d.D = (int32_t)q->size(3);
    d.Hkv = (int32_t)k->size(1); d.S_max = (int32_t)k->size(2);
    d.q_stride_b = q->stride(0); d.q_stride_t = q->stride(1); d.q_stride_h = q->stride(2);
    d.kv_stride_b = k->stride(0); d.kv_stride_h = k->stride(1); d.kv_stride_s = k->stride(2);
    at::Tensor fresh;
    if (out == nullptr) { fresh = at::empty(q->sizes(), q->options().memory_format(c10::nullopt)); out = &fresh; }
    const radar_status rc = call(lib.tree_attention, q->data_ptr(), k->data_ptr(), v->data_ptr(), parents, ctx, nodes, out->data_ptr(),
                                               Reader::pointer<float>(lse), &d, ws, ws_bytes, stream());
    if (rc != RADAR_OK) Py_RETURN_NONE;
    return fresh.defined() ? THPVariable_Wrap(std::move(fresh)) : done(rc, out_obj);
}

// the outputs every expansion call has, in the order of the C call
struct ExpandOutputs {
    int32_t *cand_tokens; float *cand_scores;
    int32_t *frontier_pool_idx, *frontier_tokens; float *frontier_scores, *frontier_conf;
    int32_t *pool_tokens; float *pool_scores; int32_t *pool_parents;
    explicit ExpandOutputs(Reader &r)
        : cand_tokens(r.ip()), cand_scores(r.fp()), frontier_pool_idx(r.ip()), frontier_tokens(r.ip()), frontier_scores(r.fp()),
          frontier_conf(r.fp()), pool_tokens(r.ip()), pool_scores(r.fp()), pool_parents(r.ip()) {}
};

// h, c, uniform (each may be None), then the five outputs; `per` sequences
bool read_policy(Reader &r, const radar_policy_params *pp, int64_t per, radar_policy_io *io) {
    const at::Tensor *h = r.f32(true), *c = r.f32(true), *u = r.f32(true);
    if (!r.ok || (h == nullptr) != (c == nullptr)) return false;
    if (h && (h->numel() != per * pp->H || c->numel() != per * pp->H)) return false;
    if (u && per > 1 && u->numel() != per) return false;
    io->h_in = Reader::pointer<float>(h); io->c_in = Reader::pointer<float>(c); io->uniform = Reader::pointer<float>(u);
    io->h_out = r.fp(); io->c_out = r.fp(); io->logits = r.fp(); io->probs = r.fp(); io->action = r.ip();
    return r.ok;
}

// B (0: a call without a batch dimension), logits, parent_scores, parent_pool_idx, k, pool_count, pool_capacity,
// outputs, states (None: none), params address (0: none) [, h, c, uniform, h_out, c_out, logits, probs, action],
// workspace
PyObject *draft_expand(PyObject *, PyObject *const *args, Py_ssize_t n) {
    Reader r(args, n);
    const int32_t B = r.integer();
    const at::Tensor *x = r.f32();
    const float *ps = r.fp();
    const int32_t *pi = r.ip();
    radar_expand_desc d{};
    d.k = r.integer(); d.pool_count = r.integer(); d.pool_capacity = r.integer();
    const ExpandOutputs o(r);
    radar_cycle_state *states = reinterpret_cast<radar_cycle_state *>(r.ip(true));
    const radar_policy_params *pp = r.address<radar_policy_params>();
    radar_policy_io io{};
    if (!r.ok || (pp && !read_policy(r, pp, B > 0 ? B : 1, &io))) Py_RETURN_NONE;
    void *ws; size_t ws_bytes;
    r.workspace(&ws, &ws_bytes);
    if (!r.ok || x->dim() != (B > 0 ? 3 : 2)) Py_RETURN_NONE;
    d.F = (int32_t)x->size(-2); d.V = (int32_t)x->size(-1);
    const float *lg = Reader::pointer<float>(x);
    const radar_policy_io *iop = pp ? &io : nullptr;
    radar_status rc;
    if (B > 0)
        rc = call(lib.draft_expand_batch, lg, ps, pi, o.cand_tokens, o.cand_scores, o.frontier_pool_idx, o.frontier_tokens, o.frontier_scores,
                                    o.frontier_conf, o.pool_tokens, o.pool_scores, o.pool_parents, &d, B, pp, iop, states, ws, ws_bytes, stream());
    else if (states)
        rc = call(lib.draft_expand_cycle, lg, ps, pi, o.cand_tokens, o.cand_scores, o.frontier_pool_idx, o.frontier_tokens, o.frontier_scores,
                                    o.frontier_conf, o.pool_tokens, o.pool_scores, o.pool_parents, &d, pp, iop, states, ws, ws_bytes, stream());
    else if (pp)
        rc = call(lib.draft_expand_policy, lg, ps, pi, o.cand_tokens, o.cand_scores, o.frontier_pool_idx, o.frontier_tokens, o.frontier_scores,
                                     o.frontier_conf, o.pool_tokens, o.pool_scores, o.pool_parents, &d, pp, iop, ws, ws_bytes, stream());
    else
        rc = call(lib.draft_expand, lg, ps, pi, o.cand_tokens, o.cand_scores, o.frontier_pool_idx, o.frontier_tokens, o.frontier_scores,
                              o.frontier_conf, o.pool_tokens, o.pool_scores, o.pool_parents, &d, ws, ws_bytes, stream());
    return done(rc);
}

// B (0: no batch dimension), pool tokens, scores, parents, states (None: none), pool_count, pool_capacity, N,
// root (an integer; with B > 0 a tensor), tree tokens, parents, scores, depth, pool_idx, n_nodes
PyObject *draft_rerank(PyObject *, PyObject *const *args, Py_ssize_t n) {
    Reader r(args, n);
    const int32_t B = r.integer();
    const int32_t *pt = r.ip(); const float *psc = r.fp(); const int32_t *pp = r.ip();
    const radar_cycle_state *st = reinterpret_cast<const radar_cycle_state *>(r.ip(true));
    const int32_t count = r.integer(), cap = r.integer(), N = r.integer();
    const int32_t *roots = B > 0 ? r.ip() : nullptr;
    const int32_t root = B > 0 ? 0 : r.integer();
    int32_t *tt = r.ip(), *tp = r.ip(); float *ts = r.fp(); int32_t *td = r.ip(), *ti = r.ip(), *nn = r.ip();
    if (!r.ok) Py_RETURN_NONE;
    if (B > 0) return done(call(lib.draft_rerank_batch, pt, psc, pp, st, count, cap, B, N, roots, tt, tp, ts, td, ti, nn, nullptr, 0, stream()));
    if (st) return done(call(lib.draft_rerank_cycle, pt, psc, pp, st, count, N, root, tt, tp, ts, td, ti, nn, nullptr, 0, stream()));
    return done(call(lib.draft_rerank, pt, psc, pp, count, N, root, tt, tp, ts, td, ti, nn, nullptr, 0, stream()));
}

// Outputs of a verification call: the caller's, or fresh ones cut from one allocation.
struct AcceptOutputs {
    at::Tensor own[3];
    int32_t *len = nullptr, *path = nullptr, *bonus = nullptr;
    bool given = false;
    void read(Reader &r) {                       // accept_len, accept_path, bonus_token; three None: allocate
        const at::Tensor *l = r.i32(true), *p = r.i32(true), *b = r.i32(true);
        given = l && p && b;
        if (!given && (l || p || b)) r.fail();
        if (given) { len = Reader::pointer<int32_t>(l); path = Reader::pointer<int32_t>(p); bonus = Reader::pointer<int32_t>(b); }
    }
    void allocate(const at::Tensor &like, int64_t B, int64_t D1) {
        if (given) return;
        const auto opt = like.options().dtype(at::kInt);
        own[0] = at::empty({B}, opt); own[1] = at::empty({B, D1}, opt); own[2] = at::empty({B}, opt);
        len = Reader::pointer<int32_t>(&own[0]); path = Reader::pointer<int32_t>(&own[1]); bonus = Reader::pointer<int32_t>(&own[2]);
    }
    PyObject *result(radar_status rc) {          // True where the caller keeps its own outputs, else the three tensors
        if (rc != RADAR_OK) Py_RETURN_NONE;
        if (given) Py_RETURN_TRUE;
        PyObject *t = PyTuple_New(3);
        for (int i = 0; t && i < 3; ++i) {
            PyObject *o = THPVariable_Wrap(std::move(own[i]));
            if (o == nullptr) { Py_DECREF(t); return nullptr; }
            PyTuple_SET_ITEM(t, i, o);
        }
        return t;
    }
};

// target_logits, draft_tokens, parents, n_nodes, uniforms, mode, temperature, D_max, outputs, workspace
PyObject *verify_accept(PyObject *, PyObject *const *args, Py_ssize_t n) {
    Reader r(args, n);
    const at::Tensor *x = r.f32();
    const int32_t *tok = r.ip(), *par = r.ip(), *nn = r.ip(true);
    const float *uni = r.fp(true);
    radar_accept_desc d{};
    d.mode = r.integer(); d.temperature = r.real(); d.D_max = r.integer();
    AcceptOutputs o;
    o.read(r);
    void *ws; size_t ws_bytes;
    r.workspace(&ws, &ws_bytes);
    if (!r.ok || x->dim() != 3 || d.D_max < 0) Py_RETURN_NONE;
    d.B = (int32_t)x->size(0); d.T_max = (int32_t)x->size(1); d.V = (int32_t)x->size(2);
    o.allocate(*x, d.B, (int64_t)d.D_max + 1);
    return o.result(call(lib.verify_accept, Reader::pointer<float>(x), tok, par, nn, uni, o.len, o.path, o.bonus, &d, ws, ws_bytes, stream()));
}

// target_logits, draft_logits, q_rows, draft_tokens, parents, n_nodes, uniforms, temperature, draft_temperature, D_max,
// walk_spin_limit, outputs, workspace
PyObject *verify_accept_q(PyObject *, PyObject *const *args, Py_ssize_t n) {
    Reader r(args, n);
    const at::Tensor *x = r.f32(), *y = r.f32();
    const int32_t *qr = r.ip(true), *tok = r.ip(), *par = r.ip(), *nn = r.ip(true);
    const at::Tensor *uni = r.f32();
    radar_accept_q_desc d{};
    d.temperature = r.real(); d.draft_temperature = r.real(); d.D_max = r.integer(); d.walk_spin_limit = r.integer();
    AcceptOutputs o;
    o.read(r);
    void *ws; size_t ws_bytes;
    r.workspace(&ws, &ws_bytes);
    if (!r.ok || x->dim() != 3 || y->dim() != 3 || d.D_max < 0) Py_RETURN_NONE;
    d.B = (int32_t)x->size(0); d.T_max = (int32_t)x->size(1); d.V = (int32_t)x->size(2); d.Tq = (int32_t)y->size(1);
    if (y->size(0) != d.B || y->size(2) != d.V || uni->dim() != 2 || uni->size(0) != d.B || uni->size(1) != d.T_max + 1) Py_RETURN_NONE;
    o.allocate(*x, d.B, (int64_t)d.D_max + 1);
    return o.result(call(lib.verify_accept_q, Reader::pointer<float>(x), Reader::pointer<float>(y), qr, tok, par, nn, Reader::pointer<float>(uni),
                                        o.len, o.path, o.bonus, &d, ws, ws_bytes, stream()));
}

// target_logits, draft_tokens, parents, n_nodes, temperature, D_max, dist (None: allocated here), workspace -> dist
PyObject *accept_length_distribution(PyObject *, PyObject *const *args, Py_ssize_t n) {
    Reader r(args, n);
    const at::Tensor *x = r.f32();
    const int32_t *tok = r.ip(), *par = r.ip(), *nn = r.ip(true);
    radar_accept_desc d{};
    d.mode = RADAR_ACCEPT_SAMPLE; d.temperature = r.real(); d.D_max = r.integer();
    PyObject *out_obj = r.peek();
    const at::Tensor *out = r.tensor(at::kDouble, true, true);
    void *ws; size_t ws_bytes;
    r.workspace(&ws, &ws_bytes);
    if (!r.ok || x->dim() != 3 || d.D_max < 0) Py_RETURN_NONE;
    d.B = (int32_t)x->size(0); d.T_max = (int32_t)x->size(1); d.V = (int32_t)x->size(2);
    at::Tensor fresh;
    if (out == nullptr) { fresh = at::empty({d.B, (int64_t)d.D_max + 1}, x->options().dtype(at::kDouble)); out = &fresh; }
    const radar_status rc = call(lib.accept_length_distribution, Reader::pointer<float>(x), tok, par, nn, Reader::pointer<double>(out), &d, ws, ws_bytes, stream());
    if (rc != RADAR_OK) Py_RETURN_NONE;
    return fresh.defined() ? THPVariable_Wrap(std::move(fresh)) : done(rc, out_obj);
}

// conf, params address, h, c, uniforms, h_out, c_out, logits, probs, action
PyObject *policy_step(PyObject *, PyObject *const *args, Py_ssize_t n) {
    Reader r(args, n);
    const at::Tensor *conf = r.f32();
    const radar_policy_params *pp = r.address<radar_policy_params>();
    if (!r.ok || !pp || conf->dim() != 2 || conf->size(1) != pp->k) Py_RETURN_NONE;
    const int64_t B = conf->size(0);
    const at::Tensor *h = r.f32(true), *c = r.f32(true), *u = r.f32(true);
    if (!r.ok || (h == nullptr) != (c == nullptr)) Py_RETURN_NONE;
    for (const at::Tensor *t : {h, c})
        if (t && (t->dim() != 2 || t->size(0) != B || t->size(1) != pp->H)) Py_RETURN_NONE;
    if (u && (u->dim() != 1 || u->size(0) != B)) Py_RETURN_NONE;
    float *ho = r.fp(), *co = r.fp(), *lg = r.fp(), *pr = r.fp();
    int32_t *act = r.ip();
    if (!r.ok) Py_RETURN_NONE;
    return done(call(lib.policy_step, Reader::pointer<float>(conf), Reader::pointer<float>(h), Reader::pointer<float>(c), pp,
                                Reader::pointer<float>(u), ho, co, lg, pr, act, (int32_t)B, stream()));
}

// the library's path: looks its entry points up (it is the copy that ctypes has loaded already)
PyObject *bind(PyObject *, PyObject *path) {
    const char *p = PyUnicode_AsUTF8(path);
    if (p == nullptr) return nullptr;
    void *so = dlopen(p, RTLD_NOW | RTLD_LOCAL);
    if (so == nullptr) { PyErr_SetString(PyExc_RuntimeError, dlerror()); return nullptr; }
    bool all = true;
    auto find = [&](auto &fn, const char *name) {
        fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>(dlsym(so, name));
        all = all && fn != nullptr;
    };
    find(lib.tree_attention, "radar_tree_attention");
    find(lib.draft_expand, "radar_draft_expand");
    find(lib.draft_expand_policy, "radar_draft_expand_policy");
    find(lib.draft_expand_cycle, "radar_draft_expand_cycle");
    find(lib.draft_expand_batch, "radar_draft_expand_batch");
    find(lib.draft_rerank, "radar_draft_rerank");
    find(lib.draft_rerank_cycle, "radar_draft_rerank_cycle");
    find(lib.draft_rerank_batch, "radar_draft_rerank_batch");
    find(lib.verify_accept, "radar_verify_accept");
    find(lib.verify_accept_q, "radar_verify_accept_q");
    find(lib.accept_length_distribution, "radar_accept_length_distribution");
    find(lib.policy_step, "radar_policy_step");
    if (!all) { PyErr_Format(PyExc_RuntimeError, "%s lacks an entry point", p); return nullptr; }
    Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    FAST(tree_attention), FAST(draft_expand), FAST(draft_rerank), FAST(verify_accept), FAST(verify_accept_q),
    FAST(accept_length_distribution), FAST(policy_step),
    {"bind", bind, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "argument marshalling of the hot calls", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
