// The calls of binding.py without the Python work per call: tensors are checked and turned into pointers here, the
// current stream is asked for here, and the C ABI is entered through the function table that binding.py hands over
// (so that SPECPV_LIB keeps choosing the library).  Each function takes the arguments of the Python call of its name
// and returns its status, or None where an argument is not what the call takes: binding.py then goes through its own
// checks, which say what is wrong.
// What it is for: a partial step is two launches of 2.4 us each on the host; the Python checks, the ctypes conversion
// and the lookup of the stream took another 6 us per call, and 140 us for the commit of 32 layers.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <initializer_list>
#include <memory>
#include <vector>

#include "specpv.h"

namespace {

enum Fn { kSummarize, kSelect, kPartial, kPartialStatic, kRefresh, kGather, kCommit, kCommitLayers, kFns };
void *g_fn[kFns];
PyObject *s_c, *s_q, *s_kd;

template <typename F> F fn(Fn i) { return (F)g_fn[i]; }

// The C descriptor behind the attribute `c` of a KV, Tree or SelectCfg object (a ctypes structure).
template <typename S> class Desc {
public:
    Desc() = default;
    explicit Desc(PyObject *o) { open(o); }
    void open(PyObject *o)   // once
    {
        PyObject *c = PyObject_GetAttr(o, s_c);
        if (!c || PyObject_GetBuffer(c, &view_, PyBUF_SIMPLE) != 0) PyErr_Clear();
        else if ((size_t)view_.len == sizeof(S)) p_ = (const S *)view_.buf;
        Py_XDECREF(c);
    }
    ~Desc()
    {
        if (view_.obj) PyBuffer_Release(&view_);
    }
    Desc(const Desc &) = delete;
    Desc &operator=(const Desc &) = delete;
    explicit operator bool() const { return p_ != nullptr; }
    const S *operator->() const { return p_; }
    const S *get() const { return p_; }

private:
    Py_buffer view_ = {};
    const S *p_ = nullptr;
};

at::ScalarType scalar(const specpv_kv *kv) { return kv->dtype == SPECPV_BF16 ? at::kBFloat16 : at::kFloat; }

// A contiguous GPU tensor of this type and shape.
bool tensor(PyObject *o, at::ScalarType dt, std::initializer_list<int64_t> shape, void **out)
{
    if (!THPVariable_Check(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != dt || !t.is_contiguous() || t.dim() != (int64_t)shape.size()) return false;
    int64_t d = 0;
    for (int64_t x : shape)
        if (t.size(d++) != x) return false;
    *out = t.data_ptr();
    return true;
}
bool tensor_or_none(PyObject *o, at::ScalarType dt, std::initializer_list<int64_t> shape, void **out)
{
    *out = nullptr;
    return o == Py_None || tensor(o, dt, shape, out);
}
bool workspace(PyObject *o, void **out, size_t *bytes)
{
    *out = nullptr;
    *bytes = 0;
    if (o == Py_None) return true;
    if (!THPVariable_Check(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) return false;
    *out = t.data_ptr();
    *bytes = t.nbytes();
    return true;
}
// The last extent of a rank-3 tensor (the entries of a list row).
bool last_extent(PyObject *o, int64_t *n)
{
    if (!THPVariable_Check(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (t.dim() != 3) return false;
    *n = t.size(2);
    return true;
}
bool integer(PyObject *o, int32_t *v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    if (over || x < INT32_MIN || x > INT32_MAX) return false;
    *v = (int32_t)x;
    return true;
}

// A reference that is given back, also where what follows throws.
struct Ref {
    PyObject *o;
    explicit Ref(PyObject *p) : o(p) {}
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};
// kv and tree belong together (binding.py: _match)
bool match(const Desc<specpv_kv> &kv, PyObject *tree_obj, const Desc<specpv_tree> &tree)
{
    if (!kv || !tree) return false;
    const Ref q(PyObject_GetAttr(tree_obj, s_q)), kd(PyObject_GetAttr(tree_obj, s_kd));
    void *p = nullptr;
    bool ok = q.o && kd.o && tensor(q.o, scalar(kv.get()), {kv->batch, tree->M - tree->n_key_only, tree->n_q_heads, kv->head_dim}, &p) && p == tree->q;
    if (ok && kd.o != Py_None) ok = tensor(kd.o, scalar(kv.get()), {kv->batch, tree->M, kv->n_kv_heads, kv->head_dim}, &p) && p == tree->kd;
    if (PyErr_Occurred()) PyErr_Clear();
    return ok;
}
bool lists(const specpv_kv *kv, PyObject *idx, PyObject *cnt, int64_t n_sel, void **pi, void **pc)
{
    return tensor(idx, at::kInt, {kv->batch, kv->n_kv_heads, n_sel}, pi) && tensor(cnt, at::kInt, {kv->batch, kv->n_kv_heads}, pc);
}
bool summaries(const specpv_kv *kv, PyObject *kmax, PyObject *kmin, void **px, void **pn)
{
    return tensor(kmax, scalar(kv), {kv->batch, kv->n_kv_heads, kv->max_blocks, kv->head_dim}, px) &&
           tensor(kmin, scalar(kv), {kv->batch, kv->n_kv_heads, kv->max_blocks, kv->head_dim}, pn);
}
int64_t row_entries(const specpv_select_cfg *c) { return (int64_t)c->n_sink_blocks + c->k_blocks + c->n_recent_blocks + c->n_extra_slots; }

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// Enters the library without the interpreter's lock (as ctypes does).  The C ABI throws nothing.
template <typename F> PyObject *enter(F f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// What stands in the method table.  torch reports by C++ exceptions what a tensor cannot give (no storage under vmap or
// while tracing, no GPU for a stream), and none may leave through the interpreter's frames: the call then goes to
// binding.py like any other that is not taken here, and asking for the same thing there raises the Python error.
typedef PyObject *(*Method)(PyObject *, PyObject *const *, Py_ssize_t);
template <Method M> PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    try {
        return M(self, a, n);
    } catch (const std::exception &) {   // (not the unwinding of a thread that ends while the interpreter does)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

#define SPECPV_ARGS(N) \
    if (n != (N)) Py_RETURN_NONE

PyObject *summarize(PyObject *, PyObject *const *a, Py_ssize_t n)   // kv, blk_begin, blk_end, kmax, kmin
{
    SPECPV_ARGS(5);
    Desc<specpv_kv> kv(a[0]);
    int32_t lo, hi;
    void *kx, *kn;
    if (!kv || !integer(a[1], &lo) || !integer(a[2], &hi) || !summaries(kv.get(), a[3], a[4], &kx, &kn)) Py_RETURN_NONE;
    void *st = stream();
    return enter([&] { return fn<decltype(&specpv_block_summarize)>(kSummarize)(kv.get(), lo, hi, kx, kn, st); });
}

PyObject *select(PyObject *, PyObject *const *a, Py_ssize_t n)   // kv, tree, kmax, kmin, cfg, sel_idx, sel_count, scores, workspace
{
    SPECPV_ARGS(9);
    Desc<specpv_kv> kv(a[0]);
    Desc<specpv_tree> tree(a[1]);
    Desc<specpv_select_cfg> cfg(a[4]);
    void *kx, *kn, *si, *sc, *so, *ws;
    size_t wb;
    if (!cfg || !match(kv, a[1], tree) || !summaries(kv.get(), a[2], a[3], &kx, &kn) || !lists(kv.get(), a[5], a[6], row_entries(cfg.get()), &si, &sc) ||
        !tensor_or_none(a[7], at::kFloat, {kv->batch, kv->n_kv_heads, kv->max_blocks}, &so) || !workspace(a[8], &ws, &wb))
        Py_RETURN_NONE;
    void *st = stream();
    return enter([&] {
        return fn<decltype(&specpv_select_blocks)>(kSelect)(kv.get(), tree.get(), kx, kn, cfg.get(), (int32_t *)si, (int32_t *)sc, (float *)so, ws, wb, st);
    });
}

PyObject *partial_any(PyObject *const *a, bool own_scratch)   // kv, tree, sel_idx, sel_count, out, lse[, workspace]
{
    Desc<specpv_kv> kv(a[0]);
    Desc<specpv_tree> tree(a[1]);
    if (!match(kv, a[1], tree)) Py_RETURN_NONE;
    const int64_t Mq = tree->M - tree->n_key_only;
    void *si = nullptr, *sc = nullptr, *out, *lse, *ws = nullptr;
    size_t wb = 0;
    int64_t n_sel = 0;
    if (a[2] != Py_None && (!last_extent(a[2], &n_sel) || !lists(kv.get(), a[2], a[3], n_sel, &si, &sc))) Py_RETURN_NONE;
    if (a[2] == Py_None && a[3] != Py_None) Py_RETURN_NONE;
    if (!tensor(a[4], scalar(kv.get()), {kv->batch, Mq, tree->n_q_heads, kv->head_dim}, &out) ||
        !tensor_or_none(a[5], at::kFloat, {kv->batch, Mq, tree->n_q_heads}, &lse) || (!own_scratch && !workspace(a[6], &ws, &wb)) || n_sel > INT32_MAX)
        Py_RETURN_NONE;
    void *st = stream();
    return enter([&] {
        if (own_scratch)
            return fn<decltype(&specpv_partial_verify_attn_static)>(kPartialStatic)(kv.get(), tree.get(), (int32_t *)si, (int32_t *)sc, (int32_t)n_sel, out,
                                                                                    (float *)lse, st);
        return fn<decltype(&specpv_partial_verify_attn)>(kPartial)(kv.get(), tree.get(), (int32_t *)si, (int32_t *)sc, (int32_t)n_sel, out, (float *)lse, ws, wb, st);
    });
}
PyObject *partial(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    SPECPV_ARGS(7);
    return partial_any(a, false);
}
PyObject *partial_static(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    SPECPV_ARGS(6);
    return partial_any(a, true);
}

PyObject *refresh(PyObject *, PyObject *const *a, Py_ssize_t n)
{   // kv, tree, kmax, kmin, stale_blk_begin, cfg, out, lse, sel_idx, sel_count, scores, workspace
    SPECPV_ARGS(12);
    Desc<specpv_kv> kv(a[0]);
    Desc<specpv_tree> tree(a[1]);
    Desc<specpv_select_cfg> cfg(a[5]);
    if (!cfg || !match(kv, a[1], tree)) Py_RETURN_NONE;
    const int64_t Mq = tree->M - tree->n_key_only;
    int32_t stale;
    void *kx, *kn, *out, *lse, *si, *sc, *so, *ws;
    size_t wb;
    if (!summaries(kv.get(), a[2], a[3], &kx, &kn) || !integer(a[4], &stale) || !tensor(a[6], scalar(kv.get()), {kv->batch, Mq, tree->n_q_heads, kv->head_dim}, &out) ||
        !tensor_or_none(a[7], at::kFloat, {kv->batch, Mq, tree->n_q_heads}, &lse) || !lists(kv.get(), a[8], a[9], row_entries(cfg.get()), &si, &sc) ||
        !tensor_or_none(a[10], at::kFloat, {kv->batch, kv->n_kv_heads, kv->max_blocks}, &so) || !workspace(a[11], &ws, &wb))
        Py_RETURN_NONE;
    void *st = stream();
    return enter([&] {
        return fn<decltype(&specpv_full_verify_refresh)>(kRefresh)(kv.get(), tree.get(), kx, kn, stale, cfg.get(), out, (float *)lse, (int32_t *)si, (int32_t *)sc,
                                                                   (float *)so, ws, wb, st);
    });
}

PyObject *gather(PyObject *, PyObject *const *a, Py_ssize_t n)   // kv, sel_idx, sel_count, out_k, out_v, out_len
{
    SPECPV_ARGS(6);
    Desc<specpv_kv> kv(a[0]);
    int64_t n_sel = 0;
    void *si, *sc, *ok, *ov, *ol;
    if (!kv || !last_extent(a[1], &n_sel) || n_sel > INT32_MAX || !lists(kv.get(), a[1], a[2], n_sel, &si, &sc)) Py_RETURN_NONE;
    const int64_t rows = n_sel * kv->block_size;
    if (!tensor(a[3], scalar(kv.get()), {kv->batch, kv->n_kv_heads, rows, kv->head_dim}, &ok) ||
        !tensor(a[4], scalar(kv.get()), {kv->batch, kv->n_kv_heads, rows, kv->head_dim}, &ov))
        Py_RETURN_NONE;
    ol = nullptr;
    if (a[5] != Py_None) {   // (its extent is the caller's affair, as in binding.py)
        if (!THPVariable_Check(a[5])) Py_RETURN_NONE;
        const at::Tensor &t = THPVariable_Unpack(a[5]);
        if (!t.is_cuda() || t.scalar_type() != at::kInt || !t.is_contiguous()) Py_RETURN_NONE;
        ol = t.data_ptr();
    }
    void *st = stream();
    return enter([&] {
        return fn<decltype(&specpv_gather_blocks)>(kGather)(kv.get(), (int32_t *)si, (int32_t *)sc, (int32_t)n_sel, ok, ov, (int32_t *)ol, st);
    });
}

// One list (or tuple) of a per-layer argument.
struct Items {
    PyObject *seq = nullptr;
    explicit Items(PyObject *o)
    {
        if (PyList_CheckExact(o) || PyTuple_CheckExact(o)) seq = o;
    }
    Py_ssize_t size() const { return seq ? PySequence_Fast_GET_SIZE(seq) : -1; }
    PyObject *operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(seq, i); }
};

PyObject *commit_layers(PyObject *, PyObject *const *a, Py_ssize_t n)
{   // kvs, buf_ks, buf_vs, pending_cap, M_tree, n_pending, accepted, n_accepted, mode, kmaxs, kmins, workspace, sel_idxs, sel_counts, dropped
    SPECPV_ARGS(15);
    const Items kvs(a[0]), bks(a[1]), bvs(a[2]);
    const Py_ssize_t nl = kvs.size();
    int32_t cap, mt, mode;
    if (nl < 1 || nl > SPECPV_MAX_LAYERS || bks.size() != nl || bvs.size() != nl || !integer(a[3], &cap) || !integer(a[4], &mt) || !integer(a[8], &mode))
        Py_RETURN_NONE;
    const bool sums = a[9] != Py_None, with_lists = a[12] != Py_None;
    if (sums != (a[10] != Py_None) || with_lists != (a[13] != Py_None)) Py_RETURN_NONE;
    const Items kxs(a[9]), kns(a[10]), sis(a[12]), scs(a[13]);
    if (sums && (kxs.size() != nl || kns.size() != nl)) Py_RETURN_NONE;
    if (with_lists && (sis.size() != nl || scs.size() != nl)) Py_RETURN_NONE;
    const std::unique_ptr<Desc<specpv_kv>[]> d(new Desc<specpv_kv>[nl]);
    const specpv_kv *kv[SPECPV_MAX_LAYERS];
    void *bk[SPECPV_MAX_LAYERS], *bv[SPECPV_MAX_LAYERS], *kx[SPECPV_MAX_LAYERS], *kn[SPECPV_MAX_LAYERS];
    specpv_lists ls[SPECPV_MAX_LAYERS];
    for (Py_ssize_t l = 0; l < nl; ++l) {
        d[l].open(kvs[l]);
        if (!d[l]) Py_RETURN_NONE;
        kv[l] = d[l].get();
        const specpv_kv *k0 = kv[0];
        if (!tensor(bks[l], scalar(k0), {k0->batch, (int64_t)cap + mt, k0->n_kv_heads, k0->head_dim}, &bk[l]) ||
            !tensor(bvs[l], scalar(k0), {k0->batch, (int64_t)cap + mt, k0->n_kv_heads, k0->head_dim}, &bv[l]))
            Py_RETURN_NONE;
        if (sums && !summaries(k0, kxs[l], kns[l], &kx[l], &kn[l])) Py_RETURN_NONE;
        if (with_lists) {
            int64_t n_sel;
            void *pi, *pc;
            if (!last_extent(sis[l], &n_sel) || n_sel > INT32_MAX || !lists(k0, sis[l], scs[l], n_sel, &pi, &pc)) Py_RETURN_NONE;
            ls[l] = specpv_lists{(int32_t *)pi, (int32_t *)pc, (int32_t)n_sel};
        }
    }
    const specpv_kv *k0 = kv[0];
    if (!THPVariable_Check(a[6])) Py_RETURN_NONE;
    const at::Tensor &acc = THPVariable_Unpack(a[6]);
    if (acc.dim() != 2) Py_RETURN_NONE;
    const int64_t max_accept = acc.size(1);
    void *np_, *ac, *na, *dr, *ws;
    size_t wb;
    if (!tensor(a[5], at::kInt, {k0->batch}, &np_) || !tensor(a[6], at::kInt, {k0->batch, max_accept}, &ac) || !tensor(a[7], at::kInt, {k0->batch}, &na) ||
        max_accept > INT32_MAX || !workspace(a[11], &ws, &wb) || !tensor_or_none(a[14], at::kInt, {k0->batch, 2}, &dr))
        Py_RETURN_NONE;
    void *st = stream();
    return enter([&] {
        return fn<decltype(&specpv_commit_accepted_layers)>(kCommitLayers)(
            kv, bk, bv, (int32_t)nl, cap, mt, (int32_t *)np_, (int32_t *)ac, (int32_t *)na, (int32_t)max_accept, (specpv_mode)mode,
            sums ? kx : nullptr, sums ? kn : nullptr, with_lists ? ls : nullptr, (int32_t *)dr, ws, wb, st);
    });
}

PyObject *commit(PyObject *, PyObject *const *a, Py_ssize_t n)
{   // kv, buf_k, buf_v, pending_cap, M_tree, n_pending, accepted, n_accepted, mode, kmax, kmin, workspace, sel_idx, sel_count, dropped
    SPECPV_ARGS(15);
    Desc<specpv_kv> kv(a[0]);
    int32_t cap, mt, mode;
    if (!kv || !integer(a[3], &cap) || !integer(a[4], &mt) || !integer(a[8], &mode) || !THPVariable_Check(a[6])) Py_RETURN_NONE;
    const at::Tensor &acc = THPVariable_Unpack(a[6]);
    if (acc.dim() != 2) Py_RETURN_NONE;
    const int64_t max_accept = acc.size(1);
    const at::ScalarType dt = scalar(kv.get());
    const int64_t nb = kv->max_blocks;
    void *bk, *bv, *kx, *kn, *np_, *ac, *na, *dr, *ws, *pi = nullptr, *pc = nullptr;
    size_t wb;
    int64_t n_sel = 0;
    if (!tensor(a[1], dt, {kv->batch, (int64_t)cap + mt, kv->n_kv_heads, kv->head_dim}, &bk) ||
        !tensor(a[2], dt, {kv->batch, (int64_t)cap + mt, kv->n_kv_heads, kv->head_dim}, &bv) || !tensor(a[5], at::kInt, {kv->batch}, &np_) ||
        !tensor(a[6], at::kInt, {kv->batch, max_accept}, &ac) || max_accept > INT32_MAX || !tensor(a[7], at::kInt, {kv->batch}, &na) ||
        !tensor_or_none(a[9], dt, {kv->batch, kv->n_kv_heads, nb, kv->head_dim}, &kx) ||
        !tensor_or_none(a[10], dt, {kv->batch, kv->n_kv_heads, nb, kv->head_dim}, &kn) || !workspace(a[11], &ws, &wb) ||
        !tensor_or_none(a[14], at::kInt, {kv->batch, 2}, &dr))
        Py_RETURN_NONE;
    if (a[12] != Py_None && (!last_extent(a[12], &n_sel) || n_sel > INT32_MAX || !lists(kv.get(), a[12], a[13], n_sel, &pi, &pc))) Py_RETURN_NONE;
    const specpv_lists ls{(int32_t *)pi, (int32_t *)pc, (int32_t)n_sel};
    void *st = stream();
    return enter([&] {
        return fn<decltype(&specpv_commit_accepted)>(kCommit)(kv.get(), bk, bv, cap, mt, (int32_t *)np_, (int32_t *)ac, (int32_t *)na, (int32_t)max_accept,
                                                              (specpv_mode)mode, kx, kn, pi ? &ls : nullptr, (int32_t *)dr, ws, wb, st);
    });
}

PyObject *set_table(PyObject *, PyObject *const *a, Py_ssize_t n)   // the addresses of the library's functions, in the order of Fn
{
    if (n != kFns) {
        PyErr_SetString(PyExc_TypeError, "one address per function");
        return nullptr;
    }
    for (int i = 0; i < kFns; ++i) {
        void *p = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
        g_fn[i] = p;
    }
    Py_RETURN_NONE;
}

#define SPECPV_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))guarded<NAME>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SPECPV_METHOD(set_table), SPECPV_METHOD(summarize), SPECPV_METHOD(select),        SPECPV_METHOD(partial), SPECPV_METHOD(partial_static),
                         SPECPV_METHOD(refresh),   SPECPV_METHOD(gather),    SPECPV_METHOD(commit_layers), SPECPV_METHOD(commit),  {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "The calls of binding.py without the Python work per call.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    s_c = PyUnicode_InternFromString("c");
    s_q = PyUnicode_InternFromString("q");
    s_kd = PyUnicode_InternFromString("kd");
    if (!s_c || !s_q || !s_kd) return nullptr;
    return PyModule_Create(&module);
}
