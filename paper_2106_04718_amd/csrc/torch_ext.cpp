// Fast front of the Python binding: checks the tensors of a call and makes the
// call of the C ABI in one step of native code.
//
// Reading the shapes, types, devices and pointers of six or seven tensors from
// Python took 5 to 6 us a call, more than the kernels of a small decode step;
// here it takes a few tenths of a microsecond.  Every function returns the
// status of its C entry point, or None for anything that is not the plain case
// (an argument of another type, shape, layout or device, a tensor subclass or
// wrapper, a device that is not current): the caller then takes the general
// path in Python, which says what is wrong.  So a call is accepted here only
// if that path accepts it, with the same arguments for the C entry point.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "fastseq_hip.h"

namespace {

PyObject *g_raw_stream = nullptr;   // torch's current raw stream of a device index
PyObject *g_cur_device = nullptr;   // torch's current device index

// Thrown nowhere: `ok` turns false at the first argument that is not plain.
struct Args {
    PyObject *const *a;
    bool ok = true;
    int dev = -1;

    // A dense tensor on the common device, of exactly torch's tensor type.
    const at::Tensor *tensor(int i) {
        static const at::Tensor none;
        if (!ok || !THPVariable_CheckExact(a[i])) {
            ok = false;
            return &none;
        }
        const at::Tensor &t = THPVariable_Unpack(a[i]);
        if (!t.defined() || t.layout() != at::kStrided || !t.has_storage() || !t.is_cuda()) {
            ok = false;
            return &none;
        }
        const int d = (int)t.get_device();
        if (dev < 0) dev = d;
        ok = ok && d == dev;
        return &t;
    }
    long long integer(int i) {
        if (!ok || !PyLong_CheckExact(a[i])) {
            ok = false;
            return 0;
        }
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(a[i], &over);
        ok = ok && over == 0 && v >= INT_MIN && v <= INT_MAX;
        return v;
    }
    void need(bool c) { ok = ok && c; }
};

bool is4(const at::Tensor &t) { return t.dim() == 4 && t.is_contiguous(); }
bool same(const at::Tensor &x, const at::Tensor &y) { return x.sizes() == y.sizes() && x.scalar_type() == y.scalar_type(); }
bool fits(int64_t v) { return v <= INT_MAX; }
int code(at::ScalarType t) { return t == at::kFloat ? FS_F32 : t == at::kBFloat16 ? FS_BF16 : -1; }
// int32 [n], contiguous
bool ints(const at::Tensor &t, int64_t n) {
    return t.scalar_type() == at::kInt && t.dim() == 1 && t.size(0) == n && t.is_contiguous();
}
// int32 [rows, cols] with unit column stride; its leading dimension in ld
bool table(const at::Tensor &t, int64_t rows, int &ld) {
    if (t.scalar_type() != at::kInt || t.dim() != 2 || t.size(0) != rows || rows < 1) return false;
    if (t.size(1) > 1 && t.stride(1) != 1) return false;
    const int64_t l = rows > 1 ? t.stride(0) : t.size(1);
    if (l < 0 || !fits(l) || !fits(t.size(1))) return false;
    ld = (int)l;
    return true;
}

// The stream of the tensors' device, which must be current.
bool stream_of(Args &g, void *&s) {
    if (!g.ok || g.dev < 0) return false;
    PyObject *cur = PyObject_CallNoArgs(g_cur_device);
    if (!cur) return false;
    const long c = PyLong_AsLong(cur);
    if (c != g.dev) {
        Py_DECREF(cur);
        return false;
    }
    PyObject *p = PyObject_CallOneArg(g_raw_stream, cur);
    Py_DECREF(cur);
    if (!p) return false;
    s = PyLong_AsVoidPtr(p);
    Py_DECREF(p);
    return !PyErr_Occurred();
}

PyObject *declined() {
    PyErr_Clear();
    Py_RETURN_NONE;
}

// Sizes of an attention call's q [B, k, H, D] and keys [B, H, S, D]
struct Sizes {
    int B, k, H, D, S, dtype;
};
bool attn_sizes(const at::Tensor &q, const at::Tensor &K, const at::Tensor &V, const at::Tensor &len, Sizes &z) {
    if (!is4(q) || !is4(K) || !is4(V) || !same(K, V) || K.scalar_type() != q.scalar_type()) return false;
    z.dtype = code(q.scalar_type());
    if (z.dtype < 0 || K.size(0) != q.size(0) || K.size(1) != q.size(2) || K.size(3) != q.size(3)) return false;
    for (int i = 0; i < 4; ++i)
        if (!fits(q.size(i)) || !fits(K.size(i))) return false;
    z.B = (int)q.size(0), z.k = (int)q.size(1), z.H = (int)q.size(2), z.D = (int)q.size(3), z.S = (int)K.size(2);
    return ints(len, q.size(0));
}

// beam_cross_attn(q, K, V, src_len, out, workspace)
PyObject *cross_attn(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 6) return declined();
    Args g{a};
    const at::Tensor &q = *g.tensor(0), &K = *g.tensor(1), &V = *g.tensor(2), &len = *g.tensor(3), &out = *g.tensor(4),
                     &ws = *g.tensor(5);
    Sizes z;
    void *s = nullptr;
    if (!g.ok || !attn_sizes(q, K, V, len, z) || !same(out, q) || !out.is_contiguous() || !ws.is_contiguous() ||
        !stream_of(g, s))
        return declined();
    return PyLong_FromLong(fs_beam_cross_attn(q.data_ptr(), K.data_ptr(), V.data_ptr(),
                                              static_cast<const int32_t *>(len.data_ptr()), out.data_ptr(), z.B, z.k,
                                              z.H, z.S, z.D, z.dtype, ws.data_ptr(), ws.nbytes(), s));
}

// beam_decode_step(q, K, V, src_len, tokens, n, logits, t or -1, out, workspace)
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 10) return declined();
    Args g{a};
    const at::Tensor &q = *g.tensor(0), &K = *g.tensor(1), &V = *g.tensor(2), &len = *g.tensor(3), &tok = *g.tensor(4),
                     &lg = *g.tensor(6), &out = *g.tensor(8), &ws = *g.tensor(9);
    const long long ng = g.integer(5);
    long long t = g.integer(7);
    Sizes z;
    int ld = 0;
    void *s = nullptr;
    if (!g.ok || !attn_sizes(q, K, V, len, z) || !same(out, q) || !out.is_contiguous() || !ws.is_contiguous())
        return declined();
    const int64_t rows = (int64_t)z.B * z.k;
    if (!table(tok, rows, ld) || lg.dim() != 2 || lg.scalar_type() != at::kFloat || lg.size(0) != rows ||
        !lg.is_contiguous() || !fits(lg.size(1)))
        return declined();
    if (t < 0) t = tok.size(1);
    if (t > tok.size(1) || !stream_of(g, s)) return declined();
    return PyLong_FromLong(fs_beam_decode_step(
        q.data_ptr(), K.data_ptr(), V.data_ptr(), static_cast<const int32_t *>(len.data_ptr()), out.data_ptr(), z.B,
        z.k, z.H, z.S, z.D, z.dtype, static_cast<const int32_t *>(tok.data_ptr()), ld, (int)t, (int)ng,
        static_cast<float *>(lg.data_ptr()), (int)lg.size(1), ws.data_ptr(), ws.nbytes(), s));
}

// beam_prefix_attn(q, Kp, Vp, prefix_len, Kt, Vt, t, out, workspace, anc or None)
PyObject *prefix_attn(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 10) return declined();
    Args g{a};
    const at::Tensor &q = *g.tensor(0), &K = *g.tensor(1), &V = *g.tensor(2), &len = *g.tensor(3), &Kt = *g.tensor(4),
                     &Vt = *g.tensor(5), &out = *g.tensor(7), &ws = *g.tensor(8);
    const long long t = g.integer(6);
    Sizes z;
    int ld = 0;
    void *s = nullptr;
    if (!g.ok || !attn_sizes(q, K, V, len, z) || !same(out, q) || !out.is_contiguous() || !ws.is_contiguous())
        return declined();
    const int64_t rows = (int64_t)z.B * z.k;
    if (!is4(Kt) || !is4(Vt) || !same(Kt, Vt) || Kt.scalar_type() != q.scalar_type() || Kt.size(0) != rows ||
        Kt.size(1) != z.H || Kt.size(3) != z.D || !fits(Kt.size(2)))
        return declined();
    const int T = (int)Kt.size(2);
    const int32_t *anc = nullptr;
    if (a[9] != Py_None) {
        const at::Tensor &tb = *g.tensor(9);
        if (!g.ok || !tb.is_contiguous() || !table(tb, rows, ld)) return declined();
        anc = static_cast<const int32_t *>(tb.data_ptr());
    }
    if (!stream_of(g, s)) return declined();
    const int32_t *lp = static_cast<const int32_t *>(len.data_ptr());
    if (a[9] != Py_None)
        return PyLong_FromLong(fs_beam_prefix_attn_indirect(
            q.data_ptr(), K.data_ptr(), V.data_ptr(), lp, Kt.data_ptr(), Vt.data_ptr(), anc, ld, T, (int)t,
            out.data_ptr(), z.B, z.k, z.H, z.S, z.D, z.dtype, ws.data_ptr(), ws.nbytes(), s));
    return PyLong_FromLong(fs_beam_prefix_attn(q.data_ptr(), K.data_ptr(), V.data_ptr(), lp, Kt.data_ptr(),
                                               Vt.data_ptr(), T, (int)t, out.data_ptr(), z.B, z.k, z.H, z.S, z.D,
                                               z.dtype, ws.data_ptr(), ws.nbytes(), s));
}

// ngram_block(tokens, n, logits, t or -1)
PyObject *ngram_block(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 4) return declined();
    Args g{a};
    const at::Tensor &tok = *g.tensor(0), &lg = *g.tensor(2);
    const long long ng = g.integer(1);
    long long t = g.integer(3);
    int ld = 0;
    void *s = nullptr;
    if (!g.ok || lg.dim() != 2 || lg.scalar_type() != at::kFloat || !lg.is_contiguous() || !fits(lg.size(0)) ||
        !fits(lg.size(1)) || !table(tok, lg.size(0), ld))
        return declined();
    if (t < 0) t = tok.size(1);
    if (t > tok.size(1) || !stream_of(g, s)) return declined();
    return PyLong_FromLong(fs_ngram_block(static_cast<const int32_t *>(tok.data_ptr()), ld, (int)lg.size(0), (int)t,
                                          (int)ng, static_cast<float *>(lg.data_ptr()), (int)lg.size(1), s));
}

// beam_select(logits, beam_scores, k, c, tokens (unread for n == 0), n, t or -1, scores, beam, token, workspace)
PyObject *select(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 11) return declined();
    Args g{a};
    const at::Tensor &lg = *g.tensor(0), &bs = *g.tensor(1), &o0 = *g.tensor(7), &o1 = *g.tensor(8),
                     &o2 = *g.tensor(9), &ws = *g.tensor(10);
    const long long k = g.integer(2), c = g.integer(3), ng = g.integer(5);
    long long t = g.integer(6);
    const int32_t *tokens = nullptr;
    int ld = 0;
    void *s = nullptr;
    if (!g.ok || ng < 0 || k < 1 || lg.dim() != 2 || lg.scalar_type() != at::kFloat || !lg.is_contiguous() ||
        lg.size(0) % k || !fits(lg.size(0)) || !fits(lg.size(1)) || bs.scalar_type() != at::kFloat || bs.dim() != 1 ||
        bs.size(0) != lg.size(0) || !bs.is_contiguous() || !ws.is_contiguous())
        return declined();
    const int64_t rows = lg.size(0), B = rows / k;
    auto out = [&](const at::Tensor &o, at::ScalarType ty) {
        return o.dim() == 2 && o.size(0) == B && o.size(1) == c && o.scalar_type() == ty && o.is_contiguous();
    };
    if (!out(o0, at::kFloat) || !out(o1, at::kInt) || !out(o2, at::kInt)) return declined();
    if (ng > 0) {
        const at::Tensor &tok = *g.tensor(4);
        if (!g.ok || !table(tok, rows, ld)) return declined();
        if (t < 0) t = tok.size(1);
        if (t > tok.size(1)) return declined();
        tokens = static_cast<const int32_t *>(tok.data_ptr());
    } else {
        t = 0;
    }
    if (!stream_of(g, s)) return declined();
    return PyLong_FromLong(fs_beam_select(
        static_cast<const float *>(lg.data_ptr()), static_cast<const float *>(bs.data_ptr()),
        tokens, ld, (int)t, (int)ng, static_cast<float *>(o0.data_ptr()),
        static_cast<int32_t *>(o1.data_ptr()), static_cast<int32_t *>(o2.data_ptr()), (int)B, (int)k,
        (int)lg.size(1), (int)c, ws.data_ptr(), ws.nbytes(), s));
}

// cache_reorder(K, V, parent, k, t or -1)
PyObject *cache_reorder(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 5) return declined();
    Args g{a};
    const at::Tensor &K = *g.tensor(0), &V = *g.tensor(1), &par = *g.tensor(2);
    const long long k = g.integer(3);
    long long t = g.integer(4);
    void *s = nullptr;
    if (!g.ok || k < 1 || !is4(K) || !is4(V) || !same(K, V) || code(K.scalar_type()) < 0 || K.size(0) % k ||
        !ints(par, K.size(0)))
        return declined();
    for (int i = 0; i < 4; ++i)
        if (!fits(K.size(i))) return declined();
    if (t < 0) t = K.size(2);
    if (!stream_of(g, s)) return declined();
    return PyLong_FromLong(fs_cache_reorder(K.data_ptr(), V.data_ptr(), static_cast<const int32_t *>(par.data_ptr()),
                                            (int)(K.size(0) / k), (int)k, (int)K.size(1), (int)K.size(2), (int)t,
                                            (int)K.size(3), code(K.scalar_type()), s));
}

// ancestry_step(anc, parent, k, t)
PyObject *ancestry_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 4) return declined();
    Args g{a};
    const at::Tensor &anc = *g.tensor(0), &par = *g.tensor(1);
    const long long k = g.integer(2), t = g.integer(3);
    int ld = 0;
    void *s = nullptr;
    if (!g.ok || k < 1 || anc.dim() != 2 || anc.size(0) % k || !fits(anc.size(0)) || !anc.is_contiguous() ||
        !table(anc, anc.size(0), ld) || !ints(par, anc.size(0)) || !stream_of(g, s))
        return declined();
    return PyLong_FromLong(fs_beam_ancestry_step(static_cast<int32_t *>(anc.data_ptr()), ld,
                                                 static_cast<const int32_t *>(par.data_ptr()),
                                                 (int)(anc.size(0) / k), (int)k, (int)t, s));
}

// A torch accessor throws for a tensor whose data must not be touched (one made
// by a tracer, for instance); no exception may cross into the interpreter, so
// such a call is declined too and the general path raises torch's own error.
using Fast = PyObject *(PyObject *, PyObject *const *, Py_ssize_t);
template <Fast F>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n) noexcept {
    try {
        return F(self, a, n);
    } catch (...) {
        return declined();
    }
}

#define FS_FAST(f) (PyCFunction)(void (*)(void)) guarded<f>, METH_FASTCALL
PyMethodDef methods[] = {
    {"beam_cross_attn", FS_FAST(cross_attn), "(q, K, V, src_len, out, workspace) -> status, or None: not the plain case"},
    {"beam_decode_step", FS_FAST(decode_step), "(q, K, V, src_len, tokens, n, logits, t or -1, out, workspace)"},
    {"beam_prefix_attn", FS_FAST(prefix_attn), "(q, Kp, Vp, prefix_len, Kt, Vt, t, out, workspace, anc or None)"},
    {"ngram_block", FS_FAST(ngram_block), "(tokens, n, logits, t or -1)"},
    {"beam_select", FS_FAST(select), "(logits, beam_scores, k, c, tokens or None, n, t or -1, scores, beam, token, workspace)"},
    {"cache_reorder", FS_FAST(cache_reorder), "(K, V, parent, k, t or -1)"},
    {"ancestry_step", FS_FAST(ancestry_step), "(anc, parent, k, t)"},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastseq_torch", "Native argument checks of the tensor front end", -1,
                      methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastseq_torch(void) {
    // torch's own readers of the current device and stream
    PyObject *c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    g_cur_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    Py_DECREF(c);
    if (!g_raw_stream || !g_cur_device) return nullptr;
    return PyModule_Create(&module);
}
