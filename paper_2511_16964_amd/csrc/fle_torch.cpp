// The package's functions as one call from Python into native code: tensors are read, checked, allocated and handed to
// libfle without the interpreter in between.  A call at the size of one small layer spends its time there: an fp32 layer of 64 x
// 256 x 256 took 8.6 us a call through ctypes, of which the GPU works 5.
//
// Every function here returns None for whatever it does not take (anything but plain tensors on the current GPU that the
// library accepts as they are); the caller then goes the way through binding.Call and its like, which raises the errors.
// Nothing is kept between calls.  Scratch memory comes from torch's allocator under the current stream, the one the kernels
// are enqueued on, and goes back to it at the end of the call, in stream order.  What is read of a tensor is a raw pointer, so every
// tensor of a call is held until its kernels are enqueued: the arguments by the caller, those in an epilogue by a tuple
// of the list's entries that the call takes first (the list itself may be changed by another thread as soon as the interpreter
// lock is given up, and by a number's own conversion before that).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cmath>

#include "fle.h"

namespace {

using at::Tensor;

PyObject *g_names[FLE_LAYERNORM_PRE + 1];  // op names, interned, by kind
PyObject *g_raw_stream;                    // torch._C._cuda_getCurrentRawStream

// The device that everything in a call lives on, and where the work goes.
struct Place {
    c10::DeviceIndex dev;
    void *stream;
};

// A tensor whose memory is what its sizes and strides say: no subclass, wrapper, lazy conjugate or other layout.
const Tensor *plain(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || at::isTensorSubclassLike(t) || t.is_conj() || t.is_neg() || t._is_zerotensor()) return nullptr;
    return t.numel() > 0 ? &t : nullptr;
}

bool open_place(const Tensor &x, Place *pl) {
    if (c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled()) return false;
    const c10::Device cur = c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice();
    pl->dev = x.device().index();
    if (cur.index() != pl->dev) return false;
    PyObject *i = PyLong_FromLong(pl->dev);
    PyObject *s = i ? PyObject_CallOneArg(g_raw_stream, i) : nullptr;
    Py_XDECREF(i);
    if (!s) return false;
    pl->stream = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !PyErr_Occurred();
}

int dtype_code(at::ScalarType t) {
    switch (t) {
    case at::kFloat: return FLE_F32;
    case at::kBFloat16: return FLE_BF16;
    case at::kHalf: return FLE_F16;
    case at::kFloat8_e4m3fn: return FLE_F8E4M3;
    default: return -1;
    }
}

bool vector_of(const Tensor *t, int64_t n, at::ScalarType dt, const Place &pl) {
    return t && t->dim() == 1 && t->size(0) == n && (n <= 1 || t->stride(0) == 1) && t->scalar_type() == dt && t->device().index() == pl.dev;
}
bool matrix_of(const Tensor *t, int64_t M, int64_t N, at::ScalarType dt, const Place &pl) {
    return t && t->dim() == 2 && t->size(0) == M && t->size(1) == N && (N <= 1 || t->stride(1) == 1) && t->scalar_type() == dt && t->device().index() == pl.dev;
}

Tensor fresh(at::IntArrayRef sizes, at::ScalarType dt, const Place &pl) {
    return at::empty(sizes, at::TensorOptions().dtype(dt).device(c10::Device(c10::DeviceType::CUDA, pl.dev)));
}

struct Ops {
    fle_op op[FLE_MAX_OPS];
    int n = 0;
    fle_op &add(int kind) {
        op[n] = fle_op{};
        op[n].kind = kind;
        return op[n++];
    }
};

// Plans, allocates the scratch memory and enqueues (the interpreter lock is given up meanwhile: a launch may wait for a full queue).
bool enqueue(fle_problem &p, const fle_groups *g, const Place &pl) {
    p.stream = pl.stream;
    fle_status s = FLE_OK;
    PyThreadState *save = PyEval_SaveThread();
    try {
        size_t need = 0;
        s = g ? fle_workspace_size_grouped(&p, g, &need) : fle_workspace_size(&p, &need);
        if (s == FLE_OK) {
            Tensor ws;
            if (need > 0) {
                ws = fresh({int64_t(need)}, at::kByte, pl);
                p.workspace = ws.data_ptr();
                p.workspace_bytes = need;
            }
            s = g ? fle_run_grouped(&p, g) : fle_run(&p);
        }
    } catch (...) {
        PyEval_RestoreThread(save);
        throw;
    }
    PyEval_RestoreThread(save);
    return s == FLE_OK;
}

// x [M,K], w [N,K] (grouped: [G,N,K]), b and out into a problem.
void set_problem(fle_problem &p, fle_groups *g, const Tensor &x, const Tensor &w, const Tensor *b, const Tensor &out, bool lse, const Ops &ops) {
    const int64_t M = x.size(0), K = x.size(1), N = w.size(-2);
    p = fle_problem{};
    p.M = M; p.N = N; p.K = K;
    p.dtype = dtype_code(x.scalar_type());
    p.x = x.data_ptr(); p.ldx = M > 1 ? x.stride(0) : std::max(K, x.stride(0));
    p.w = w.data_ptr(); p.ldw = N > 1 ? w.stride(-2) : std::max(K, w.stride(-2));
    p.b = b ? b->data_ptr() : nullptr;
    p.out = out.data_ptr();
    p.ldo = lse ? 0 : M > 1 ? out.stride(0) : std::max(N, out.stride(0));
    p.ops = const_cast<fle_op *>(ops.op);
    p.n_ops = ops.n;
    if (g) {
        const int64_t G = w.size(0);
        g->n_groups = int32_t(G);
        g->w_group_stride = G > 1 ? w.stride(0) : 0;
        g->b_group_stride = b && b->dim() == 2 && G > 1 ? b->stride(0) : 0;
    }
}

// One entry of an epilogue list.
bool read_op(PyObject *e, Ops &ops, int64_t M, int64_t N, int64_t K, at::ScalarType io, const Place &pl, bool *lse) {
    if (!PyTuple_CheckExact(e) || PyTuple_GET_SIZE(e) < 1 || ops.n >= FLE_MAX_OPS) return false;
    const Py_ssize_t len = PyTuple_GET_SIZE(e);
    PyObject *name = PyTuple_GET_ITEM(e, 0);
    int kind = -1;
    for (int k = 0; k <= FLE_LAYERNORM_PRE && kind < 0; ++k)
        if (g_names[k] == name) kind = k;
    for (int k = 0; k <= FLE_LAYERNORM_PRE && kind < 0 && PyUnicode_CheckExact(name); ++k)
        if (g_names[k] && PyUnicode_Compare(g_names[k], name) == 0) kind = k;
    if (kind < 0) return false;
    fle_op &op = ops.add(kind);
    *lse = kind == FLE_LOGSUMEXP;
    auto number = [&](PyObject *v, float *to) {
        if (!PyFloat_Check(v) && !PyLong_Check(v)) return false;
        const double d = PyFloat_AsDouble(v);
        if (d == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return false; }
        *to = float(d);
        return true;
    };
    switch (kind) {
    case FLE_SCALE: return len >= 2 && number(PyTuple_GET_ITEM(e, 1), &op.alpha);
    case FLE_RESIDUAL:
    case FLE_STORE: {
        const Tensor *t = len >= 2 ? plain(PyTuple_GET_ITEM(e, 1)) : nullptr;
        if (!matrix_of(t, M, N, io, pl)) return false;
        op.p0 = t->data_ptr();
        op.ld = M > 1 ? t->stride(0) : std::max(N, t->stride(0));
        return true;
    }
    case FLE_LAYERNORM:
    case FLE_LAYERNORM_PRE: {
        if (len < 4 || !number(PyTuple_GET_ITEM(e, 3), &op.alpha)) return false;
        for (int i = 1; i <= 2; ++i) {
            PyObject *o = PyTuple_GET_ITEM(e, i);
            if (o == Py_None) continue;
            const Tensor *t = plain(o);
            if (!vector_of(t, kind == FLE_LAYERNORM ? N : K, io, pl)) return false;
            (i == 1 ? op.p0 : op.p1) = t->data_ptr();
        }
        return true;
    }
    case FLE_MXSCALE:
        for (int i = 1; i <= 2; ++i) {
            const Tensor *t = len >= 3 ? plain(PyTuple_GET_ITEM(e, i)) : nullptr;
            if (!matrix_of(t, i == 1 ? M : N, K / 32, at::kByte, pl) || !t->is_contiguous()) return false;
            (i == 1 ? op.p0 : op.p1) = t->data_ptr();
        }
        return true;
    default: return true;
    }
}

// A reference that ends with the scope.
struct Held {
    PyObject *p;
    explicit Held(PyObject *q) : p(q) {}
    ~Held() { Py_XDECREF(p); }
    Held(const Held &) = delete;
    Held &operator=(const Held &) = delete;
};

PyObject *not_here() {
    if (PyErr_Occurred()) PyErr_Clear();
    Py_RETURN_NONE;
}

PyObject *linear_impl(PyObject *const *args, bool grouped) {
    const Tensor *x = plain(args[0]), *w = plain(args[1]);
    PyObject *const o_b = args[2], *const list = args[3], *const o_out = args[4];
    if (!x || !w || x->dim() != 2 || w->dim() != (grouped ? 3 : 2) || w->size(-1) != x->size(1)) return not_here();
    Place pl;
    if (!open_place(*x, &pl)) return not_here();
    const int64_t M = x->size(0), K = x->size(1), N = w->size(-2);
    const at::ScalarType dt = x->scalar_type(), io = dt == at::kFloat8_e4m3fn ? at::kBFloat16 : dt;
    if (dtype_code(dt) < 0 || w->scalar_type() != dt || w->device().index() != pl.dev) return not_here();
    if (K > 1 && (x->stride(1) != 1 || w->stride(-1) != 1)) return not_here();
    const Tensor *b = nullptr;
    if (o_b != Py_None) {
        b = plain(o_b);
        if (!b || !(grouped && b->dim() == 2 ? matrix_of(b, w->size(0), N, io, pl) : vector_of(b, N, io, pl))) return not_here();
    }
    fle_groups g{};
    if (grouped) {
        const Tensor *off = plain(args[5]);
        if (!off || off->scalar_type() != at::kLong || off->dim() != 1 || off->size(0) != w->size(0) + 1 || !off->is_contiguous() || off->device().index() != pl.dev) return not_here();
        g.row_offsets = reinterpret_cast<const int64_t *>(off->data_ptr());
    }
    Ops ops;
    bool lse = false;
    if (!PyList_CheckExact(list) && !PyTuple_CheckExact(list)) return not_here();
    const Held entries(PySequence_Tuple(list));  // (a tuple itself, or the list's entries of now; an entry is a tuple and does not change)
    if (!entries.p) return not_here();
    const Py_ssize_t n = PyTuple_GET_SIZE(entries.p);
    for (Py_ssize_t i = 0; i < n; ++i)
        if (!read_op(PyTuple_GET_ITEM(entries.p, i), ops, M, N, K, io, pl, &lse)) return not_here();
    Tensor out;
    if (o_out != Py_None) {
        const Tensor *t = plain(o_out);
        if (!(lse ? vector_of(t, M, io, pl) : matrix_of(t, M, N, io, pl)) || (!lse && M > 1 && t->stride(0) < N)) return not_here();
        out = *t;
    } else {
        out = lse ? fresh({M}, io, pl) : fresh({M, N}, io, pl);
    }
    fle_problem p;
    set_problem(p, grouped ? &g : nullptr, *x, *w, b, out, lse, ops);
    if (!enqueue(p, grouped ? &g : nullptr, pl)) return not_here();
    if (o_out != Py_None) {
        Py_INCREF(o_out);
        return o_out;
    }
    return THPVariable_Wrap(std::move(out));
}

// (x, w, b, epilogue, out)
PyObject *linear(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 5) return not_here();
    try {
        return linear_impl(args, false);
    } catch (...) {  // (out of memory, say: the other way meets it again and raises it as torch does)
        return not_here();
    }
}

// (x, w, b, epilogue, out, offsets)
PyObject *grouped_linear(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 6) return not_here();
    try {
        return linear_impl(args, true);
    } catch (...) {
        return not_here();
    }
}

// Token and sequence stride of a [B,T,H,D] tensor with packed (h, d).
bool strides_of(const Tensor &t, int64_t *ld, int64_t *sb) {
    const int64_t B = t.size(0), T = t.size(1), H = t.size(2), D = t.size(3);
    if ((D > 1 && t.stride(3) != 1) || (H > 1 && t.stride(2) != D)) return false;
    *ld = T > 1 ? t.stride(1) : H * D;
    *sb = B > 1 ? t.stride(0) : 0;
    return true;
}

bool attend(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &o, int causal, float scale, const Place &pl) {
    fle_attention p{};
    p.dtype = dtype_code(q.scalar_type());
    p.causal = causal;
    p.B = q.size(0); p.T = q.size(1); p.H = q.size(2); p.D = q.size(3); p.Tk = k.size(1);
    p.q = q.data_ptr(); p.k = k.data_ptr(); p.v = v.data_ptr(); p.o = o.data_ptr();
    if (!strides_of(q, &p.ldq, &p.sbq) || !strides_of(k, &p.ldk, &p.sbk) || !strides_of(v, &p.ldv, &p.sbv) || !strides_of(o, &p.ldo, &p.sbo)) return false;
    p.scale = scale;
    p.stream = pl.stream;
    fle_status s = FLE_OK;
    PyThreadState *save = PyEval_SaveThread();
    try {
        size_t need = 0;
        s = fle_attention_workspace_size(&p, &need);
        if (s == FLE_OK) {
            Tensor ws;
            if (need > 0) ws = fresh({int64_t(need)}, at::kByte, pl);
            s = fle_attention_run_ws(&p, need > 0 ? ws.data_ptr() : nullptr, need);
        }
    } catch (...) {
        PyEval_RestoreThread(save);
        throw;
    }
    PyEval_RestoreThread(save);
    return s == FLE_OK;
}

bool mask_of(PyObject *o, int *causal) {
    if (!PyLong_Check(o)) return false;  // (bool among them)
    const long v = PyLong_AsLong(o);
    if (v < 0 || v > 0x7fffffff) return false;
    *causal = int(v);
    return true;
}

// (q, k, v, causal, scale)
PyObject *attention(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 5) return not_here();
    try {
        const Tensor *q = plain(args[0]), *k = plain(args[1]), *v = plain(args[2]);
        int causal = 0;
        float scale = 0.0f;
        if (!q || !k || !v || q->dim() != 4 || k->dim() != 4 || v->sizes() != k->sizes() || q->size(0) != k->size(0) || q->size(2) != k->size(2) || q->size(3) != k->size(3)) return not_here();
        if (!mask_of(args[3], &causal)) return not_here();
        if (args[4] != Py_None) {
            if (!PyFloat_CheckExact(args[4])) return not_here();
            scale = float(PyFloat_AS_DOUBLE(args[4]));
        }
        Place pl;
        if (!open_place(*q, &pl) || k->device().index() != pl.dev || v->device().index() != pl.dev) return not_here();
        const at::ScalarType dt = q->scalar_type();
        if (k->scalar_type() != dt || v->scalar_type() != dt || (dt != at::kBFloat16 && dt != at::kHalf)) return not_here();
        Tensor out = fresh(q->sizes(), dt, pl);
        if (!attend(*q, *k, *v, out, causal, scale, pl)) return not_here();
        return THPVariable_Wrap(std::move(out));
    } catch (...) {
        return not_here();
    }
}

// (x, n, w_qkv, b_qkv, w_o, b_o, heads, causal, ln_mid, w1, b1, w2, b2, ln_out) -> (x', n')
PyObject *transformer_layer(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 14) return not_here();
    try {
        const Tensor *x = plain(args[0]), *nx = plain(args[1]), *wq = plain(args[2]), *wo = plain(args[4]), *w1 = plain(args[9]), *b1 = plain(args[10]), *w2 = plain(args[11]), *b2 = plain(args[12]);
        const Tensor *bq = args[3] == Py_None ? nullptr : plain(args[3]), *bo = args[5] == Py_None ? nullptr : plain(args[5]);
        if (!x || !nx || !wq || !wo || !w1 || !b1 || !w2 || !b2 || (args[3] != Py_None && !bq) || (args[5] != Py_None && !bo)) return not_here();
        if (x->dim() != 3 || nx->sizes() != x->sizes() || !x->is_contiguous() || !nx->is_contiguous() || !PyLong_CheckExact(args[6])) return not_here();
        const int64_t B = x->size(0), T = x->size(1), C = x->size(2), M = B * T, H = PyLong_AsLong(args[6]);
        int causal = 0;
        if (H < 1 || C % H || !mask_of(args[7], &causal) || w1->dim() != 2) return not_here();
        const int64_t D = C / H, F = w1->size(0);
        Place pl;
        if (!open_place(*x, &pl)) return not_here();
        const at::ScalarType dt = x->scalar_type();
        if ((dt != at::kBFloat16 && dt != at::kHalf) || nx->scalar_type() != dt || nx->device().index() != pl.dev) return not_here();
        if (!matrix_of(wq, 3 * C, C, dt, pl) || !matrix_of(wo, C, C, dt, pl) || !matrix_of(w1, F, C, dt, pl) || !matrix_of(w2, C, F, dt, pl)) return not_here();
        if ((bq && !vector_of(bq, 3 * C, dt, pl)) || (bo && !vector_of(bo, C, dt, pl)) || !vector_of(b1, F, dt, pl) || !vector_of(b2, C, dt, pl)) return not_here();
        fle_op norm[2];
        for (int i = 0; i < 2; ++i) {  // (gamma, beta, eps), read as an epilogue entry is
            PyObject *ln = args[i == 0 ? 8 : 13];
            if (!PyTuple_CheckExact(ln) || PyTuple_GET_SIZE(ln) < 3) return not_here();
            PyObject *e = PyTuple_Pack(4, g_names[FLE_LAYERNORM], PyTuple_GET_ITEM(ln, 0), PyTuple_GET_ITEM(ln, 1), PyTuple_GET_ITEM(ln, 2));
            if (!e) return not_here();
            Ops one;
            bool lse = false;
            const bool ok = read_op(e, one, M, C, C, dt, pl, &lse);  // (the tensors live on in ln)
            Py_DECREF(e);
            if (!ok) return not_here();
            norm[i] = one.op[0];
        }
        const Tensor x2 = x->view({M, C}), n2 = nx->view({M, C});
        const Tensor qkv = fresh({M, 3 * C}, dt, pl), o = fresh({M, C}, dt, pl), h = fresh({M, C}, dt, pl), m = fresh({M, C}, dt, pl), u = fresh({M, F}, dt, pl);
        Tensor xo = fresh({B, T, C}, dt, pl), no = fresh({B, T, C}, dt, pl);
        const Tensor q5 = qkv.view({B, T, 3, H, D}), o4 = o.view({B, T, H, D}), xo2 = xo.view({M, C}), no2 = no.view({M, C});
        auto step = [&](const Tensor &in, const Tensor &w, const Tensor *b, const Tensor &out, const Ops &ops) {
            fle_problem p;
            set_problem(p, nullptr, in, w, b, out, false, ops);
            return enqueue(p, nullptr, pl);
        };
        auto add_store_norm = [&](Ops &ops, const Tensor &res, const Tensor &to, const fle_op &ln) {
            fle_op &r = ops.add(FLE_RESIDUAL);
            r.p0 = res.data_ptr(); r.ld = C;
            fle_op &s = ops.add(FLE_STORE);
            s.p0 = to.data_ptr(); s.ld = C;
            ops.op[ops.n++] = ln;
        };
        Ops a, c, d, e;
        if (bq) a.add(FLE_BIAS);
        if (bo) c.add(FLE_BIAS);
        add_store_norm(c, x2, h, norm[0]);
        d.add(FLE_BIAS);
        d.add(FLE_GELU_ERF);
        e.add(FLE_BIAS);
        add_store_norm(e, h, xo2, norm[1]);
        if (!step(n2, *wq, bq, qkv, a)) return not_here();
        if (!attend(q5.select(2, 0), q5.select(2, 1), q5.select(2, 2), o4, causal, 0.0f, pl)) return not_here();
        if (!step(o, *wo, bo, m, c) || !step(m, *w1, b1, u, d) || !step(u, *w2, b2, no2, e)) return not_here();
        PyObject *px = THPVariable_Wrap(std::move(xo)), *pn = THPVariable_Wrap(std::move(no));
        PyObject *r = px && pn ? PyTuple_Pack(2, px, pn) : nullptr;
        Py_XDECREF(px);
        Py_XDECREF(pn);
        return r;
    } catch (...) {
        return not_here();
    }
}

PyMethodDef methods[] = {
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, "linear(x, w, b, epilogue, out) -> tensor, or None where it does not apply"},
    {"grouped_linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(grouped_linear)), METH_FASTCALL, "grouped_linear(x, w, b, epilogue, out, offsets) -> tensor or None"},
    {"attention", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(attention)), METH_FASTCALL, "attention(q, k, v, causal, scale) -> tensor or None"},
    {"transformer_layer", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(transformer_layer)), METH_FASTCALL, "transformer_layer(...) -> (x', n') or None"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fle_torch", "libfle's calls on torch tensors, marshalled natively", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fle_torch(void) {
    static const struct { int kind; const char *name; } names[] = {
        {FLE_BIAS, "bias"}, {FLE_SCALE, "scale"}, {FLE_RELU, "relu"}, {FLE_GELU_ERF, "gelu_erf"}, {FLE_GELU_TANH, "gelu_tanh"}, {FLE_RESIDUAL, "residual"}, {FLE_LAYERNORM, "layernorm"},
        {FLE_SOFTMAX, "softmax"}, {FLE_LOGSUMEXP, "logsumexp"}, {FLE_STORE, "store"}, {FLE_MXSCALE, "mxscale"}, {FLE_LAYERNORM_PRE, "layernorm_pre"}};
    for (const auto &n : names) {
        g_names[n.kind] = PyUnicode_InternFromString(n.name);
        if (!g_names[n.kind]) return nullptr;
    }
    PyObject *c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    Py_DECREF(c);
    if (!g_raw_stream) return nullptr;
    return PyModule_Create(&module);
}
