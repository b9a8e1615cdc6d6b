// The calls of include/kvc.h that a serving loop makes for every layer, from Python objects: argument checks and
// marshalling in native code (a CPython extension over torch's tensor type).
//
// Every function takes the arguments of its counterpart in binding.py, with the stream as an integer handle, and
// returns the status of the library call, or None when an argument is not what the common case looks like (not
// exactly a torch.Tensor, a nested one, another device, dtype or shape, not contiguous, nothing to write to) or
// torch throws while it is looked at: nothing has been called then, and binding.py takes its general path, which
// says what is wrong.  The library's functions are bound by address, so that the module works with whatever build
// of the library binding.py has loaded.
//
// A decode call costs the host 10.8 us through ctypes and attribute look-ups, most of it Python; a call on a few
// short sequences is over sooner than that on the device.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "kvc.h"

namespace {

decltype(&kvc_paged_attention_decode) g_decode;
decltype(&kvc_paged_attention_decode_workspace_bytes) g_workspace_bytes;
decltype(&kvc_paged_attention_decode_scheduled) g_scheduled;
decltype(&kvc_attn_schedule_build) g_build;
decltype(&kvc_paged_attention_prefill) g_prefill;
decltype(&kvc_kv_cache_append) g_append;
decltype(&kvc_kv_block_copy) g_copy;
PyTypeObject *g_desc_type;  // binding.AttnDesc, the ctypes structure of kvc_attn_desc

// Arguments of one call; `ok` turns false at the first one that is not of the common kind.
struct Args {
    PyObject *const *a;
    Py_ssize_t n, at = 0;
    bool ok = true;

    PyObject *next() { return at < n ? a[at++] : (ok = false, Py_None); }
    // a plain tensor (no subclass, no grad-mode wrapper) with storage; null otherwise
    const at::Tensor *any_tensor() {
        PyObject *o = next();
        if (!ok || !THPVariable_CheckExact(o)) return ok = false, nullptr;
        const at::Tensor &t = THPVariable_Unpack(o);
        // a nested tensor calls itself strided and contiguous but has no sizes
        if (!t.defined() || t.is_nested() || t.layout() != at::kStrided || !t.has_storage()) return ok = false, nullptr;
        return &t;
    }
    const at::Tensor *device_tensor() {
        const at::Tensor *t = any_tensor();
        if (t && !(t->is_cuda() && t->is_contiguous())) ok = false;
        return ok ? t : nullptr;
    }
    double number() {
        PyObject *o = next();
        if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return ok = false, 0.0;
        const double x = PyFloat_AsDouble(o);
        if (x == -1.0 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return x;
    }
    int64_t integer() {
        PyObject *o = next();
        if (!PyLong_CheckExact(o)) return ok = false, 0;
        const long long x = PyLong_AsLongLong(o);
        if (x == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return x;
    }
    int32_t int32() {
        const int64_t x = integer();
        if (x != int32_t(x)) ok = false;
        return int32_t(x);
    }
    void *stream() {
        PyObject *o = next();
        if (!PyLong_CheckExact(o)) return ok = false, nullptr;
        void *p = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return p;
    }
    bool descriptor(kvc_attn_desc *d) {
        PyObject *o = next();
        Py_buffer b;
        if (!ok || !PyObject_TypeCheck(o, g_desc_type) || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return ok = false; }
        if (b.len == Py_ssize_t(sizeof *d)) memcpy(d, b.buf, sizeof *d); else ok = false;
        PyBuffer_Release(&b);
        return ok;
    }
    bool done() const { return ok && at == n; }
};

int dtype_code(const at::Tensor &t) {
    return t.scalar_type() == at::kFloat ? KVC_F32 : t.scalar_type() == at::kBFloat16 ? KVC_BF16 : -1;
}
bool is_int32(const at::Tensor &t) { return t.scalar_type() == at::kInt; }
size_t bytes_of(const at::Tensor &t) { return size_t(t.numel()) * t.element_size(); }
bool fits(int64_t x) { return x == int32_t(x); }
// at least the rows of q that the descriptor speaks of
bool holds_rows(const at::Tensor &t, const kvc_attn_desc &d) {
    return t.numel() >= int64_t(d.num_seqs) * d.num_q_heads * d.head_dim;
}

// Runs the library call (which does not throw; nothing else may be in it) without the interpreter lock.
template <class Call>
PyObject *run(Call call) {
    PyThreadState *s = PyEval_SaveThread();
    const int rc = call();
    PyEval_RestoreThread(s);
    return PyLong_FromLong(rc);
}

// The address of a tensor's data, as data_ptr() gives it to Python; not ok where that raises.
struct Data {
    void *p = nullptr;
    bool ok = false;
    explicit Data(const at::Tensor *t) {
        try {
            p = t->data_ptr();
            ok = true;
        } catch (...) {
        }
    }
};

// q, k_cache, v_cache, block_tables, context_lens, scale, out, desc, workspace | None, stream
PyObject *decode(PyObject *const *args, Py_ssize_t n) {
    Args a{args, n};
    const at::Tensor *q = a.device_tensor(), *k = a.device_tensor(), *v = a.device_tensor();
    const at::Tensor *bt = a.device_tensor(), *cl = a.device_tensor();
    const double scale = a.number();
    const at::Tensor *out = a.device_tensor();
    kvc_attn_desc d;
    if (!a.ok || !a.descriptor(&d)) Py_RETURN_NONE;
    const at::Tensor *ws = nullptr;
    if (a.at < n && args[a.at] == Py_None) a.at++; else ws = a.device_tensor();
    void *stream = a.stream();
    if (!a.done()) Py_RETURN_NONE;
    if (v->sizes() != k->sizes() || v->scalar_type() != q->scalar_type() || k->scalar_type() != q->scalar_type() ||
        !is_int32(*bt) || !is_int32(*cl) || q->dim() < 1 || bt->dim() < 1 || bt->size(0) != q->size(0) || cl->dim() != 1 ||
        cl->size(0) != q->size(0) || out->sizes() != q->sizes() || out->scalar_type() != q->scalar_type())
        Py_RETURN_NONE;
    if (!ws && g_workspace_bytes(&d) != 0) Py_RETURN_NONE;  // the general path allocates one
    const Data dq(q), dk(k), dv(v), db(bt), dc(cl), dout(out), dw(ws ? ws : q);
    if (!(dq.ok && dk.ok && dv.ok && db.ok && dc.ok && dout.ok && dw.ok)) Py_RETURN_NONE;
    const size_t ws_bytes = ws ? bytes_of(*ws) : 0;
    return run([&] {
        return g_decode(dq.p, dk.p, dv.p, static_cast<const int32_t *>(db.p), static_cast<const int32_t *>(dc.p), float(scale),
                        dout.p, &d, ws ? dw.p : nullptr, ws_bytes, stream);
    });
}

// q, k_cache, v_cache, schedule, scale, out, desc, workspace, stream
PyObject *scheduled(PyObject *const *args, Py_ssize_t n) {
    Args a{args, n};
    const at::Tensor *q = a.device_tensor(), *k = a.device_tensor(), *v = a.device_tensor(), *sched = a.device_tensor();
    const double scale = a.number();
    const at::Tensor *out = a.device_tensor();
    kvc_attn_desc d;
    if (!a.ok || !a.descriptor(&d)) Py_RETURN_NONE;
    const at::Tensor *ws = a.device_tensor();
    void *stream = a.stream();
    if (!a.done()) Py_RETURN_NONE;
    if (v->sizes() != k->sizes() || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type() ||
        out->scalar_type() != q->scalar_type() || !holds_rows(*q, d) || !holds_rows(*out, d))
        Py_RETURN_NONE;
    const Data dq(q), dk(k), dv(v), ds(sched), dout(out), dw(ws);
    if (!(dq.ok && dk.ok && dv.ok && ds.ok && dout.ok && dw.ok)) Py_RETURN_NONE;
    const size_t sched_bytes = size_t(sched->numel()), ws_bytes = bytes_of(*ws);
    return run([&] { return g_scheduled(dq.p, dk.p, dv.p, ds.p, sched_bytes, float(scale), dout.p, &d, dw.p, ws_bytes, stream); });
}

// block_tables, context_lens, desc, schedule, stream
PyObject *schedule_build(PyObject *const *args, Py_ssize_t n) {
    Args a{args, n};
    const at::Tensor *bt = a.device_tensor(), *cl = a.device_tensor();
    kvc_attn_desc d;
    if (!a.ok || !a.descriptor(&d)) Py_RETURN_NONE;
    const at::Tensor *sched = a.device_tensor();
    void *stream = a.stream();
    if (!a.done()) Py_RETURN_NONE;
    if (!is_int32(*bt) || !is_int32(*cl) || bt->numel() < int64_t(d.num_seqs) * d.max_blocks_per_seq || cl->numel() < d.num_seqs)
        Py_RETURN_NONE;
    const Data db(bt), dc(cl), ds(sched);
    if (!(db.ok && dc.ok && ds.ok)) Py_RETURN_NONE;
    const size_t sched_bytes = size_t(sched->numel());
    return run([&] {
        return g_build(static_cast<const int32_t *>(db.p), static_cast<const int32_t *>(dc.p), &d, ds.p, sched_bytes, stream);
    });
}

// q, k_cache, v_cache, block_tables, context_lens, q_start, scale, max_query_len, out, kernel, stream
PyObject *prefill(PyObject *const *args, Py_ssize_t n) {
    Args a{args, n};
    const at::Tensor *q = a.device_tensor(), *k = a.device_tensor(), *v = a.device_tensor();
    const at::Tensor *bt = a.device_tensor(), *cl = a.device_tensor(), *qs = a.device_tensor();
    const double scale = a.number();
    const int32_t max_query_len = a.int32();
    const at::Tensor *out = a.device_tensor();
    const int32_t kernel = a.int32();
    void *stream = a.stream();
    if (!a.done()) Py_RETURN_NONE;
    if (!is_int32(*qs) || !is_int32(*bt) || !is_int32(*cl) || cl->dim() != 1 || qs->dim() != 1 || qs->size(0) != cl->size(0) + 1 ||
        v->sizes() != k->sizes() || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type() ||
        q->dim() != 3 || k->dim() != 4 || bt->dim() != 2 || k->size(3) != q->size(2) || bt->size(0) != cl->size(0) ||
        dtype_code(*q) < 0 || out->scalar_type() != q->scalar_type() || out->numel() < q->numel())
        Py_RETURN_NONE;
    for (int64_t x : {cl->size(0), q->size(0), q->size(1), q->size(2), k->size(0), k->size(1), k->size(2), bt->size(1)})
        if (!fits(x)) Py_RETURN_NONE;
    const kvc_attn_desc d = {int32_t(cl->size(0)), int32_t(q->size(1)), int32_t(k->size(1)), int32_t(q->size(2)), int32_t(k->size(2)),
                             int32_t(bt->size(1)), int32_t(k->size(0)), dtype_code(*q), 0, 0, kernel, 0};
    const Data dq(q), dk(k), dv(v), db(bt), dc(cl), ds(qs), dout(out);
    if (!(dq.ok && dk.ok && dv.ok && db.ok && dc.ok && ds.ok && dout.ok)) Py_RETURN_NONE;
    const int32_t total_q = int32_t(q->size(0));
    return run([&] {
        return g_prefill(dq.p, dk.p, dv.p, static_cast<const int32_t *>(db.p), static_cast<const int32_t *>(dc.p),
                         static_cast<const int32_t *>(ds.p), float(scale), dout.p, &d, total_q, max_query_len, stream);
    });
}

// k_new, v_new, k_cache, v_cache, block_tables, positions, stream
PyObject *append(PyObject *const *args, Py_ssize_t n) {
    Args a{args, n};
    const at::Tensor *kn = a.device_tensor(), *vn = a.device_tensor(), *k = a.device_tensor(), *v = a.device_tensor();
    const at::Tensor *bt = a.device_tensor(), *pos = a.device_tensor();
    void *stream = a.stream();
    if (!a.done()) Py_RETURN_NONE;
    if (kn->dim() != 3 || vn->sizes() != kn->sizes() || k->dim() != 4 || v->sizes() != k->sizes() || k->size(1) != kn->size(1) ||
        k->size(3) != kn->size(2) || vn->scalar_type() != kn->scalar_type() || k->scalar_type() != kn->scalar_type() ||
        v->scalar_type() != kn->scalar_type() || !is_int32(*bt) || !is_int32(*pos) || pos->dim() != 1 ||
        pos->size(0) != kn->size(0) || bt->dim() != 2 || bt->size(0) != kn->size(0) || dtype_code(*kn) < 0)
        Py_RETURN_NONE;
    for (int64_t x : {kn->size(0), kn->size(1), kn->size(2), k->size(0), k->size(2), bt->size(1)})
        if (!fits(x)) Py_RETURN_NONE;
    const int32_t heads = int32_t(kn->size(1));
    const kvc_attn_desc d = {int32_t(kn->size(0)), heads, heads, int32_t(kn->size(2)), int32_t(k->size(2)), int32_t(bt->size(1)),
                             int32_t(k->size(0)), dtype_code(*kn), 0, 0, KVC_KERNEL_VALU, 0};
    const Data dkn(kn), dvn(vn), dk(k), dv(v), db(bt), dp(pos);
    if (!(dkn.ok && dvn.ok && dk.ok && dv.ok && db.ok && dp.ok)) Py_RETURN_NONE;
    return run([&] {
        return g_append(dkn.p, dvn.p, dk.p, dv.p, static_cast<const int32_t *>(db.p), static_cast<const int32_t *>(dp.p), &d, stream);
    });
}

bool pool_of(const at::Tensor &t, kvc_pool *p) {
    if (t.dim() < 3 || t.size(0) < 1 || t.size(1) < 1 || !fits(t.size(0))) return false;
    const Data d(&t);
    const int64_t block_bytes = t.numel() / (t.size(0) * t.size(1)) * int64_t(t.element_size());
    *p = kvc_pool{d.p, t.size(1), block_bytes, t.size(1) * block_bytes, int32_t(t.size(0)), 0};
    return d.ok;
}

// src, dst ([planes][blocks][...] on the device), block_mapping, stream
PyObject *block_copy(PyObject *const *args, Py_ssize_t n) {
    Args a{args, n};
    const at::Tensor *src = a.device_tensor(), *dst = a.device_tensor(), *map = a.device_tensor();
    void *stream = a.stream();
    if (!a.done() || map->scalar_type() != at::kLong) Py_RETURN_NONE;
    kvc_pool s, d;
    const Data dm(map);
    if (!pool_of(*src, &s) || !pool_of(*dst, &d) || !dm.ok) Py_RETURN_NONE;
    const int64_t pairs = map->numel() / 2;
    return run([&] { return g_copy(&s, &d, static_cast<const int64_t *>(dm.p), pairs, stream); });
}

// addresses of the library's functions, in the order of the assignments, and the descriptor's type
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 8 || !PyType_Check(args[7])) {
        PyErr_SetString(PyExc_TypeError, "bind takes the addresses of seven functions and the descriptor's type");
        return nullptr;
    }
    void *f[7];
    for (int i = 0; i < 7; ++i) {
        f[i] = PyLong_AsVoidPtr(args[i]);
        if (!f[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a function address is null");
            return nullptr;
        }
    }
    g_decode = reinterpret_cast<decltype(g_decode)>(f[0]);
    g_workspace_bytes = reinterpret_cast<decltype(g_workspace_bytes)>(f[1]);
    g_scheduled = reinterpret_cast<decltype(g_scheduled)>(f[2]);
    g_build = reinterpret_cast<decltype(g_build)>(f[3]);
    g_prefill = reinterpret_cast<decltype(g_prefill)>(f[4]);
    g_append = reinterpret_cast<decltype(g_append)>(f[5]);
    g_copy = reinterpret_cast<decltype(g_copy)>(f[6]);
    Py_INCREF(args[7]);
    Py_XDECREF(reinterpret_cast<PyObject *>(g_desc_type));
    g_desc_type = reinterpret_cast<PyTypeObject *>(args[7]);
    Py_RETURN_NONE;
}

// The interpreter's frames are C: what torch throws (sizes() or data_ptr() of a tensor of an unusual kind) ends here.
template <PyObject *(*Call)(PyObject *const *, Py_ssize_t)>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    try {
        return Call(args, n);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

#define KVC_METHOD(name, function) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(function)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {KVC_METHOD("bind", bind),
                           KVC_METHOD("decode", entry<decode>),
                           KVC_METHOD("scheduled", entry<scheduled>),
                           KVC_METHOD("schedule_build", entry<schedule_build>),
                           KVC_METHOD("prefill", entry<prefill>),
                           KVC_METHOD("append", entry<append>),
                           KVC_METHOD("block_copy", entry<block_copy>),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "kvc_call", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_kvc_call() { return PyModule_Create(&g_module); }
