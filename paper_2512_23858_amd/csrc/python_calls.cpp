// Native argument marshalling of the Python package: one C function per launching call.  Each takes the Shape object and
// torch tensors (or None) by position, checks device, layout and element type, and hands raw pointers and the current
// stream to the C ABI.  It returns the C ABI's status, or kCheckFailed when an argument does not pass; the Python side then
// runs its own checks, which raise the matching exception.
//
// Host time per call matters: a short verification step is made of calls whose kernels take a few microseconds, and the
// stream runs dry when the host cannot enqueue that fast.  Marshalling through ctypes took 6-7 us per call beside two
// launches of 3-4 us each; this takes well under one.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ygg.h"

namespace {

constexpr long kCheckFailed = -1;

PyObject* g_field[12];
const char* const kField[12] = {"batch", "n_q_heads", "n_kv_heads", "head_dim", "depth", "width", "n_nodes", "vocab",
                                "kv_dtype", "softmax_scale", "kv_capacity", "max_seq_len"};

PyObject* attribute(PyObject* o, int i) {   // new reference
    PyObject** d = _PyObject_GetDictPtr(o);
    if (d && *d)
        if (PyObject* v = PyDict_GetItemWithError(*d, g_field[i])) {   // the usual case: an instance's own field
            Py_INCREF(v);
            return v;
        }
    PyErr_Clear();
    return PyObject_GetAttr(o, g_field[i]);
}

bool read_int(PyObject* o, int i, int64_t lo, int64_t hi, int64_t& out) {
    PyObject* v = attribute(o, i);
    if (!v) return false;
    out = PyLong_AsLongLong(v);
    Py_DECREF(v);
    return !(out == -1 && PyErr_Occurred()) && out >= lo && out <= hi;
}

// False (no exception set) if a field is missing, not a number or out of the C type's range.
bool read_shape(PyObject* o, ygg_shape& s) {
    int32_t* const dst[12] = {&s.batch, &s.n_q_heads, &s.n_kv_heads, &s.head_dim, &s.depth, &s.width, &s.n_nodes, &s.vocab,
                              &s.kv_dtype, nullptr, nullptr, &s.max_seq_len};
    bool ok = true;
    for (int i = 0; i < 12 && ok; ++i) {
        int64_t v = 0;
        if (i == 9) {
            PyObject* f = attribute(o, i);
            const double x = f ? PyFloat_AsDouble(f) : -1.0;
            Py_XDECREF(f);
            ok = !PyErr_Occurred();
            s.softmax_scale = (float)x;
        } else if (i == 10) {
            ok = read_int(o, i, INT64_MIN, INT64_MAX, s.kv_capacity);
        } else if ((ok = read_int(o, i, INT32_MIN, INT32_MAX, v))) {
            *dst[i] = (int32_t)v;
        }
    }
    PyErr_Clear();
    return ok;
}

// The tensor arguments of one call: pointers come out in order, and one failed check marks the call.
struct Args {
    PyObject* const* a;
    bool ok = true;
    void* ptr(int i, at::ScalarType want, bool any = false) {
        PyObject* o = a[i];
        if (o == Py_None) return nullptr;
        if (!THPVariable_Check(o)) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous() || (!any && t.scalar_type() != want)) { ok = false; return nullptr; }
        return t.data_ptr();
    }
    template <typename T> T* typed(int i, at::ScalarType want) { return static_cast<T*>(ptr(i, want)); }
    int32_t* ints(int i) { return typed<int32_t>(i, at::kInt); }
    float* floats(int i) { return typed<float>(i, at::kFloat); }
    void* scratch(int i, size_t& bytes) {
        void* p = ptr(i, at::kByte, true);
        bytes = p ? THPVariable_Unpack(a[i]).nbytes() : 0;
        return p;
    }
    bool number(int i, int32_t& out) {
        const int64_t v = PyLong_AsLongLong(a[i]);
        if ((v == -1 && PyErr_Occurred()) || v < INT32_MIN || v > INT32_MAX) { PyErr_Clear(); return ok = false; }
        out = (int32_t)v;
        return true;
    }
};

at::ScalarType kv_type(const ygg_shape& s) {
    return s.kv_dtype == YGG_F32 ? at::kFloat : s.kv_dtype == YGG_BF16 ? at::kBFloat16 : at::kByte;
}

template <typename F>
PyObject* finish(bool ok, F&& call) {
    if (!ok) return PyLong_FromLong(kCheckFailed);
    void* stream = c10::hip::getCurrentHIPStream().stream();
    int32_t rc;
    Py_BEGIN_ALLOW_THREADS   // a launch waits when the queue is full
    rc = call(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

bool arity(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd positional arguments, got %zd", want, n);
    return false;
}

// (shape, q, k_cache, v_cache, seq_lens, k_tree, v_tree, parent_idx, out, lse, workspace, main_kernel_only)
PyObject* tree_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 12)) return nullptr;
    ygg_shape s{};
    Args t{a};
    t.ok = read_shape(a[0], s) && s.kv_dtype >= 0 && s.kv_dtype <= 2;
    const at::ScalarType dt = kv_type(s);
    void *q = t.ptr(1, dt), *kc = t.ptr(2, dt), *vc = t.ptr(3, dt), *kt = t.ptr(5, dt), *vt = t.ptr(6, dt), *out = t.ptr(8, dt);
    int32_t *lens = t.ints(4), *parent = t.ints(7);
    float* lse = t.floats(9);
    size_t wn;
    void* ws = t.scratch(10, wn);
    const bool main_only = a[11] == Py_True;
    return finish(t.ok, [&](void* st) {
        return (main_only ? ygg_debug_tree_attention_main : ygg_tree_attention)(&s, q, kc, vc, lens, kt, vt, parent, out, lse, ws, wn, st);
    });
}

// (shape, q, k_cache, v_cache, seq_lens, k_tree, v_tree, k_scale, v_scale, parent_idx, out, lse, workspace)
PyObject* tree_attention_fp8kv(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 13)) return nullptr;
    ygg_shape s{};
    Args t{a};
    t.ok = read_shape(a[0], s);
    void *q = t.ptr(1, at::kBFloat16), *kc = t.ptr(2, at::kByte), *vc = t.ptr(3, at::kByte), *kt = t.ptr(5, at::kByte),
         *vt = t.ptr(6, at::kByte), *out = t.ptr(10, at::kBFloat16);
    int32_t *lens = t.ints(4), *parent = t.ints(9);
    float *ks = t.floats(7), *vs = t.floats(8), *lse = t.floats(11);
    size_t wn;
    void* ws = t.scratch(12, wn);
    return finish(t.ok, [&](void* st) {
        return ygg_tree_attention_fp8kv(&s, q, kc, vc, lens, kt, vt, ks, vs, parent, out, lse, ws, wn, st);
    });
}

// (shape, d, draft_logits, parent_idx, token_ids, cum_logprob, workspace)
PyObject* equal_growth_expand(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 7)) return nullptr;
    ygg_shape s{};
    Args t{a};
    t.ok = read_shape(a[0], s);
    int32_t d = 0;
    t.number(1, d);
    float *x = t.floats(2), *cum = t.floats(5);
    int32_t *parent = t.ints(3), *token = t.ints(4);
    size_t wn;
    void* ws = t.scratch(6, wn);
    return finish(t.ok, [&](void* st) { return ygg_equal_growth_expand(&s, d, x, parent, token, cum, ws, wn, st); });
}

// (shape, d, draft_logits, parent_idx, token_ids, cum_logprob)
PyObject* equal_growth_expand_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 6)) return nullptr;
    ygg_shape s{};
    Args t{a};
    t.ok = read_shape(a[0], s);
    int32_t d = 0;
    t.number(1, d);
    float *x = t.floats(2), *cum = t.floats(5);
    int32_t *parent = t.ints(3), *token = t.ints(4);
    return finish(t.ok, [&](void* st) { return ygg_equal_growth_expand_static(&s, d, x, parent, token, cum, st); });
}

// (shape, t, draft_logits, parent_idx, token_ids, cum_logprob, pool, workspace)
PyObject* equal_growth_attach(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 8)) return nullptr;
    ygg_shape s{};
    Args t{a};
    t.ok = read_shape(a[0], s);
    int32_t step = 0;
    t.number(1, step);
    float *x = t.floats(2), *cum = t.floats(5);
    int32_t *parent = t.ints(3), *token = t.ints(4);
    size_t pn, wn;
    void *pool = t.scratch(6, pn), *ws = t.scratch(7, wn);
    return finish(t.ok, [&](void* st) { return ygg_equal_growth_attach(&s, step, x, parent, token, cum, pool, pn, ws, wn, st); });
}

// (shape, w_verify, parent_idx, token_ids, cum_logprob, kept_nodes, new_parent, new_token, expected_len, best_width,
//  t_verifier, t_draft)
PyObject* prune_for_verification(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 12)) return nullptr;
    ygg_shape s{};
    Args t{a};
    t.ok = read_shape(a[0], s);
    int32_t w = 0;
    t.number(1, w);
    int32_t *parent = t.ints(2), *token = t.ints(3), *kept = t.ints(5), *np = t.ints(6), *nt = t.ints(7), *best = t.ints(9);
    float *cum = t.floats(4), *expected = t.floats(8), *tv = t.floats(10);
    const double td = PyFloat_AsDouble(a[11]);
    if (PyErr_Occurred()) { PyErr_Clear(); t.ok = false; }
    return finish(t.ok, [&](void* st) {
        return ygg_prune_for_verification(&s, w, parent, token, cum, tv, (float)td, kept, np, nt, expected, best, st);
    });
}

// (shape, n_layers, parent_idx, token_ids, k_tree, v_tree, k_cache, v_cache, seq_lens, accept_len, accept_path,
//  bonus_token, target_logits, target_tokens, workspace)
PyObject* accept_and_compact(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!arity(n, 15)) return nullptr;
    ygg_shape s{};
    Args t{a};
    t.ok = read_shape(a[0], s) && s.kv_dtype >= 0 && s.kv_dtype <= 2;
    const at::ScalarType dt = kv_type(s);
    int32_t layers = 0;
    t.number(1, layers);
    int32_t *parent = t.ints(2), *token = t.ints(3), *lens = t.ints(8), *alen = t.ints(9), *path = t.ints(10), *bonus = t.ints(11),
            *tokens = t.ints(13);
    void *kt = t.ptr(4, dt), *vt = t.ptr(5, dt), *kc = t.ptr(6, dt), *vc = t.ptr(7, dt);
    float* logits = t.floats(12);
    size_t wn;
    void* ws = t.scratch(14, wn);
    return finish(t.ok, [&](void* st) {
        return ygg_accept_and_compact(&s, layers, logits, tokens, parent, token, kt, vt, kc, vc, lens, alen, path, bonus, ws, wn, st);
    });
}

// torch reports its errors (no device, a tensor without storage) as C++ exceptions
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    try {
        return F(self, a, n);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define YGG_CALL(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<name>)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    YGG_CALL(tree_attention), YGG_CALL(tree_attention_fp8kv), YGG_CALL(equal_growth_expand), YGG_CALL(equal_growth_expand_static),
    YGG_CALL(equal_growth_attach), YGG_CALL(prune_for_verification), YGG_CALL(accept_and_compact), {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_calls", "native argument marshalling of the launching calls", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
    for (int i = 0; i < 12; ++i)
        if (!(g_field[i] = PyUnicode_InternFromString(kField[i]))) return nullptr;
    return PyModule_Create(&kModule);
}
