// The argument checks of binding.py's calls, in native code, for the calls a serving loop makes step after step: everything given (outputs,
// workspace), plain tensors on the device, plain numbers.  Each function checks what the Python beside it checks, calls the C ABI
// and returns its status; for anything else it does nothing and returns None, and the Python goes through the same checks
// one by one and says what is wrong (or takes what is not plain).  What bounds a step of few short requests is the host:
// appended and decoded with three peers, 4 requests, the two calls took 9.4 us of Python beside 10 us in the library and the runtime.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <initializer_list>

#include "esp.h"

namespace {

PyObject* g_stream = nullptr;                      // binding._stream
decltype(&esp_kv_append) p_append;
decltype(&esp_partial_attn_decode) p_decode;
decltype(&esp_partial_attn_decode_merge) p_decode_merge;
decltype(&esp_partial_attn_prefill) p_prefill;
decltype(&esp_partial_attn_prefill_f32) p_prefill_f32;
decltype(&esp_merge_partials) p_merge;
decltype(&esp_merge_partials_f32) p_merge_f32;

// a plain torch.Tensor (no subclass: it may answer for itself) with storage on the device
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}
// the same, of this type, contiguous
const at::Tensor* dev(PyObject* o, at::ScalarType type) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}
// an output that this many elements of are written
const at::Tensor* out(PyObject* o, at::ScalarType type, int64_t numel) {
    const at::Tensor* t = dev(o, type);
    return t && t->numel() >= numel ? t : nullptr;
}
const at::Tensor* scratch(PyObject* o) {
    const at::Tensor* t = plain(o);
    return t && t->is_contiguous() ? t : nullptr;
}
bool small(PyObject* o, int32_t& v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    v = (int32_t)x;
    return !over && x == v;
}
bool scale_of(PyObject* o, int64_t D, float& v) {
    if (o == Py_None) { v = (float)std::pow((double)D, -0.5); return D > 0; }
    if (!PyFloat_CheckExact(o)) return false;
    v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
bool fits(std::initializer_list<int64_t> sizes) {
    for (int64_t s : sizes) if (s > INT32_MAX) return false;
    return true;
}
bool stream_of(void*& s) {
    PyObject* r = PyObject_CallNoArgs(g_stream);
    if (!r) return false;
    s = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}
// pointers of a list or tuple of tensors of one type, each of the shape `like`
struct Parts { int32_t n = 0; const void* p[ESP_MAX_PARTIALS]; };
bool parts_of(PyObject* seq, at::ScalarType type, at::IntArrayRef like, Parts& out) {
    if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    if (n > ESP_MAX_PARTIALS) return false;
    for (Py_ssize_t i = 0; i < n; ++i) {
        const at::Tensor* t = dev(PySequence_Fast_GET_ITEM(seq, i), type);
        if (!t || t->sizes() != like) return false;
        out.p[i] = t->data_ptr();
    }
    out.n = (int32_t)n;
    return true;
}

template <class F> PyObject* status_of(F call) {
    esp_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}
// a tensor may refuse to be looked at (no storage, one that stands for others): the Python meets the same and says so
template <class F> PyObject* guarded(F body) {
    PyObject* r = nullptr;
    try { r = body(); } catch (...) {}
    if (r) return r;
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

constexpr auto BF16 = at::kBFloat16;
constexpr auto F32 = at::kFloat;
constexpr auto I32 = at::kInt;

// k, v, slot_idx, k_pool, v_pool
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        if (n != 5) return nullptr;
        const at::Tensor *k = dev(a[0], BF16), *v = dev(a[1], BF16), *slots = dev(a[2], I32), *kp = dev(a[3], BF16), *vp = dev(a[4], BF16);
        if (!k || !v || !slots || !kp || !vp || k->dim() != 3 || kp->dim() != 3 || slots->dim() != 1) return nullptr;
        const int64_t T = k->size(0), H = k->size(1), D = k->size(2);
        if (v->sizes() != k->sizes() || slots->size(0) != T || vp->sizes() != kp->sizes() || kp->size(1) != H || kp->size(2) != D) return nullptr;
        void* s;
        if (!fits({T, H, D}) || !stream_of(s)) return nullptr;
        const void *pk = k->data_ptr(), *pv = v->data_ptr();
        void *ppk = kp->data_ptr(), *ppv = vp->data_ptr();
        const int32_t* ps = (const int32_t*)slots->data_ptr();
        const int64_t S = kp->size(0);
        return status_of([&] { return p_append(pk, pv, ps, (int32_t)T, ppk, ppv, S, (int32_t)H, (int32_t)D, s); });
    });
}

// q, k_pool, v_pool, slot_idx, seq_offsets, max_len, softmax_scale, O, LSE, workspace[, peer_O, peer_LSE]
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        if (n != 10 && n != 12) return nullptr;
        const at::Tensor *q = dev(a[0], BF16), *kp = dev(a[1], BF16), *vp = dev(a[2], BF16), *slots = dev(a[3], I32), *off = dev(a[4], I32);
        if (!q || !kp || !vp || !slots || !off || q->dim() != 3 || kp->dim() != 3) return nullptr;
        const int64_t B = q->size(0), Hq = q->size(1), D = q->size(2), S = kp->size(0), H = kp->size(1), total = slots->numel();
        const at::Tensor *O = out(a[7], BF16, q->numel()), *L = out(a[8], F32, B * Hq), *ws = scratch(a[9]);
        if (!O || !L || !ws) return nullptr;
        int32_t max_len;
        float scale;
        if (vp->sizes() != kp->sizes() || kp->size(2) != D || off->numel() != B + 1 || !small(a[5], max_len) || !scale_of(a[6], D, scale))
            return nullptr;
        Parts po, pl;
        if (n == 12 && (!parts_of(a[10], BF16, q->sizes(), po) || !parts_of(a[11], F32, q->sizes().slice(0, 2), pl) || po.n != pl.n)) return nullptr;
        void* s;
        if (!fits({B, Hq, D, H, total}) || !stream_of(s)) return nullptr;
        const void *pq = q->data_ptr(), *pk = kp->data_ptr(), *pv = vp->data_ptr();
        const int32_t *ps = (const int32_t*)slots->data_ptr(), *pf = (const int32_t*)off->data_ptr();
        void *pO = O->data_ptr(), *pw = ws->data_ptr();
        float* pL = (float*)L->data_ptr();
        const size_t wn = (size_t)ws->numel();
        return status_of([&] {
            if (n == 10)
                return p_decode(pq, pk, pv, S, ps, pf, (int32_t)B, (int32_t)total, max_len, (int32_t)Hq, (int32_t)H, (int32_t)D, scale, pO, pL, pw, wn, s);
            return p_decode_merge(pq, pk, pv, S, ps, pf, (int32_t)B, (int32_t)total, max_len, (int32_t)Hq, (int32_t)H, (int32_t)D, scale,
                                  po.p, (const float* const*)pl.p, po.n, pO, pL, pw, wn, s);
        });
    });
}

// q, k, v, q_pos, kv_pos, cu_q, cu_kv, max_q, max_kv, softmax_scale, causal, O, LSE, workspace
PyObject* prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        if (n != 14) return nullptr;
        const at::Tensor *q = dev(a[0], BF16), *k = dev(a[1], BF16), *v = dev(a[2], BF16), *qp = dev(a[3], I32), *kp = dev(a[4], I32);
        const at::Tensor *O = plain(a[11]), *L = dev(a[12], F32), *ws = scratch(a[13]);
        if (!q || !k || !v || !qp || !kp || !O || !L || !ws || q->dim() != 3 || k->dim() != 3 || qp->dim() != 1 || kp->dim() != 1) return nullptr;
        const bool f32 = O->scalar_type() == F32;
        const int64_t Tq = q->size(0), Hq = q->size(1), D = q->size(2), Tk = k->size(0), H = k->size(1);
        if ((!f32 && O->scalar_type() != BF16) || !O->is_contiguous() || O->sizes() != q->sizes() || L->sizes() != q->sizes().slice(0, 2)) return nullptr;
        if (v->sizes() != k->sizes() || k->size(2) != D || qp->size(0) != Tq || kp->size(0) != Tk) return nullptr;
        int64_t batch = 1;
        int32_t max_q = (int32_t)Tq, max_kv = (int32_t)Tk;
        const int32_t *cq = nullptr, *ck = nullptr;
        if (a[5] != Py_None) {
            const at::Tensor *tq = dev(a[5], I32), *tk = dev(a[6], I32);
            if (!tq || !tk || tk->numel() != tq->numel() || !small(a[7], max_q) || !small(a[8], max_kv)) return nullptr;
            batch = tq->numel() - 1;
            cq = (const int32_t*)tq->data_ptr();
            ck = (const int32_t*)tk->data_ptr();
        } else if (a[6] != Py_None) {
            return nullptr;
        }
        float scale;
        if (!scale_of(a[9], D, scale) || !PyBool_Check(a[10])) return nullptr;
        void* s;
        if (!fits({Tq, Tk, Hq, H, D, batch}) || !stream_of(s)) return nullptr;
        const int32_t causal = a[10] == Py_True ? 1 : 0;
        const void *pq = q->data_ptr(), *pk = k->data_ptr(), *pv = v->data_ptr();
        const int32_t *pqp = (const int32_t*)qp->data_ptr(), *pkp = (const int32_t*)kp->data_ptr();
        void *pO = O->data_ptr(), *pw = ws->data_ptr();
        float* pL = (float*)L->data_ptr();
        const size_t wn = (size_t)ws->numel();
        return status_of([&] {
            if (f32)
                return p_prefill_f32(pq, pk, pv, pqp, pkp, cq, ck, (int32_t)batch, (int32_t)Tq, (int32_t)Tk, max_q, max_kv, (int32_t)Hq, (int32_t)H,
                                     (int32_t)D, scale, causal, (float*)pO, pL, pw, wn, s);
            return p_prefill(pq, pk, pv, pqp, pkp, cq, ck, (int32_t)batch, (int32_t)Tq, (int32_t)Tk, max_q, max_kv, (int32_t)Hq, (int32_t)H,
                             (int32_t)D, scale, causal, pO, pL, pw, wn, s);
        });
    });
}

// O_parts, LSE_parts, O, LSE
PyObject* merge(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        if (n != 4 || (!PyList_CheckExact(a[0]) && !PyTuple_CheckExact(a[0])) || PySequence_Fast_GET_SIZE(a[0]) == 0) return nullptr;
        const at::Tensor* first = plain(PySequence_Fast_GET_ITEM(a[0], 0));
        if (!first || first->dim() < 2) return nullptr;
        const bool f32 = first->scalar_type() == F32;
        Parts po, pl;
        const auto sizes = first->sizes();
        if ((!f32 && first->scalar_type() != BF16) || !parts_of(a[0], first->scalar_type(), sizes, po) ||
            !parts_of(a[1], F32, sizes.slice(0, sizes.size() - 1), pl) || po.n != pl.n) return nullptr;
        const int64_t Hq = sizes[sizes.size() - 2], D = sizes[sizes.size() - 1];
        int64_t T = 1;
        for (size_t i = 0; i + 2 < sizes.size(); ++i) T *= sizes[i];
        const at::Tensor *O = out(a[2], BF16, first->numel()), *L = out(a[3], F32, T * Hq);
        if (!O || !L) return nullptr;
        void* s;
        if (!fits({T, Hq, D}) || !stream_of(s)) return nullptr;
        void* pO = O->data_ptr();
        float* pL = (float*)L->data_ptr();
        return status_of([&] {
            if (f32) return p_merge_f32((const float* const*)po.p, (const float* const*)pl.p, po.n, (int32_t)T, (int32_t)Hq, (int32_t)D, pO, pL, s);
            return p_merge(po.p, (const float* const*)pl.p, po.n, (int32_t)T, (int32_t)Hq, (int32_t)D, pO, pL, s);
        });
    });
}

// the stream function, then the addresses of the C ABI's functions in the order below
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 8) { PyErr_SetString(PyExc_TypeError, "bind: the stream function and seven addresses"); return nullptr; }
    void* at[7];
    for (int i = 0; i < 7; ++i) {
        at[i] = PyLong_AsVoidPtr(a[i + 1]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(a[0]);
    Py_XSETREF(g_stream, a[0]);
    p_append = (decltype(p_append))at[0];
    p_decode = (decltype(p_decode))at[1];
    p_decode_merge = (decltype(p_decode_merge))at[2];
    p_prefill = (decltype(p_prefill))at[3];
    p_prefill_f32 = (decltype(p_prefill_f32))at[4];
    p_merge = (decltype(p_merge))at[5];
    p_merge_f32 = (decltype(p_merge_f32))at[6];
    Py_RETURN_NONE;
}

#define ESP_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ESP_METHOD(bind), ESP_METHOD(kv_append), ESP_METHOD(decode), ESP_METHOD(prefill), ESP_METHOD(merge), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
