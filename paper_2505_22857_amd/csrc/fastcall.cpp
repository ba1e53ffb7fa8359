// The per-call path of the Python binding for the calls that a decoder makes
// once per frame (advance, fused_greedy_step, fused_topk): argument checks,
// output allocation and the C ABI call without interpreter work in between.
// Each function answers the ordinary call (plain contiguous device tensors,
// the current stream) and returns None for anything else, which the Python
// method then handles, and reports, by itself; a failing C call returns its
// code.  Everything that can fail otherwise, the results' Python objects among
// it, comes before the C call: after it the step has been enqueued, and None
// would make the Python method enqueue it a second time.
//
// An enqueued call cost the host 4.4 us (advance) to 9.9 us (top-k, three
// outputs allocated), more than the kernels of small batches take, and 2.4 us
// of it are the launch: 3.1 us and 6.0 us here.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "ngpu_lm.h"

namespace {

// The library's entry points, bound from the handle that the binding loaded.
decltype(&ngpu_lm_advance) g_advance;
decltype(&ngpu_lm_fused_greedy_step) g_step;
decltype(&ngpu_lm_fused_topk) g_topk;

PyObject *none() {
    PyErr_Clear();   // the Python method meets the error again, or does not
    Py_RETURN_NONE;
}

struct Ref {   // an owned reference
    PyObject *p = nullptr;
    Ref() = default;
    explicit Ref(PyObject *o) : p(o) {}
    Ref(const Ref &) = delete;
    ~Ref() { Py_XDECREF(p); }
    PyObject *release() {
        PyObject *o = p;
        p = nullptr;
        return o;
    }
};

const at::Tensor *tensor_of(PyObject *o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.scalar_type() == type && t.layout() == at::kStrided && t.is_cuda() ? &t : nullptr;
}
const at::Tensor *dense(PyObject *o, at::ScalarType type) {
    const at::Tensor *t = tensor_of(o, type);
    return t && t->is_contiguous() ? t : nullptr;
}

// An output: the caller's contiguous tensor of at least n entries, or a new one.
struct Output {
    Ref object;
    at::Tensor t;
    bool set(PyObject *o, at::ScalarType type, int64_t n, at::IntArrayRef shape, const at::Tensor &like) {
        if (o == Py_None) {
            t = at::empty(shape, like.options().dtype(type));
            object.p = THPVariable_Wrap(t);
            return object.p && t.is_contiguous();
        }
        const at::Tensor *x = dense(o, type);
        if (!x || x->numel() < n) return false;
        Py_INCREF(o);
        object.p = o;
        t = *x;
        return true;
    }
};

bool whole(PyObject *o, int64_t &v) {   // an int (no conversion that could run user code)
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool real(PyObject *o, float &v) {
    if (!PyFloat_CheckExact(o)) return false;
    v = static_cast<float>(PyFloat_AS_DOUBLE(o));
    return true;
}

template <class F>
int without_gil(F f) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// advance(handle, V, states, scores or None, next or None)
PyObject *advance(PyObject *, PyObject *const *a, Py_ssize_t n) try {
    int64_t h, V;
    if (n != 5 || !whole(a[0], h) || !whole(a[1], V)) return none();
    const at::Tensor *states = dense(a[2], at::kInt);
    if (!states) return none();
    const int64_t B = states->numel();
    Output scores, next;
    if (!scores.set(a[3], at::kFloat, B * V, {B, V}, *states) || !next.set(a[4], at::kInt, B * V, {B, V}, *states))
        return none();
    const auto *st = static_cast<const int32_t *>(states->data_ptr());
    auto *sc = static_cast<float *>(scores.t.data_ptr());
    auto *nx = static_cast<int32_t *>(next.t.data_ptr());
    Ref result(PyTuple_Pack(2, scores.object.p, next.object.p));
    if (!result.p) return none();
    void *stream = current_stream();
    const int rc = without_gil([&] { return g_advance(reinterpret_cast<const ngpu_lm *>(h), st, B, sc, nx, stream); });
    return rc != NGPU_OK ? PyLong_FromLong(rc) : result.release();
} catch (const std::exception &) {
    return none();   // nothing was enqueued: the C call, and what follows it, throws nothing
}

// step(handle, V, asr, lam, states, prev or None, mode, tokens or None)
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n) try {
    int64_t h, V, mode;
    float lam;
    if (n != 8 || !whole(a[0], h) || !whole(a[1], V) || !real(a[3], lam) || !whole(a[6], mode) || mode < 0 || mode > 3)
        return none();
    const at::Tensor *asr = tensor_of(a[2], at::kFloat), *states = dense(a[4], at::kInt);
    const at::Tensor *prev = a[5] == Py_None ? nullptr : dense(a[5], at::kInt);
    if (!asr || !states || (a[5] != Py_None && !prev) || asr->dim() != 2 || asr->stride(1) != 1) return none();
    const int64_t B = asr->size(0);
    if (asr->size(1) < V + (mode != NGPU_FUSION_PLAIN) || states->numel() != B || (prev && prev->numel() != B))
        return none();
    Output tokens;
    if (!tokens.set(a[7], at::kInt, B, {B}, *asr)) return none();
    const auto *row = static_cast<const float *>(asr->data_ptr());
    auto *st = static_cast<int32_t *>(states->data_ptr());
    auto *pv = prev ? static_cast<int32_t *>(prev->data_ptr()) : nullptr;
    auto *tk = static_cast<int32_t *>(tokens.t.data_ptr());
    const int64_t ld = asr->stride(0);
    void *stream = current_stream();
    const int rc = without_gil([&] {
        return g_step(reinterpret_cast<const ngpu_lm *>(h), row, B, ld, static_cast<int32_t>(mode), lam, st, pv, tk,
                      stream);
    });
    return rc != NGPU_OK ? PyLong_FromLong(rc) : tokens.object.release();
} catch (const std::exception &) {
    return none();
}

// topk(handle, V, asr, lam, k, states, tokens or None, scores or None, next or None)
PyObject *topk(PyObject *, PyObject *const *a, Py_ssize_t n) try {
    int64_t h, V, k;
    float lam;
    if (n != 9 || !whole(a[0], h) || !whole(a[1], V) || !real(a[3], lam) || !whole(a[4], k) || k < 1 ||
        k > NGPU_LM_MAX_TOPK)
        return none();
    const at::Tensor *asr = tensor_of(a[2], at::kFloat), *states = dense(a[5], at::kInt);
    if (!asr || !states || asr->dim() != 2 || asr->stride(1) != 1) return none();
    const int64_t B = asr->size(0);
    if (asr->size(1) < V || states->numel() != B) return none();
    Output tokens, scores, next;
    if (!tokens.set(a[6], at::kInt, B * k, {B, k}, *asr) || !scores.set(a[7], at::kFloat, B * k, {B, k}, *asr) ||
        !next.set(a[8], at::kInt, B * k, {B, k}, *asr))
        return none();
    const auto *row = static_cast<const float *>(asr->data_ptr());
    const auto *st = static_cast<const int32_t *>(states->data_ptr());
    auto *tk = static_cast<int32_t *>(tokens.t.data_ptr());
    auto *sc = static_cast<float *>(scores.t.data_ptr());
    auto *nx = static_cast<int32_t *>(next.t.data_ptr());
    const int64_t ld = asr->stride(0);
    Ref result(PyTuple_Pack(3, tokens.object.p, scores.object.p, next.object.p));
    if (!result.p) return none();
    void *stream = current_stream();
    const int rc = without_gil([&] {
        return g_topk(reinterpret_cast<const ngpu_lm *>(h), row, B, ld, lam, static_cast<int32_t>(k), st, tk, sc, nx,
                      stream);
    });
    return rc != NGPU_OK ? PyLong_FromLong(rc) : result.release();
} catch (const std::exception &) {
    return none();
}

// bind(addresses of ngpu_lm_advance, ngpu_lm_fused_greedy_step, ngpu_lm_fused_topk)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
    int64_t p[3];
    if (n != 3 || !whole(a[0], p[0]) || !whole(a[1], p[1]) || !whole(a[2], p[2])) {
        PyErr_SetString(PyExc_TypeError, "bind takes three addresses");
        return nullptr;
    }
    g_advance = reinterpret_cast<decltype(g_advance)>(p[0]);
    g_step = reinterpret_cast<decltype(g_step)>(p[1]);
    g_topk = reinterpret_cast<decltype(g_topk)>(p[2]);
    return none();
}

// The torch.__version__ of the headers this was compiled with.
PyObject *torch_version(PyObject *, PyObject *const *, Py_ssize_t) { return PyUnicode_FromString(NGPU_TORCH_VERSION); }

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyMethodDef method(const char *name) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(F)), METH_FASTCALL, nullptr};
}
PyMethodDef g_methods[] = {method<advance>("advance"), method<step>("step"), method<topk>("topk"),
                           method<bind>("bind"), method<torch_version>("torch_version"),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&g_module); }
