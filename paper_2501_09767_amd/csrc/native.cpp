// The calls of lemo.py that a layer makes over and over, marshalled in native code: 0.4 us beside the launch where ctypes and the
// checks in Python take 3 to 4 (three calls of a small binary32 layer: 22 us enqueued from Python, 9.6 so).
//
// Every function takes the arguments of the call of the same name in order and answers None when anything about them is not
// the plain case -- another type, layout, device or size than the checks in lemo.py let through, an output still to be allocated,
// a value that the C ABI refuses -- and has then done nothing: the caller goes the long way, which raises what it always
// raised.  Otherwise the call's return code.  The GIL is released around the call, as ctypes does.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include "lemo.h"

namespace {

PyObject *current_device = nullptr, *raw_stream = nullptr;  // Python callables: () -> device, (device) -> stream address

struct NotPlain {};  // go the long way

void need(bool ok) {
    if (!ok) throw NotPlain{};
}

// a tensor of exactly torch's own class, on the GPU, with storage and elements
const at::Tensor& tensor(PyObject* o, int64_t dim) {
    need(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    need(t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && t.dim() == dim && t.numel() > 0);
    return t;
}
lemo_dtype_t dtype(const at::Tensor& t) {
    if (t.scalar_type() == at::kFloat) return LEMO_F32;
    need(t.scalar_type() == at::kBFloat16);
    return LEMO_BF16;
}
int64_t whole(PyObject* o) {
    need(PyLong_CheckExact(o));
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    need(!over);
    return v;
}
int32_t whole32(PyObject* o) {
    const int64_t v = whole(o);
    need(v >= INT32_MIN && v <= INT32_MAX);
    return (int32_t)v;
}
int32_t size32(int64_t v) {
    need(v <= INT32_MAX);
    return (int32_t)v;
}
float real(PyObject* o) {
    need(PyFloat_CheckExact(o));
    return (float)PyFloat_AS_DOUBLE(o);
}
// a list of rows, or none
const at::Tensor* index(PyObject* o) {
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o, 1);
    need(t.scalar_type() == at::kInt && t.is_contiguous());
    return &t;
}
const int32_t* rows(const at::Tensor* t) { return t ? static_cast<const int32_t*>(t->data_ptr()) : nullptr; }
const at::Tensor& matrix(PyObject* o) {  // rows contiguous
    const at::Tensor& t = tensor(o, 2);
    need(t.stride(1) == 1);
    return t;
}
const at::Tensor& heads(PyObject* o) {  // [S,H,d], d contiguous
    const at::Tensor& t = tensor(o, 3);
    need(t.stride(2) == 1);
    return t;
}
const void* bias_of(PyObject* o, const at::Tensor& like, int64_t n) {
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o, 1);
    need(t.scalar_type() == like.scalar_type() && t.size(0) == n && t.is_contiguous());
    return t.data_ptr();
}
float* plane(PyObject* o, int64_t h, int64_t s) {
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o, 2);
    need(t.scalar_type() == at::kFloat && t.size(0) == h && t.size(1) == s && t.is_contiguous());
    return static_cast<float*>(t.data_ptr());
}
struct Bytes { void* p; size_t n; };
Bytes workspace(PyObject* o) {
    need(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    need(t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage());
    return {t.data_ptr(), (size_t)t.numel() * t.element_size()};
}
void* stream() {
    PyObject* dev = PyObject_CallNoArgs(current_device);
    if (!dev) { PyErr_Clear(); throw NotPlain{}; }
    PyObject* s = PyObject_CallOneArg(raw_stream, dev);
    Py_DECREF(dev);
    if (!s) { PyErr_Clear(); throw NotPlain{}; }
    void* p = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (PyErr_Occurred()) { PyErr_Clear(); throw NotPlain{}; }
    return p;
}
// what the C ABI refuses has had no effect and is left to the long way; a launch that failed is reported
template <typename F> PyObject* call(F f) {
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = f();
    Py_END_ALLOW_THREADS;
    if (rc != LEMO_OK && rc != LEMO_ERR_HIP) Py_RETURN_NONE;
    return PyLong_FromLong(rc);
}
// no C++ exception leaves this file: tensors that refuse to tell their address (inside vmap, for instance) throw c10::Error
template <Py_ssize_t N, PyObject* (*F)(PyObject* const*)> PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != N || !raw_stream) Py_RETURN_NONE;
    try {
        return F(a);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyObject* score_segments(PyObject* const* a) {  // Q K L flags scale scores colsum diag workspace
    const at::Tensor &Q = heads(a[0]), &K = heads(a[1]);
    const int64_t S = Q.size(0), H = Q.size(1), d = Q.size(2);
    const lemo_dtype_t dt = dtype(Q);
    need(K.size(0) == S && K.size(2) == d && K.scalar_type() == Q.scalar_type());
    const at::Tensor& scores = tensor(a[5], 1);
    need(scores.scalar_type() == at::kFloat && scores.size(0) == S && scores.is_contiguous());
    float *col = plane(a[6], H, S), *dg = plane(a[7], H, S);
    const Bytes ws = workspace(a[8]);
    const int32_t L = whole32(a[2]), flags = whole32(a[3]), h = size32(H), hkv = size32(K.size(1)), dd = size32(d);
    const float scale = real(a[4]);
    void *q = Q.data_ptr(), *k = K.data_ptr(), *sc = scores.data_ptr(), *st = stream();
    const int64_t q0 = Q.stride(0), q1 = Q.stride(1), k0 = K.stride(0), k1 = K.stride(1);
    return call([=] {
        return lemo_score_segments(q, k, S, h, hkv, dd, dt, q0, q1, k0, k1, scale, L, (uint32_t)flags, (float*)sc, col, dg, ws.p, ws.n, st);
    });
}

PyObject* select_topk(PyObject* const* a) {  // scores L k kept_idx
    const at::Tensor& scores = tensor(a[0], 1);
    const at::Tensor* kept = index(a[3]);
    need(scores.scalar_type() == at::kFloat && scores.is_contiguous() && kept);
    const int64_t S = scores.size(0);
    const int32_t L = whole32(a[1]), k = whole32(a[2]);
    need(kept->numel() == lemo_kept_count(S, L, k));
    void *sc = scores.data_ptr(), *ki = kept->data_ptr(), *st = stream();
    return call([=] { return lemo_select_topk((const float*)sc, S, L, k, (int32_t*)ki, st); });
}

PyObject* kept_attention(PyObject* const* a) {  // Q K V kept_idx flags scale O workspace M
    const at::Tensor &Q = heads(a[0]), &K = heads(a[1]), &V = heads(a[2]), &O = heads(a[6]);
    const at::Tensor* kept = index(a[3]);
    const int64_t S = Q.size(0), H = Q.size(1), d = Q.size(2);
    const lemo_dtype_t dt = dtype(Q);
    need(K.size(0) == S && K.size(2) == d && K.scalar_type() == Q.scalar_type() && V.sizes() == K.sizes() && V.scalar_type() == K.scalar_type());
    const int64_t M = a[8] != Py_None ? whole(a[8]) : kept ? kept->numel() : S;
    need(M > 0 && (!kept || kept->numel() >= M) && O.scalar_type() == Q.scalar_type() && O.size(0) >= M && O.size(1) == H && O.size(2) == d);
    const Bytes ws = workspace(a[7]);
    const int32_t flags = whole32(a[4]), h = size32(H), hkv = size32(K.size(1)), dd = size32(d);
    const float scale = real(a[5]);
    const int32_t* ki = rows(kept);
    void *q = Q.data_ptr(), *k = K.data_ptr(), *v = V.data_ptr(), *o = O.data_ptr(), *st = stream();
    const int64_t q0 = Q.stride(0), q1 = Q.stride(1), k0 = K.stride(0), k1 = K.stride(1), v0 = V.stride(0), v1 = V.stride(1), o0 = O.stride(0), o1 = O.stride(1);
    return call([=] {
        return lemo_kept_attention(q, k, v, S, h, hkv, dd, dt, q0, q1, k0, k1, v0, v1, ki, M, scale, (uint32_t)flags, o, o0, o1, ws.p, ws.n, st);
    });
}

PyObject* gather_gemm(PyObject* const* a) {  // X kept_idx W bias Y M
    const at::Tensor &X = matrix(a[0]), &W = matrix(a[2]), &Y = matrix(a[4]);
    const at::Tensor* kept = index(a[1]);
    const lemo_dtype_t dt = dtype(X);
    const int64_t S = X.size(0), C = X.size(1), N = W.size(0);
    need(W.size(1) == C && W.scalar_type() == X.scalar_type());
    const int64_t M = a[5] != Py_None ? whole(a[5]) : kept ? kept->numel() : S;
    need(M > 0 && (!kept || kept->numel() >= M) && Y.scalar_type() == X.scalar_type() && Y.size(0) >= M && Y.size(1) == N);
    const void* b = bias_of(a[3], X, N);
    const int32_t* ki = rows(kept);
    const int32_t c = size32(C), n = size32(N);
    void *x = X.data_ptr(), *w = W.data_ptr(), *y = Y.data_ptr(), *st = stream();
    const int64_t x0 = X.stride(0), w0 = W.stride(0), y0 = Y.stride(0);
    return call([=] { return lemo_gather_gemm(x, S, x0, ki, M, w, w0, b, y, y0, c, n, dt, st); });
}

PyObject* gather_gemm_add(PyObject* const* a) {  // X kept_idx W R out_idx bias M
    const at::Tensor &X = matrix(a[0]), &W = matrix(a[2]), &R = matrix(a[3]);
    const at::Tensor *kept = index(a[1]), *out = index(a[4]);
    const lemo_dtype_t dt = dtype(X);
    const int64_t S = X.size(0), C = X.size(1), N = W.size(0);
    need(W.size(1) == C && W.scalar_type() == X.scalar_type() && R.scalar_type() == X.scalar_type() && R.size(1) == N);
    const int64_t M = a[6] != Py_None ? whole(a[6]) : kept ? kept->numel() : out ? out->numel() : S;
    need(M > 0 && (!kept || kept->numel() >= M) && (!out || out->numel() >= M));
    const void* b = bias_of(a[5], X, N);
    const int32_t *ki = rows(kept), *oi = rows(out);
    const int32_t c = size32(C), n = size32(N);
    void *x = X.data_ptr(), *w = W.data_ptr(), *r = R.data_ptr(), *st = stream();
    const int64_t x0 = X.stride(0), w0 = W.stride(0), r0 = R.stride(0), rs = R.size(0);
    return call([=] { return lemo_gather_gemm_add(x, S, x0, ki, M, w, w0, b, r, r0, rs, oi, c, n, dt, st); });
}

PyObject* gather_gemm_dx(PyObject* const* a) {  // dY W dX out_idx
    const at::Tensor &dY = matrix(a[0]), &W = matrix(a[1]), &dX = matrix(a[2]);
    const at::Tensor* out = index(a[3]);
    const lemo_dtype_t dt = dtype(W);
    const int64_t M = dY.size(0), N = dY.size(1), C = W.size(1);
    need(dY.scalar_type() == W.scalar_type() && dX.scalar_type() == W.scalar_type() && W.size(0) == N && dX.size(1) == C && (!out || out->numel() == M));
    const int32_t* oi = rows(out);
    const int32_t c = size32(C), n = size32(N);
    void *y = dY.data_ptr(), *w = W.data_ptr(), *x = dX.data_ptr(), *st = stream();
    const int64_t y0 = dY.stride(0), w0 = W.stride(0), x0 = dX.stride(0), xs = dX.size(0);
    return call([=] { return lemo_gather_gemm_dx(y, y0, M, w, w0, x, x0, xs, oi, c, n, dt, st); });
}

PyObject* gather_gemm_dw(PyObject* const* a) {  // dY X kept_idx dW workspace
    const at::Tensor &dY = matrix(a[0]), &X = matrix(a[1]), &dW = matrix(a[3]);
    const at::Tensor* kept = index(a[2]);
    const lemo_dtype_t dt = dtype(X);
    const int64_t M = dY.size(0), N = dY.size(1), S = X.size(0), C = X.size(1);
    need(dY.scalar_type() == X.scalar_type() && dW.scalar_type() == X.scalar_type() && dW.size(0) == N && dW.size(1) == C && (!kept || kept->numel() == M));
    Bytes ws{nullptr, 0};
    if (a[4] != Py_None) ws = workspace(a[4]);
    else need(dt == LEMO_BF16);  // binary32 needs one, which lemo.py allocates
    const int32_t* ki = rows(kept);
    const int32_t c = size32(C), n = size32(N);
    void *y = dY.data_ptr(), *x = X.data_ptr(), *w = dW.data_ptr(), *st = stream();
    const int64_t y0 = dY.stride(0), x0 = X.stride(0), w0 = dW.stride(0);
    return call([=] { return lemo_gather_gemm_dw(y, y0, x, S, x0, ki, M, w, w0, c, n, dt, ws.p, ws.n, st); });
}

PyObject* scatter_grad(PyObject* const* a) {  // G kept_idx dX mode
    const at::Tensor &G = matrix(a[0]), &dX = matrix(a[2]);
    const at::Tensor* kept = index(a[1]);
    const lemo_dtype_t gt = dtype(G), xt = dtype(dX);
    const int64_t M = G.size(0), C = G.size(1);
    need(kept && dX.size(1) == C && kept->numel() == M);
    const int32_t mode = whole32(a[3]), c = size32(C);
    const int32_t* ki = rows(kept);
    void *g = G.data_ptr(), *x = dX.data_ptr(), *st = stream();
    const int64_t g0 = G.stride(0), x0 = dX.stride(0), xs = dX.size(0);
    return call([=] { return lemo_scatter_grad(g, g0, ki, M, x, x0, xs, c, gt, xt, mode, st); });
}

PyObject* set_stream_source(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "set_stream_source(current_device, raw_stream)");
        return nullptr;
    }
    Py_XSETREF(current_device, Py_NewRef(a[0]));
    Py_XSETREF(raw_stream, Py_NewRef(a[1]));
    Py_RETURN_NONE;
}

#define LEMO_FAST(name, n) {#name, (PyCFunction)(void*)(guarded<n, name>), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {LEMO_FAST(score_segments, 9), LEMO_FAST(select_topk, 4), LEMO_FAST(kept_attention, 9), LEMO_FAST(gather_gemm, 6),
                         LEMO_FAST(gather_gemm_add, 7), LEMO_FAST(gather_gemm_dx, 4), LEMO_FAST(gather_gemm_dw, 5), LEMO_FAST(scatter_grad, 4),
                         {"set_stream_source", (PyCFunction)(void*)set_stream_source, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "lemo_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_lemo_native() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", LEMO_TORCH_VERSION) != 0) Py_CLEAR(m);  // (build.py)
    return m;
}
