// The accepting path of the binding's calls in native code: checks the tensors of a call and hands their
// pointers to the C ABI.  A decode step is a 5 us kernel; checking six tensors and marshalling thirteen
// arguments in Python took the host 9.
//
// Every function answers None when it does not take the call (an argument that is not a plain dense
// device tensor of the expected sizes, an option it does not know); the caller then goes through its own
// checks, which name what is wrong.  Nothing is kept between calls.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include <stddef.h>
#include <stdint.h>

namespace {

// addresses of the library's entry points, set once by bind()
typedef int (*step_fn)(const void *, const void *, const void *, float *, float *, void *, int, int, int, int, float, int, void *);
typedef int (*fwd_fn)(const void *, const void *, const void *, void *, float *, int, int, int, int, int, float, int, void *,
                      size_t, void *);
typedef int (*bwd_fn)(const void *, const void *, const void *, const void *, const float *, const void *, const void *, void *,
                      void *, void *, int, int, int, int, int, float, int, void *, size_t, void *);
typedef size_t (*ws_fn)(int, int, int, int, int, int);
step_fn g_step = nullptr;
// causal, causal token-major, non-causal, non-causal token-major; workspaces: causal, non-causal
fwd_fn g_fwd[4] = {};
bwd_fn g_bwd[4] = {};
ws_fn g_fwd_ws[2] = {}, g_bwd_ws[2] = {};

// a plain dense tensor on a device: no subclass, no wrapper of a transform, no mode's stand-in
const at::Tensor *plain(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    static const c10::DispatchKeySet wrappers{c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                              c10::DispatchKey::Functionalize, c10::DispatchKey::Python};
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.key_set().has_any(wrappers)) return nullptr;
    return t.is_contiguous() ? &t : nullptr;
}
// ... of these sizes, element type and device
const at::Tensor *like(PyObject *o, at::IntArrayRef sizes, at::ScalarType dt, const at::Device &dev) {
    const at::Tensor *t = plain(o);
    return t != nullptr && t->sizes() == sizes && t->scalar_type() == dt && t->device() == dev ? t : nullptr;
}
// element-type code of a call, -1: not taken here
int type_code(at::ScalarType dt, PyObject *features) {
    const int base = dt == at::kFloat ? 0 : dt == at::kBFloat16 ? 1 : -1;
    if (base < 0) return -1;
    return features == Py_False ? base : features == Py_True ? base + 2 : -1;
}
void *stream() { return c10::hip::getCurrentHIPStream().stream(); }
bool fits(const at::Tensor &t) {       // sizes the C ABI takes as int
    for (const int64_t n : t.sizes())
        if (n > 0x7fffffff) return false;
    return true;
}
PyObject *not_taken() { Py_RETURN_NONE; }

// step(q, k, v, S, z, out, eps, features) -> status
PyObject *py_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 8 || g_step == nullptr) return not_taken();
    const double eps = PyFloat_AsDouble(a[6]);
    if (eps == -1.0 && PyErr_Occurred()) return nullptr;
    int st;
    try {
        const at::Tensor *q = plain(a[0]), *v = plain(a[2]);
        if (q == nullptr || v == nullptr || q->dim() != 3 || v->dim() != 3 || !fits(*q) || !fits(*v)) return not_taken();
        const int64_t B = q->size(0), H = q->size(1), D = q->size(2), M = v->size(2);
        const at::ScalarType dt = q->scalar_type();
        const at::Device dev = q->device();
        const int code = type_code(dt, a[7]);
        const at::Tensor *k = like(a[1], q->sizes(), dt, dev), *out = like(a[5], v->sizes(), dt, dev);
        const at::Tensor *S = like(a[3], {B, H, D, M}, at::kFloat, dev), *z = like(a[4], {B, H, D}, at::kFloat, dev);
        if (code < 0 || k == nullptr || out == nullptr || S == nullptr || z == nullptr || v->size(0) != B || v->size(1) != H ||
            v->scalar_type() != dt || v->device() != dev)
            return not_taken();
        const void *pq = q->data_ptr(), *pk = k->data_ptr(), *pv = v->data_ptr();
        float *pS = static_cast<float *>(S->data_ptr()), *pz = static_cast<float *>(z->data_ptr());
        void *po = out->data_ptr(), *s = stream();
        Py_BEGIN_ALLOW_THREADS
        st = g_step(pq, pk, pv, pS, pz, po, (int)B, (int)H, (int)D, (int)M, (float)eps, code, s);
        Py_END_ALLOW_THREADS
    } catch (...) {
        return not_taken();
    }
    return PyLong_FromLong(st);
}

struct Sizes {
    int64_t B, H, N, D, M;
    at::ScalarType dt;
    at::Device dev = at::Device(at::kCPU);
    int code;
};
// Q, K, V of an N-sized call; kind & 1: token-major
bool inputs(int kind, PyObject *q, PyObject *k, PyObject *v, PyObject *features, Sizes &z, const at::Tensor *(&t)[3]) {
    t[0] = plain(q), t[2] = plain(v);
    if (t[0] == nullptr || t[2] == nullptr || t[0]->dim() != 4 || t[2]->dim() != 4 || !fits(*t[0]) || !fits(*t[2])) return false;
    z.dt = t[0]->scalar_type(), z.dev = t[0]->device();
    z.code = type_code(z.dt, features);
    z.B = t[0]->size(0), z.H = t[0]->size(kind & 1 ? 2 : 1), z.N = t[0]->size(kind & 1 ? 1 : 2), z.D = t[0]->size(3), z.M = t[2]->size(3);
    t[1] = like(k, t[0]->sizes(), z.dt, z.dev);
    return z.code >= 0 && t[1] != nullptr && t[2]->scalar_type() == z.dt && t[2]->device() == z.dev &&
           t[2]->sizes().slice(0, 3) == t[0]->sizes().slice(0, 3);
}
// a workspace: the caller's (any dense tensor on the device), or a new one
bool workspace(PyObject *o, size_t need, const Sizes &z, at::Tensor &ws) {
    if (o == Py_None) {
        ws = at::empty({(int64_t)(need > 16 ? need : 16)}, at::TensorOptions().dtype(at::kByte).device(z.dev));
        return true;
    }
    const at::Tensor *t = plain(o);
    if (t == nullptr || t->device() != z.dev) return false;
    ws = *t;
    return true;
}
PyObject *answer(int st, PyObject *given, const at::Tensor &ws) {
    if (st != 0) return PyLong_FromLong(st);
    if (given != Py_None) {
        Py_INCREF(given);
        return given;
    }
    return THPVariable_Wrap(ws);
}

// fwd(kind, Q, K, V, O, den | None, ws | None, eps, features) -> the workspace, or the status of a failed call
PyObject *py_fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 9) return not_taken();
    const long kind = PyLong_AsLong(a[0]);
    const double eps = PyFloat_AsDouble(a[7]);
    if (PyErr_Occurred()) return nullptr;
    if (kind < 0 || kind > 3 || g_fwd[kind] == nullptr) return not_taken();
    try {
        Sizes z;
        const at::Tensor *in[3], *den = nullptr;
        if (!inputs((int)kind, a[1], a[2], a[3], a[8], z, in)) return not_taken();
        const at::Tensor *O = like(a[4], in[2]->sizes(), z.dt, z.dev);
        if (a[5] != Py_None) den = like(a[5], {z.B, z.H, z.N}, at::kFloat, z.dev);
        if (O == nullptr || (a[5] != Py_None && den == nullptr)) return not_taken();
        at::Tensor ws;
        if (!workspace(a[6], g_fwd_ws[kind >> 1]((int)z.B, (int)z.H, (int)z.N, (int)z.D, (int)z.M, z.code), z, ws)) return not_taken();
        const void *q = in[0]->data_ptr(), *k = in[1]->data_ptr(), *v = in[2]->data_ptr();
        void *o = O->data_ptr(), *w = ws.data_ptr(), *s = stream();
        float *d = den != nullptr ? static_cast<float *>(den->data_ptr()) : nullptr;
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = g_fwd[kind](q, k, v, o, d, (int)z.B, (int)z.H, (int)z.N, (int)z.D, (int)z.M, (float)eps, z.code, w, ws.nbytes(), s);
        Py_END_ALLOW_THREADS
        return answer(st, a[6], ws);
    } catch (...) {
        return not_taken();
    }
}

// bwd(kind, Q, K, V, O | None, den, dO, dQ, dK, dV, ws | None, fwd_ws, eps, features) -> as fwd
PyObject *py_bwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 14) return not_taken();
    const long kind = PyLong_AsLong(a[0]);
    const double eps = PyFloat_AsDouble(a[12]);
    if (PyErr_Occurred()) return nullptr;
    if (kind < 0 || kind > 3 || g_bwd[kind] == nullptr || a[5] == Py_None || a[11] == Py_None) return not_taken();
    try {
        Sizes z;
        const at::Tensor *in[3];
        if (!inputs((int)kind, a[1], a[2], a[3], a[13], z, in)) return not_taken();
        const at::IntArrayRef qk = in[0]->sizes(), vv = in[2]->sizes();
        const at::Tensor *den = like(a[5], {z.B, z.H, z.N}, at::kFloat, z.dev), *g = like(a[6], vv, z.dt, z.dev);
        const at::Tensor *dq = like(a[7], qk, z.dt, z.dev), *dk = like(a[8], qk, z.dt, z.dev), *dv = like(a[9], vv, z.dt, z.dev);
        const at::Tensor *fws = plain(a[11]);
        if (den == nullptr || g == nullptr || dq == nullptr || dk == nullptr || dv == nullptr || fws == nullptr || fws->device() != z.dev ||
            (a[4] != Py_None && like(a[4], vv, z.dt, z.dev) == nullptr) ||
            fws->nbytes() < g_fwd_ws[kind >> 1]((int)z.B, (int)z.H, (int)z.N, (int)z.D, (int)z.M, z.code))
            return not_taken();
        at::Tensor ws;
        if (!workspace(a[10], g_bwd_ws[kind >> 1]((int)z.B, (int)z.H, (int)z.N, (int)z.D, (int)z.M, z.code), z, ws)) return not_taken();
        const void *q = in[0]->data_ptr(), *k = in[1]->data_ptr(), *v = in[2]->data_ptr(), *gp = g->data_ptr(), *fp = fws->data_ptr();
        const void *o = a[4] != Py_None ? THPVariable_Unpack(a[4]).data_ptr() : nullptr;
        const float *d = static_cast<const float *>(den->data_ptr());
        void *pq = dq->data_ptr(), *pk = dk->data_ptr(), *pv = dv->data_ptr(), *w = ws.data_ptr(), *s = stream();
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = g_bwd[kind](q, k, v, o, d, fp, gp, pq, pk, pv, (int)z.B, (int)z.H, (int)z.N, (int)z.D, (int)z.M, (float)eps, z.code, w,
                         ws.nbytes(), s);
        Py_END_ALLOW_THREADS
        return answer(st, a[10], ws);
    } catch (...) {
        return not_taken();
    }
}

// bind([13 addresses]): step, fwd x 4, bwd x 4, fwd_ws x 2, bwd_ws x 2
PyObject *py_bind(PyObject *, PyObject *list) {
    if (!PyList_Check(list) || PyList_GET_SIZE(list) != 13) {
        PyErr_SetString(PyExc_ValueError, "13 addresses expected");
        return nullptr;
    }
    void *p[13];
    for (int i = 0; i < 13; ++i) {
        p[i] = PyLong_AsVoidPtr(PyList_GET_ITEM(list, i));
        if (PyErr_Occurred()) return nullptr;
    }
    g_step = reinterpret_cast<step_fn>(p[0]);
    for (int i = 0; i < 4; ++i) g_fwd[i] = reinterpret_cast<fwd_fn>(p[1 + i]), g_bwd[i] = reinterpret_cast<bwd_fn>(p[5 + i]);
    for (int i = 0; i < 2; ++i) g_fwd_ws[i] = reinterpret_cast<ws_fn>(p[9 + i]), g_bwd_ws[i] = reinterpret_cast<ws_fn>(p[11 + i]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_step)), METH_FASTCALL, nullptr},
    {"fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_fwd)), METH_FASTCALL, nullptr},
    {"bwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_bwd)), METH_FASTCALL, nullptr},
    {"bind", py_bind, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
