// The marshalling of flashd.py's three entry points of the serving path in C++: from the tensors
// to the C call, a call costs 0.4 us of host time here and 3.5 in Python, of which a call on a
// small problem takes 2.5 us more for the launch and the GPU not much longer.
//
// Each function returns the status of the C call, or None where it finds anything out of the ordinary
// (an argument that is no plain GPU tensor of the right type and shape, another current device, a
// stream handed in): nothing has been enqueued then, and the Python form of the same function takes the
// call, with all its checks and messages.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using attn_fwd_t = int (*)(const void*, const void*, const void*, void*, int, int, int, int, int, int, int, float,
                           int, void*);
using attn_fwd_kv8_t = int (*)(const void*, const void*, const void*, void*, int, int, int, int, int, int, int,
                               float, float, float, int, void*);
using attn_fwd_state_t = int (*)(const void*, const void*, const void*, void*, const float*, float*, int, int, int,
                                 int, int, int, int, int, float, int, void*);

attn_fwd_t g_attn_fwd = nullptr;
attn_fwd_kv8_t g_attn_fwd_kv8 = nullptr;
attn_fwd_state_t g_attn_fwd_state = nullptr;
PyObject* g_current_device = nullptr;       // () -> index
PyObject* g_raw_stream = nullptr;           // (index) -> handle

// A plain contiguous GPU tensor of four dimensions, or nullptr
const at::Tensor* plain(PyObject* x) {
    if (!THPVariable_CheckExact(x)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(x);
    return t.is_cuda() && t.layout() == at::kStrided && t.dim() == 4 && t.is_contiguous() ? &t : nullptr;
}

// the library's number of a storage type, or -1
int dtype_of(const at::Tensor& t) {
    switch (t.scalar_type()) {
    case at::kFloat: return 0;
    case at::kHalf: return 1;
    case at::kBFloat16: return 2;
    default: return -1;
    }
}

struct Shape { int B, Hq, Hkv, Lq, Lk, d; };

// (sizes that do not fit the C call's ints go to the Python form, which passes them as it always has)
bool shape_of(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, Shape& s) {
    const auto qs = q.sizes(), ks = k.sizes();
    if (qs[0] != ks[0] || qs[3] != ks[3] || v.sizes() != ks) return false;
    for (const int64_t n : {qs[0], qs[1], qs[2], qs[3], ks[1], ks[2]})
        if (n > 0x7fffffff) return false;
    s = {(int)qs[0], (int)qs[1], (int)ks[1], (int)qs[2], (int)ks[2], (int)qs[3]};
    return true;
}

// The handle of the current stream of q's device, which must be the current one.
bool current_stream(const at::Tensor& q, void** stream) {
    PyObject* now = PyObject_CallNoArgs(g_current_device);
    if (now == nullptr) return false;
    const bool here = PyLong_AsLong(now) == q.get_device();
    PyObject* raw = here ? PyObject_CallOneArg(g_raw_stream, now) : nullptr;
    Py_DECREF(now);
    if (raw == nullptr) return false;
    *stream = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    return PyErr_Occurred() == nullptr;
}

bool number(PyObject* x, float* out) {
    const double v = PyFloat_AsDouble(x);
    *out = (float)v;
    return !(v == -1.0 && PyErr_Occurred());
}

PyObject* other_form() {
    PyErr_Clear();
    Py_RETURN_NONE;
}

// (q, k, v, o, causal, scale)
PyObject* py_attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        if (n != 6) return other_form();
        const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *v = plain(a[2]), *o = plain(a[3]);
        Shape s;
        float scale;
        void* stream;
        if (!q || !k || !v || !o || !shape_of(*q, *k, *v, s) || o->sizes() != q->sizes()) return other_form();
        const int dt = dtype_of(*q);
        if (dt < 0 || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type() ||
            o->scalar_type() != q->scalar_type())
            return other_form();
        const int causal = PyObject_IsTrue(a[4]);
        if (causal < 0 || !number(a[5], &scale) || !current_stream(*q, &stream)) return other_form();
        void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr(), *op = o->data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_attn_fwd(qp, kp, vp, op, s.B, s.Hq, s.Hkv, s.Lq, s.Lk, s.d, causal, scale, dt, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (...) {
        return other_form();
    }
}

// (q, k8, v8, o, causal, scale, kscale, vscale)
PyObject* py_attn_fwd_kv8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        if (n != 8) return other_form();
        const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *v = plain(a[2]), *o = plain(a[3]);
        Shape s;
        float scale, kscale, vscale;
        void* stream;
        if (!q || !k || !v || !o || !shape_of(*q, *k, *v, s) || o->sizes() != q->sizes()) return other_form();
        const int dt = dtype_of(*q);
        if (dt < 1 || o->scalar_type() != q->scalar_type() || k->scalar_type() != at::kFloat8_e4m3fn ||
            v->scalar_type() != at::kFloat8_e4m3fn)
            return other_form();
        const int causal = PyObject_IsTrue(a[4]);
        if (causal < 0 || !number(a[5], &scale) || !number(a[6], &kscale) || !number(a[7], &vscale) ||
            !current_stream(*q, &stream))
            return other_form();
        void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr(), *op = o->data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_attn_fwd_kv8(qp, kp, vp, op, s.B, s.Hq, s.Hkv, s.Lq, s.Lk, s.d, causal, scale, kscale, vscale, dt,
                            stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (...) {
        return other_form();
    }
}

// (q, k, v, causal, scale, o, state_in, state_out, causal_shift), the last four or None
PyObject* py_attn_fwd_state(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        if (n != 9) return other_form();
        const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *v = plain(a[2]);
        const at::Tensor* out[3] = {nullptr, nullptr, nullptr};      // o, state_in, state_out
        Shape s;
        float scale;
        void* stream;
        if (!q || !k || !v || !shape_of(*q, *k, *v, s)) return other_form();
        const int dt = dtype_of(*q);
        if (dt < 0 || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type())
            return other_form();
        for (int i = 0; i < 3; ++i) {
            if (a[5 + i] == Py_None) continue;
            out[i] = plain(a[5 + i]);
            if (out[i] == nullptr) return other_form();
            const auto z = out[i]->sizes();
            if (z[0] != s.B || z[1] != s.Hq || z[2] != s.Lq || z[3] != s.d + (i > 0 ? 2 : 0) ||
                out[i]->scalar_type() != (i > 0 ? at::kFloat : q->scalar_type()))
                return other_form();
        }
        int shift = s.Lk - s.Lq;
        if (a[8] != Py_None) {
            const long x = PyLong_AsLong(a[8]);
            if ((x == -1 && PyErr_Occurred()) || x != (int)x) return other_form();
            shift = (int)x;
        }
        const int causal = PyObject_IsTrue(a[3]);
        if (causal < 0 || !number(a[4], &scale) || !current_stream(*q, &stream)) return other_form();
        void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
        void* op[3];
        for (int i = 0; i < 3; ++i) op[i] = out[i] ? out[i]->data_ptr() : nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_attn_fwd_state(qp, kp, vp, op[0], (const float*)op[1], (float*)op[2], s.B, s.Hq, s.Hkv, s.Lq, s.Lk,
                              s.d, causal, shift, scale, dt, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (...) {
        return other_form();
    }
}

// (address of flashd_attn_fwd, _kv8, _state, current-device function, raw-stream function)
PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "bind takes three addresses and two functions");
        return nullptr;
    }
    void* f[3];
    for (int i = 0; i < 3; ++i) f[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
    g_attn_fwd = reinterpret_cast<attn_fwd_t>(f[0]);
    g_attn_fwd_kv8 = reinterpret_cast<attn_fwd_kv8_t>(f[1]);
    g_attn_fwd_state = reinterpret_cast<attn_fwd_state_t>(f[2]);
    Py_INCREF(a[3]);
    Py_XSETREF(g_current_device, a[3]);
    Py_INCREF(a[4]);
    Py_XSETREF(g_raw_stream, a[4]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_bind)), METH_FASTCALL, nullptr},
    {"attn_fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_attn_fwd)), METH_FASTCALL, nullptr},
    {"attn_fwd_kv8", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_attn_fwd_kv8)), METH_FASTCALL,
     nullptr},
    {"attn_fwd_state", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_attn_fwd_state)), METH_FASTCALL,
     nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_flashd_binding", nullptr, -1, methods, nullptr, nullptr, nullptr,
                      nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__flashd_binding() {
    PyObject* m = PyModule_Create(&module);
    // tensors are read through torch's C++ headers, so another version's may not be handed in
    // (FLASHD_TORCH: torch.__version__ at the build)
    const char* built_for =
        "torch " FLASHD_TORCH " and Python " Py_STRINGIFY(PY_MAJOR_VERSION) "." Py_STRINGIFY(PY_MINOR_VERSION);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", built_for) != 0) Py_CLEAR(m);
    return m;
}
