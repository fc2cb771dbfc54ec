// The decode calls of the Python binding (kda.py), marshalled natively: a decode step of one sequence takes the device 4 us, and the
// checks, descriptors and ctypes of the general path 10 us of the host (measured in a loop of kda_recurrent_step, 1 sequence x 32
// heads: 9.9 us a call through kda.py alone, 4.2 to 5.0 here).
//
// Only calls that are regular in every respect are taken: plain contiguous device tensors of the expected types and shapes on
// one device.  For anything else, and for whatever cannot be told here, the functions return None, and kda.py's own path decides
// and words the error.  A status other than KDA_OK comes back as a number, which kda.py raises.  Nothing is kept between calls
// but the addresses of the library's entry points, and the entry points are handed over by kda.py, so that both ways call the
// same library.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "kda.h"

namespace {

decltype(&kda_recurrent_step) step_entry;
decltype(&kda_recurrent_steps) steps_entry;
PyObject *raw_stream;                                        // device index -> current stream, as a number

struct Irregular {};

// A tensor argument: exactly torch's own class, with memory of its own and nothing (vmap, a tracer) wrapped around it.
const at::Tensor &plain(PyObject *x)
{
    if (!THPVariable_CheckExact(x)) throw Irregular{};
    const at::Tensor &t = THPVariable_Unpack(x);
    using K = c10::DispatchKey;
    static const c10::DispatchKeySet wrapped({K::Python, K::PythonTLSSnapshot, K::Fake, K::Functionalize, K::FuncTorchBatched,
                                              K::FuncTorchGradWrapper, K::Conjugate, K::Negative, K::ZeroTensor});
    if (t.key_set().has_any(wrapped) || !t.has_storage()) throw Irregular{};
    return t;
}

struct Checked {
    c10::DeviceIndex device;
    explicit Checked(const at::Tensor &t) : device(t.device().index()) {}
    const at::Tensor &operator()(const at::Tensor &t, at::ScalarType type, at::IntArrayRef shape) const
    {
        if (!t.is_cuda() || t.device().index() != device || t.scalar_type() != type || t.sizes() != shape || !t.is_contiguous())
            throw Irregular{};
        return t;
    }
    const at::Tensor &operator()(PyObject *x, at::ScalarType type, at::IntArrayRef shape) const { return (*this)(plain(x), type, shape); }
};

float number(PyObject *x)
{
    if (PyFloat_CheckExact(x)) return (float)PyFloat_AS_DOUBLE(x);
    if (PyLong_CheckExact(x)) return (float)PyLong_AsDouble(x);
    throw Irregular{};
}

int code(at::ScalarType t)
{
    if (t == at::kFloat) return KDA_F32;
    if (t == at::kBFloat16) return KDA_BF16;
    throw Irregular{};
}

// o as the caller passed it, or a fresh one
at::Tensor output(PyObject *o, PyObject *out_dtype, const at::Tensor &v, const Checked &check)
{
    at::ScalarType type = at::kFloat;
    if (o != Py_None) type = plain(o).scalar_type();
    if (out_dtype != Py_None) {
        if (!THPDtype_Check(out_dtype)) throw Irregular{};
        const at::ScalarType asked = reinterpret_cast<THPDtype *>(out_dtype)->scalar_type;
        if (o != Py_None && asked != type) throw Irregular{};
        type = asked;
    }
    (void)code(type);
    if (o != Py_None) return check(o, type, v.sizes());
    return at::empty(v.sizes(), v.options().dtype(type));
}

void *stream_of(c10::DeviceIndex device)
{
    PyObject *index = PyLong_FromLong(device), *s = index ? PyObject_CallOneArg(raw_stream, index) : nullptr;
    Py_XDECREF(index);
    void *p = s ? PyLong_AsVoidPtr(s) : nullptr;
    Py_XDECREF(s);
    if (PyErr_Occurred()) { PyErr_Clear(); throw Irregular{}; }
    return p;
}

PyObject *finish(kda_status st, PyObject *o, const at::Tensor &out)
{
    if (st != KDA_OK) return PyLong_FromLong((long)st);
    if (o != Py_None) { Py_INCREF(o); return o; }
    return THPVariable_Wrap(out);
}

template <typename F> PyObject *guarded(F &&f)
{
    try {
        return f();
    } catch (...) {                                          // (whatever it was: kda.py meets it again, and says so)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

kda_dims decode_dims(int64_t N, int64_t tokens, int64_t H, int64_t dk, int64_t dv, int in, int out, float scale)
{
    if (N > 0x7fffffff || H > 0x7fffffff || dk > 0x7fffffff || dv > 0x7fffffff) throw Irregular{};
    kda_dims d{};
    d.batch = (int32_t)N; d.seqlen = tokens; d.heads = (int32_t)H; d.dk = (int32_t)dk; d.dv = (int32_t)dv; d.chunk = 64;
    d.num_seqs = (int32_t)N; d.in_dtype = (kda_dtype)in; d.out_dtype = (kda_dtype)out; d.scale = scale;
    return d;
}

// step(q, k, v, log_alpha, beta, S, scale, o, out_dtype)
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        if (n != 9 || !step_entry) throw Irregular{};
        const at::Tensor &q = plain(a[0]);
        if (q.dim() != 3) throw Irregular{};
        const at::Tensor &v = plain(a[2]);
        if (v.dim() != 3) throw Irregular{};
        const int64_t N = q.size(0), H = q.size(1), dk = q.size(2), dv = v.size(2);
        const at::ScalarType type = q.scalar_type();
        const Checked check(q);
        check(q, type, {N, H, dk});
        const at::Tensor &k = check(a[1], type, {N, H, dk});
        check(v, type, {N, H, dv});
        const at::Tensor &la = check(a[3], type, {N, H, dk}), &beta = check(a[4], type, {N, H});
        const at::Tensor &S = check(a[5], at::kFloat, {N, H, dk, dv});
        const int in = code(type);
        const float scale = number(a[6]);
        const at::Tensor o = output(a[7], a[8], v, check);
        const kda_dims d = decode_dims(N, 1, H, dk, dv, in, code(o.scalar_type()), scale);
        void *stream = stream_of(check.device);
        kda_status st;
        Py_BEGIN_ALLOW_THREADS
        st = step_entry(&d, q.data_ptr(), k.data_ptr(), v.data_ptr(), la.data_ptr(), beta.data_ptr(), static_cast<float *>(S.data_ptr()),
                        o.data_ptr(), stream);
        Py_END_ALLOW_THREADS
        return finish(st, a[7], o);
    });
}

// steps(q, k, v, log_alpha, beta, S_pool, state_indices, scale, o, out_dtype, form, l2norm_eps, a_scale, dt_bias, out_gate, norm_weight, rms_eps)
// form: 0 plain, 1 scalar gate, 2 fused stages with the prologue, 3 without
PyObject *steps(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        if (n != 17 || !steps_entry) throw Irregular{};
        const long form = PyLong_CheckExact(a[10]) ? PyLong_AsLong(a[10]) : -1;
        if (form < 0 || form > 3) throw Irregular{};
        const at::Tensor &q = plain(a[0]);
        if (q.dim() != 4) throw Irregular{};
        const at::Tensor &v = plain(a[2]);
        if (v.dim() != 4) throw Irregular{};
        const int64_t N = q.size(0), T = q.size(1), H = q.size(2), dk = q.size(3), dv = v.size(3);
        const at::ScalarType type = q.scalar_type();
        const Checked check(q);
        check(q, type, {N, T, H, dk});
        const at::Tensor &k = check(a[1], type, {N, T, H, dk});
        check(v, type, {N, T, H, dv});
        const at::Tensor &la = form == 1 ? check(a[3], type, {N, T, H}) : check(a[3], type, {N, T, H, dk});
        const at::Tensor &beta = check(a[4], type, {N, T, H}), &S = plain(a[5]);
        if (S.dim() != 4) throw Irregular{};
        check(S, at::kFloat, {S.size(0), H, dk, dv});
        const int32_t *indices = nullptr;
        if (a[6] != Py_None) indices = static_cast<const int32_t *>(check(a[6], at::kInt, {N}).data_ptr());
        else if (S.size(0) < N) throw Irregular{};
        const int in = code(type);
        const float scale = number(a[7]);
        kda_prologue pro{};
        kda_epilogue epi{};
        const bool gated = form >= 2 && a[14] != Py_None;
        if (form == 2) {
            pro.l2norm_eps = number(a[11]);
            if (a[12] != Py_None) pro.a_scale = static_cast<const float *>(check(a[12], at::kFloat, {H}).data_ptr());
            if (a[13] != Py_None) pro.dt_bias = static_cast<const float *>(check(a[13], at::kFloat, {H, dk}).data_ptr());
        }
        if (gated) {
            epi.rms_eps = number(a[16]);
            epi.gate = check(a[14], type, v.sizes()).data_ptr();
            if (a[15] != Py_None) epi.norm_weight = static_cast<const float *>(check(a[15], at::kFloat, {dv}).data_ptr());
        }
        const at::Tensor o = output(a[8], a[9], v, check);
        const kda_dims d = decode_dims(N, T, H, dk, dv, in, code(o.scalar_type()), scale);
        const uint32_t flags = (form == 1 ? KDA_STEPS_SCALAR_GATE : 0) | (a[8] == Py_None ? KDA_STEPS_ZERO_SKIPPED : 0);
        void *stream = stream_of(check.device);
        kda_status st;
        Py_BEGIN_ALLOW_THREADS
        st = steps_entry(&d, form == 2 ? &pro : nullptr, gated ? &epi : nullptr, q.data_ptr(), k.data_ptr(), v.data_ptr(), la.data_ptr(),
                         beta.data_ptr(), static_cast<float *>(S.data_ptr()), indices, o.data_ptr(), flags, stream);
        Py_END_ALLOW_THREADS
        return finish(st, a[8], o);
    });
}

// bind(address of kda_recurrent_step, address of kda_recurrent_steps, function from a device index to its current stream)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 3) { PyErr_SetString(PyExc_TypeError, "bind takes three arguments"); return nullptr; }
    void *one = PyLong_AsVoidPtr(a[0]), *many = PyLong_AsVoidPtr(a[1]);
    if (PyErr_Occurred()) return nullptr;
    step_entry = reinterpret_cast<decltype(step_entry)>(one);
    steps_entry = reinterpret_cast<decltype(steps_entry)>(many);
    Py_INCREF(a[2]);
    Py_XDECREF(raw_stream);
    raw_stream = a[2];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(bind)), METH_FASTCALL, nullptr},
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(step)), METH_FASTCALL, nullptr},
    {"steps", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(steps)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kda_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kda_host(void) { return PyModule_Create(&module); }
