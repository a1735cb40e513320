// The decode step's call from Python: argument checks, output allocation and the call of the C entry point in one native
// function.  A generation step at batch 1 is two launches (2.5 us each on the host, 5.6 us on the GPU), and marshalling through
// Python objects and ctypes took longer than both: 13.1 us a step.
//
// The function takes the plain case only -- ordinary contiguous GPU tensors of matching shapes and types, no tracing,
// vmap or dispatch mode in force -- and returns None for everything else, which api.py then handles (and reports) itself.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <algorithm>

#define GSA_STR2(x) #x
#define GSA_STR(x) GSA_STR2(x)

namespace {

using DecodeFn = int (*)(int32_t, int32_t, int32_t, int32_t, int32_t, int32_t, float, int32_t, float, int32_t, const void *,
                         const void *, const void *, const float *, const float *, float *, float *, void *, void *, size_t,
                         void *);   // gsa_decode_step_ex

// An ordinary dense GPU tensor (or parameter), or NULL.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    constexpr c10::DispatchKeySet special({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                           c10::DispatchKey::Functionalize, c10::DispatchKey::Negative, c10::DispatchKey::Conjugate,
                                           c10::DispatchKey::ZeroTensor});
    if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || t.key_set().has_any(special) || !t.has_storage()) return nullptr;
    return t.is_contiguous() ? &t : nullptr;
}

bool is(const at::Tensor *t, at::ScalarType type, std::initializer_list<int64_t> shape)
{
    return t && t->scalar_type() == type && t->sizes() == at::IntArrayRef(shape);
}

bool modes_in_force()
{
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Tracer) ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Functionalize);
}

// decode_step(entry, stream_of, q, k, v, g, K, V, scale, out, workspace, s, readout, gate_tau, feature_map)
//   entry: address of gsa_decode_step_ex; stream_of(device index): handle of the current stream
// -> the output tensor, the status code (an int) if the entry point returned an error, or None: not the plain case.
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 15) {
        PyErr_SetString(PyExc_TypeError, "decode_step takes 15 arguments");
        return nullptr;
    }
    HANDLE_TH_ERRORS   // C++ exceptions leave as the Python exceptions torch gives them
    if (modes_in_force()) Py_RETURN_NONE;
    const at::Tensor *q = plain(a[2]), *k = plain(a[3]), *v = plain(a[4]), *g = plain(a[5]), *K = plain(a[6]), *V = plain(a[7]);
    if (!q || !v || !g || q->dim() != 3 || v->dim() != 3 || g->dim() != 3) Py_RETURN_NONE;
    const at::ScalarType type = q->scalar_type();
    const int64_t B = q->size(0), H = q->size(1), dk = q->size(2), dv = v->size(2), m = g->size(2);
    if (type != at::kFloat && type != at::kBFloat16) Py_RETURN_NONE;
    if (std::max({B, H, dk, dv, m}) > INT32_MAX) Py_RETURN_NONE;
    if (!is(k, type, {B, H, dk}) || !is(v, type, {B, H, dv}) || !is(g, at::kFloat, {B, H, m}) ||
        !is(K, at::kFloat, {B, H, m, dk}) || !is(V, at::kFloat, {B, H, m, dv}))
        Py_RETURN_NONE;
    const at::Tensor *out = nullptr, *ws = nullptr, *s = nullptr;
    if (a[9] != Py_None && !is(out = plain(a[9]), type, {B, H, dv})) Py_RETURN_NONE;
    if (a[10] != Py_None && (!(ws = plain(a[10])) || ws->scalar_type() != at::kByte || ws->numel() == 0)) Py_RETURN_NONE;
    if (a[11] != Py_None && !is(s = plain(a[11]), at::kFloat, {B, H, m})) Py_RETURN_NONE;
    const double scale = PyFloat_AsDouble(a[8]), tau = PyFloat_AsDouble(a[13]);
    const long readout = PyLong_AsLong(a[12]), feature = PyLong_AsLong(a[14]);
    const auto entry = reinterpret_cast<DecodeFn>(PyLong_AsVoidPtr(a[0]));
    if (PyErr_Occurred() || !entry) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    PyObject *index = PyLong_FromLong(q->get_device());
    PyObject *handle = index ? PyObject_CallOneArg(a[1], index) : nullptr;
    Py_XDECREF(index);
    if (!handle) return nullptr;
    void *stream = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (PyErr_Occurred()) return nullptr;
    at::Tensor o = out ? *out : at::empty_like(*v);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = entry((int32_t)B, (int32_t)H, (int32_t)dk, (int32_t)dv, (int32_t)m, type == at::kBFloat16 ? 1 : 0, (float)scale,
               (int32_t)readout, (float)tau, (int32_t)feature, q->data_ptr(), k->data_ptr(), v->data_ptr(),
               static_cast<const float *>(g->data_ptr()), s ? static_cast<const float *>(s->data_ptr()) : nullptr,
               static_cast<float *>(K->data_ptr()), static_cast<float *>(V->data_ptr()), o.data_ptr(),
               ws ? ws->data_ptr() : nullptr, ws ? (size_t)ws->numel() : 0, stream);
    Py_END_ALLOW_THREADS
    if (rc != 0) return PyLong_FromLong(rc);
    if (out) {
        Py_INCREF(a[9]);
        return a[9];
    }
    return THPVariable_Wrap(std::move(o));
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(decode_step)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the versions of torch and Python whose headers this was compiled against; the loader compares them with its own.
PyMODINIT_FUNC PyInit__binding(void)
{
    PyObject *m = PyModule_Create(&module);
    PyObject *built = m ? Py_BuildValue("(ss)", TORCH_VERSION, GSA_STR(PY_MAJOR_VERSION) "." GSA_STR(PY_MINOR_VERSION)) : nullptr;
    if (!built || PyModule_AddObject(m, "built_for", built) < 0) {   // takes the reference when it succeeds
        Py_XDECREF(built);
        Py_XDECREF(m);
        return nullptr;
    }
    return m;
}
