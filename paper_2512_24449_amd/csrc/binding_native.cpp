// The calls of a decode step and of an append, marshalled in C++: binding.PackedKVCache tries these first.  A call whose
// arguments are not exactly what it expects (plain tensors of the right type, shape and layout) is answered with
// NotImplemented and made again by the Python code, which has the checks and raises the errors.
//
// A step of a small cache launches a few kernels of a few microseconds each, and marshalling through ctypes (1.3 us a call), checking shapes in Python (about 1)
// and torch.empty (1.5) took as long as they do.  Three steps over one
// stream of 1000 tokens 21.6 -> 18.0 us, over eight of 2296 24.8 -> 19.1; fused attention over eight of 650 13.2 -> 11.8.
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/Exceptions.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include <cstdint>
#include <cstring>
#include <string>

namespace {

// The library's entry points, by address (the library itself is loaded by binding.py), and what binding.py lends.
struct Library {
    int (*append)(void *, const void *, const void *, int32_t, void *);
    int (*append_bf16)(void *, const void *, const void *, int32_t, void *);
    int (*k_matvec)(void *, const void *, float, float *, int64_t, void *);
    int (*softmax)(void *, float *, int64_t, void *);
    int (*v_matvec)(void *, const float *, int64_t, float *, void *);
    int (*attention)(void *, const void *, float, float *, void *);
    int (*restore)(void *, int64_t);
    int (*release)(void *, void *);
    int64_t (*tokens)(const void *);
} lib;
PyObject *check_code, *get_device, *get_stream, *in_bad_fork;

constexpr int64_t HEAD_DIM = 128;

struct Calls {
    PyObject_HEAD
    void *handle;
    int64_t batch, kv_heads, q_heads;
    c10::Device device;
};

PyObject *slow() { Py_RETURN_NOTIMPLEMENTED; }

// The hipStream_t meant by a `stream` argument: torch's current stream for None, or an integer.
bool stream_of(PyObject *stream, void *&out) {
    if (stream == Py_None) {
        PyObject *bad = PyObject_CallNoArgs(in_bad_fork);
        const bool fine = bad == Py_False;
        Py_XDECREF(bad);
        PyObject *device = fine ? PyObject_CallNoArgs(get_device) : nullptr;
        PyObject *raw = device ? PyObject_CallOneArg(get_stream, device) : nullptr;
        Py_XDECREF(device);
        if (raw) out = PyLong_AsVoidPtr(raw);
        Py_XDECREF(raw);
        if (!PyErr_Occurred()) return raw != nullptr;
        PyErr_Clear();
        return false;
    }
    if (!PyLong_CheckExact(stream)) return false;
    out = PyLong_AsVoidPtr(stream);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

bool scale_of(PyObject *o, float &out) {
    if (!PyFloat_CheckExact(o)) return false;
    out = float(PyFloat_AS_DOUBLE(o));
    return true;
}

// Function and dispatch modes (tracing, fake tensors, ...) see what the Python code calls.
bool modes() { return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set(); }

bool plain(PyObject *o, c10::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.layout() == c10::kStrided && t.scalar_type() == type && t.is_contiguous();
}

bool rows(const at::Tensor &t, int64_t a, int64_t b) { return t.dim() == 3 && t.size(0) == a && t.size(1) == b; }

// `code` of the library as `result` (a new reference), or the error binding.py raises for it.
PyObject *answer(int code, const char *what, PyObject *result) {
    if (code == 0) return result;
    Py_XDECREF(result);
    PyObject *none = PyObject_CallFunction(check_code, "is", code, what);
    Py_XDECREF(none);
    if (none) PyErr_SetString(PyExc_RuntimeError, what);
    return nullptr;
}

template <class F>
int unlocked(F call) {   // as ctypes does: other Python threads run meanwhile
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = call();
    Py_END_ALLOW_THREADS
    return code;
}

at::Tensor new_floats(const Calls *c, int64_t last) {
    return at::empty({c->batch, c->q_heads, last}, at::TensorOptions().dtype(at::kFloat).device(c->device));
}

PyObject *append(Calls *c, PyObject *const *args, Py_ssize_t n) {   // k_new, v_new, stream
    HANDLE_TH_ERRORS
    void *s;
    if (n != 3 || !c->handle || modes() || !THPVariable_CheckExact(args[0])) return slow();
    const c10::ScalarType type = THPVariable_Unpack(args[0]).scalar_type();
    if ((type != at::kHalf && type != at::kBFloat16) || !plain(args[0], type) || !plain(args[1], type)) return slow();
    const at::Tensor &k = THPVariable_Unpack(args[0]), &v = THPVariable_Unpack(args[1]);
    if (k.dim() != 4 || k.sizes() != v.sizes() || k.size(0) != c->batch || k.size(2) != c->kv_heads || k.size(3) != HEAD_DIM ||
        k.size(1) > INT32_MAX || !stream_of(args[2], s))
        return slow();
    const void *kp = k.data_ptr(), *vp = v.data_ptr();
    const int32_t tokens = int32_t(k.size(1));
    const bool bf16 = type == at::kBFloat16;
    const int code = unlocked([&] { return (bf16 ? lib.append_bf16 : lib.append)(c->handle, kp, vp, tokens, s); });
    return answer(code, bf16 ? "kv_compress_append_bf16" : "kv_compress_append", Py_NewRef(Py_None));
    END_HANDLE_TH_ERRORS
}

PyObject *k_matvec(Calls *c, PyObject *const *args, Py_ssize_t n) {   // q, sm_scale, scores, stream
    HANDLE_TH_ERRORS
    void *s;
    float scale;
    if (n != 4 || !c->handle || modes() || !plain(args[0], at::kHalf) || !scale_of(args[1], scale)) return slow();
    const at::Tensor &q = THPVariable_Unpack(args[0]);
    if (!rows(q, c->batch, c->q_heads) || q.size(2) != HEAD_DIM) return slow();
    const bool fresh = args[2] == Py_None;
    if ((!fresh && (!plain(args[2], at::kFloat) || THPVariable_Unpack(args[2]).dim() != 3)) || !stream_of(args[3], s)) return slow();
    const at::Tensor scores = fresh ? new_floats(c, lib.tokens(c->handle)) : THPVariable_Unpack(args[2]);
    const void *qp = q.data_ptr();
    float *sp = static_cast<float *>(scores.data_ptr());
    const int64_t ld = scores.size(2);
    const int code = unlocked([&] { return lib.k_matvec(c->handle, qp, scale, sp, ld, s); });
    return answer(code, "kv_k_matvec", fresh ? THPVariable_Wrap(scores) : Py_NewRef(args[2]));
    END_HANDLE_TH_ERRORS
}

PyObject *softmax(Calls *c, PyObject *const *args, Py_ssize_t n) {   // scores, stream
    HANDLE_TH_ERRORS
    void *s;
    if (n != 2 || !c->handle || modes() || !plain(args[0], at::kFloat)) return slow();
    const at::Tensor &t = THPVariable_Unpack(args[0]);
    if (!rows(t, c->batch, c->q_heads) || !stream_of(args[1], s)) return slow();
    float *p = static_cast<float *>(t.data_ptr());
    const int64_t ld = t.size(2);
    const int code = unlocked([&] { return lib.softmax(c->handle, p, ld, s); });
    return answer(code, "kv_softmax", Py_NewRef(args[0]));
    END_HANDLE_TH_ERRORS
}

PyObject *v_matvec(Calls *c, PyObject *const *args, Py_ssize_t n) {   // p, stream; the output is new
    HANDLE_TH_ERRORS
    void *s;
    if (n != 2 || !c->handle || modes() || !plain(args[0], at::kFloat)) return slow();
    const at::Tensor &t = THPVariable_Unpack(args[0]);
    if (!rows(t, c->batch, c->q_heads) || !stream_of(args[1], s)) return slow();
    const at::Tensor out = new_floats(c, HEAD_DIM);
    const float *p = static_cast<const float *>(t.data_ptr());
    float *o = static_cast<float *>(out.data_ptr());
    const int64_t ld = t.size(2);
    const int code = unlocked([&] { return lib.v_matvec(c->handle, p, ld, o, s); });
    return answer(code, "kv_v_matvec", THPVariable_Wrap(out));
    END_HANDLE_TH_ERRORS
}

PyObject *attention(Calls *c, PyObject *const *args, Py_ssize_t n) {   // q, sm_scale, stream; the output is new
    HANDLE_TH_ERRORS
    void *s;
    float scale;
    if (n != 3 || !c->handle || modes() || !plain(args[0], at::kHalf) || !scale_of(args[1], scale)) return slow();
    const at::Tensor &q = THPVariable_Unpack(args[0]);
    if (!rows(q, c->batch, c->q_heads) || q.size(2) != HEAD_DIM || !stream_of(args[2], s)) return slow();
    const at::Tensor out = new_floats(c, HEAD_DIM);
    const void *qp = q.data_ptr();
    float *o = static_cast<float *>(out.data_ptr());
    const int code = unlocked([&] { return lib.attention(c->handle, qp, scale, o, s); });
    return answer(code, "kv_decode_attention", THPVariable_Wrap(out));
    END_HANDLE_TH_ERRORS
}

PyObject *restore(Calls *c, PyObject *tokens) {
    if (!c->handle || !PyLong_CheckExact(tokens)) return slow();
    int overflow;
    const long long t = PyLong_AsLongLongAndOverflow(tokens, &overflow);
    if (overflow) return slow();
    return answer(lib.restore(c->handle, t), "kv_cache_restore", Py_NewRef(Py_None));
}

PyObject *release(Calls *c, PyObject *stream) {
    void *s;
    if (!c->handle || !stream_of(stream, s)) return slow();
    return answer(unlocked([&] { return lib.release(c->handle, s); }), "kv_cache_release", Py_NewRef(Py_None));
}

PyObject *set_handle(Calls *c, PyObject *value) {   // an address, 0: every call takes the Python code
    void *h = PyLong_AsVoidPtr(value);
    if (PyErr_Occurred()) return nullptr;
    c->handle = h;
    Py_RETURN_NONE;
}

PyObject *calls_new(PyTypeObject *type, PyObject *args, PyObject *) {
    HANDLE_TH_ERRORS
    long long batch, kv_heads, q_heads;
    const char *device;
    if (!PyArg_ParseTuple(args, "LLLs", &batch, &kv_heads, &q_heads, &device)) return nullptr;
    const c10::Device d{std::string(device)};
    Calls *c = reinterpret_cast<Calls *>(type->tp_alloc(type, 0));
    if (!c) return nullptr;
    c->handle = nullptr;
    c->batch = batch, c->kv_heads = kv_heads, c->q_heads = q_heads;
    c->device = d;
    return reinterpret_cast<PyObject *>(c);
    END_HANDLE_TH_ERRORS
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef calls_methods[] = {
    FAST(append), FAST(k_matvec), FAST(softmax), FAST(v_matvec), FAST(attention),
    {"restore", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(restore)), METH_O, nullptr},
    {"release", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(release)), METH_O, nullptr},
    {"set_handle", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(set_handle)), METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// bind(addresses of the entry points in Library's order, _check, device getter, stream getter, bad-fork test)
PyObject *bind(PyObject *, PyObject *args) {
    PyObject *addresses, *check, *device, *stream, *fork;
    if (!PyArg_ParseTuple(args, "O!OOOO", &PyTuple_Type, &addresses, &check, &device, &stream, &fork)) return nullptr;
    constexpr Py_ssize_t COUNT = sizeof(Library) / sizeof(void *);
    if (PyTuple_GET_SIZE(addresses) != COUNT) return PyErr_SetString(PyExc_ValueError, "bind: wrong number of entry points"), nullptr;
    void *at[COUNT];
    for (Py_ssize_t i = 0; i < COUNT; ++i) at[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (PyErr_Occurred()) return nullptr;
    memcpy(&lib, at, sizeof(lib));
    PyObject **const lent[] = {&check_code, &get_device, &get_stream, &in_bad_fork};
    PyObject *const given[] = {check, device, stream, fork};
    for (int i = 0; i < 4; ++i) {
        Py_XDECREF(*lent[i]);
        *lent[i] = Py_NewRef(given[i]);
    }
    Py_RETURN_NONE;
}

PyMethodDef module_methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Marshalling of binding.py's frequent calls.", -1, module_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    calls_type.tp_name = "paper_2512_24449_amd._native.Calls";
    calls_type.tp_basicsize = sizeof(Calls);
    calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
    calls_type.tp_new = calls_new;
    calls_type.tp_methods = calls_methods;
    if (PyType_Ready(&calls_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddObject(m, "Calls", Py_NewRef(reinterpret_cast<PyObject *>(&calls_type))) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
