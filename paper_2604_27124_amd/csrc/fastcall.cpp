// The plain calls of binding.py in native code: checks, outputs and the launch of one call on ordinary tensors, current
// stream, outputs allocated here.  Any other call, and any that the checks or the library refuse, gives None, and the
// Python function behind it does what it always did (and raises what it always raised).
//
// A small call is bound by this work: two calls of a training step on two 256-token sequences take 12.7 us on the GPU.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <cstdint>

namespace {

typedef int (*FwdFn)(const void *, const void *, const void *, void *, const int32_t *, const float *, float, int, int, int, int, void *);
typedef int (*BwdFn)(const void *, const void *, const void *, const void *, void *, void *, void *, const int32_t *, const float *, float,
                     int, int, int, int, void *, size_t, void *);
typedef size_t (*BytesFn)(int, int, int, int);

FwdFn fwd_fn;
BwdFn bwd_fn;
BytesFn bytes_fn;

// An ordinary GPU tensor: exactly torch.Tensor, and nothing that a transform or a mode of torch has wrapped.
bool plain(PyObject *o, at::Tensor &t) {
    if (!THPVariable_CheckExact(o)) return false;
    t = THPVariable_Unpack(o);
    const auto keys = t.unsafeGetTensorImpl()->key_set();
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided &&
           !keys.has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                              c10::DispatchKey::Functionalize, c10::DispatchKey::Batched, c10::DispatchKey::Negative,
                                              c10::DispatchKey::Conjugate, c10::DispatchKey::ZeroTensor}));
}

bool rows(PyObject *o, at::Tensor &t, const at::Tensor *like) {
    return plain(o, t) && t.scalar_type() == at::kBFloat16 && t.is_contiguous() && t.dim() == 4 && (!like || t.sizes() == like->sizes());
}

bool vec(PyObject *o, at::Tensor &t, int64_t n, at::ScalarType type) {
    return plain(o, t) && t.scalar_type() == type && t.is_contiguous() && t.dim() == 1 && t.size(0) == n;
}

bool ordinary_state() {            // no mode that would want to see the calls of the Python function
    return !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled() &&
           !c10::impl::tls_local_dispatch_key_set().included_.has_any(c10::DispatchKeySet({c10::DispatchKey::FuncTorchDynamicLayerFrontMode, c10::DispatchKey::Functionalize, c10::DispatchKey::Python}));
}

struct Call {
    at::Tensor q, k, v, g, seqlens, bias;
    float scale;
    int B, N, H, d;
};

// q, k, v, [d_o,] seqlens, bias, scale
bool read(PyObject *const *args, Py_ssize_t n, bool backward, Call &c) {
    if (n != (backward ? 7 : 6) || !ordinary_state()) return false;
    const int m = backward ? 4 : 3;
    if (!rows(args[0], c.q, nullptr) || !rows(args[1], c.k, &c.q) || !rows(args[2], c.v, &c.q)) return false;
    if (backward && !rows(args[3], c.g, &c.q)) return false;
    for (int i = 0; i < 4; ++i)
        if (c.q.size(i) > INT32_MAX) return false;
    c.B = (int)c.q.size(0); c.N = (int)c.q.size(1); c.H = (int)c.q.size(2); c.d = (int)c.q.size(3);
    if (!vec(args[m], c.seqlens, c.B, at::kInt) || !vec(args[m + 1], c.bias, c.B, at::kFloat)) return false;
    if (!PyFloat_CheckExact(args[m + 2])) return false;
    c.scale = (float)PyFloat_AS_DOUBLE(args[m + 2]);
    return true;
}

void *current_stream() { return static_cast<void *>(c10::hip::getCurrentHIPStream().stream()); }

template <class T>
T *data(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }

PyObject *none() {                 // with no Python error behind it, which what threw may have left
    PyErr_Clear();
    Py_RETURN_NONE;
}

struct WithoutGil {                // other threads of the interpreter run while memory is found and the launch is made
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

PyObject *fwd(PyObject *, PyObject *const *args, Py_ssize_t n) {
    try {
        Call c;
        if (!fwd_fn || !read(args, n, false, c)) return none();
        at::Tensor o;
        int rc;
        {
            WithoutGil released;
            o = at::empty_like(c.q);
            rc = fwd_fn(data<void>(c.q), data<void>(c.k), data<void>(c.v), data<void>(o), data<int32_t>(c.seqlens), data<float>(c.bias),
                        c.scale, c.B, c.N, c.H, c.d, current_stream());
        }
        return rc ? none() : THPVariable_Wrap(std::move(o));
    } catch (...) {                // out of memory and the like: the Python function meets it again and reports it
        return none();
    }
}

PyObject *bwd(PyObject *, PyObject *const *args, Py_ssize_t n) {
    try {
        Call c;
        if (!bwd_fn || !bytes_fn || !read(args, n, true, c)) return none();
        const size_t need = bytes_fn(c.B, c.N, c.H, c.d);
        if (need && c.q.get_device() != c10::hip::current_device()) return none();   // scratch belongs to a stream of its own device
        at::Tensor dq, dk, dv, ws;
        int rc;
        {
            WithoutGil released;
            dq = at::empty_like(c.q);
            dk = at::empty_like(c.q);
            dv = at::empty_like(c.q);
            if (need) ws = at::empty({(int64_t)need}, c.q.options().dtype(at::kByte).requires_grad(false));
            rc = bwd_fn(data<void>(c.q), data<void>(c.k), data<void>(c.v), data<void>(c.g), data<void>(dq), data<void>(dk), data<void>(dv),
                        data<int32_t>(c.seqlens), data<float>(c.bias), c.scale, c.B, c.N, c.H, c.d, need ? data<void>(ws) : nullptr,
                        need, current_stream());
        }
        if (rc) return none();
        PyObject *out = PyTuple_New(3);
        at::Tensor *const grads[3] = {&dq, &dk, &dv};
        for (int i = 0; out && i < 3; ++i) {
            PyObject *const t = THPVariable_Wrap(std::move(*grads[i]));
            if (t) PyTuple_SET_ITEM(out, i, t);
            else Py_CLEAR(out);
        }
        return out;                // nullptr with the error that PyTuple_New or THPVariable_Wrap has set
    } catch (...) {
        return none();
    }
}

// The library's functions, as addresses: sigmoid_attn_fwd, sigmoid_attn_bwd, sigmoid_attn_bwd_onepass_workspace_bytes.
PyObject *use(PyObject *, PyObject *args) {
    unsigned long long f, b, s;
    if (!PyArg_ParseTuple(args, "KKK", &f, &b, &s)) return nullptr;
    fwd_fn = reinterpret_cast<FwdFn>(f);
    bwd_fn = reinterpret_cast<BwdFn>(b);
    bytes_fn = reinterpret_cast<BytesFn>(s);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(fwd)), METH_FASTCALL, nullptr},
    {"bwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(bwd)), METH_FASTCALL, nullptr},
    {"use", use, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
