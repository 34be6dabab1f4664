// The calls of a single linear layer from Python, in native code: what binding.lr_linear_fwd and binding.lr_linear_bwd do for plain
// tensors that fit each other, with the outputs allocated here.  Anything else (an argument that is no plain tensor, shapes or types
// that do not match, a mode or a transform of torch that wants to see the allocations) is answered with None, and the Python code goes
// on as if it had not asked, error messages included.
//
// A pass over a small layer is bound by this: 64 x 256 x 256 fp32, forward and backward, takes the GPU less than Python's 21 us.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

using FwdFn = int (*)(const void*, const void*, const void*, void*, void*, int64_t, int64_t, int64_t, int64_t, int, void*, size_t, void*);
using WantsFn = int (*)(int, int64_t, int64_t, int64_t, int64_t, int);
using BwdFn = int (*)(const void*, const void*, const void*, const void*, const void*, void*, void*, void*, int64_t, int64_t, int64_t, int64_t, int, int, void*,
                      size_t, void*);
using BytesFn = size_t (*)(int64_t, int64_t, int64_t, int64_t, int);

FwdFn fwd_fn; WantsFn wants_fn; BwdFn bwd_fn; BytesFn bytes_fn;
PyObject *get_device, *get_stream, *check;      // torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, binding._check

// A tensor on the GPU with a memory of its own, contiguous, nobody between it and its data
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    static const c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
                                              c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize, c10::DispatchKey::Negative,
                                              c10::DispatchKey::Conjugate, c10::DispatchKey::ZeroTensor, c10::DispatchKey::Batched});
    if (!t.defined() || t.key_set().has_any(wrapped) || t.layout() != at::kStrided || !t.is_cuda() || t.dim() != 2 || !t.has_storage() ||
        t.unsafeGetTensorImpl()->has_symbolic_sizes_strides() || !t.is_contiguous())
        return nullptr;
    return &t;
}
bool watched() {
    return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled() ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) ||
           c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Functionalize) || c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Tracer);
}
// the current stream of the current device, as the Python code asks for it
bool current_stream(void** s) {
    PyObject* dev = PyObject_CallNoArgs(get_device);
    if (!dev) return false;
    PyObject* raw = PyObject_CallOneArg(get_stream, dev);
    Py_DECREF(dev);
    if (!raw) return false;
    *s = reinterpret_cast<void*>(PyLong_AsSsize_t(raw));
    Py_DECREF(raw);
    return !PyErr_Occurred();
}
// The results, or for an error of the library what binding._check raises
PyObject* finished(PyObject* results, int code, const char* what) {
    if (code == 0) return results;
    Py_DECREF(results);
    PyObject* r = PyObject_CallFunction(check, "is", code, what);
    Py_XDECREF(r);
    return nullptr;
}
PyObject* wrap_or_none(const at::Tensor& t) {
    if (t.defined()) return THPVariable_Wrap(t);
    Py_RETURN_NONE;
}

// Everything that can fail comes before the launch: a call that is answered with None has done nothing.  Addresses are asked for with
// data_ptr(), as from Python: what materialises or refuses there does here.

// (X, A, B, save_T) -> (Y, T or None), or None
PyObject* fwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 4) { PyErr_SetString(PyExc_TypeError, "fwd(X, A, B, save_T)"); return nullptr; }
    void *stream, *x, *a, *b, *y, *t = nullptr;
    int64_t M, m, cols, r;
    int dt;
    PyObject* results;
    at::Tensor Y, T;
    try {
        const at::Tensor *X = plain(args[0]), *A = plain(args[1]), *B = plain(args[2]);
        const int save = PyObject_IsTrue(args[3]);
        if (save < 0) return nullptr;
        if (!X || !A || !B || watched()) Py_RETURN_NONE;
        const auto dtype = X->scalar_type();
        const bool f32 = dtype == at::kFloat;
        M = X->size(0); cols = X->size(1); m = A->size(0); r = A->size(1);
        if ((!f32 && dtype != at::kBFloat16) || A->scalar_type() != dtype || B->scalar_type() != dtype || B->size(0) != r || B->size(1) != cols || (f32 && !save))
            Py_RETURN_NONE;
        if (!current_stream(&stream)) return nullptr;
        const auto opt = X->options().requires_grad(false);
        dt = f32 ? 0 : 1;
        Y = at::empty({M, m}, opt);
        if (save || wants_fn(1, M, m, cols, r, dt)) T = at::empty({M, r}, opt);
        x = X->data_ptr(); a = A->data_ptr(); b = B->data_ptr(); y = Y.data_ptr();
        if (T.defined()) t = T.data_ptr();
        results = Py_BuildValue("(NN)", THPVariable_Wrap(Y), wrap_or_none(save ? T : at::Tensor()));
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;                                  // out of memory and the like: the Python code meets it again and says so
    }
    if (!results) return nullptr;
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = fwd_fn(x, a, b, y, t, M, m, cols, r, dt, nullptr, 0, stream);
    Py_END_ALLOW_THREADS
    return finished(results, code, "lr_linear_fwd");
}

// (dY, X, T, A, B, need_dX, need_dA, need_dB, dX, dA, dB, accumulate) -> (dX, dA, dB), or None
PyObject* bwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 12) { PyErr_SetString(PyExc_TypeError, "bwd takes 12 arguments"); return nullptr; }
    void *stream, *space, *in[5], *to[3];
    int64_t M, m, cols, r;
    int dt, flag[4];
    size_t size;
    PyObject* results;
    at::Tensor ws, out[3];                               // dX, dA, dB
    try {
        const at::Tensor *dY = plain(args[0]), *X = plain(args[1]), *A = plain(args[3]), *B = plain(args[4]);
        const at::Tensor* T = args[2] == Py_None ? nullptr : plain(args[2]);
        if (!dY || !X || !A || !B || (!T && args[2] != Py_None) || watched()) Py_RETURN_NONE;
        const int at_arg[4] = {5, 6, 7, 11};
        for (int i = 0; i < 4; ++i)
            if ((flag[i] = PyObject_IsTrue(args[at_arg[i]])) < 0) return nullptr;
        const auto dtype = X->scalar_type();
        const bool f32 = dtype == at::kFloat;
        M = X->size(0); cols = X->size(1); m = A->size(0); r = A->size(1);
        if ((!f32 && dtype != at::kBFloat16) || A->scalar_type() != dtype || B->scalar_type() != dtype || dY->scalar_type() != dtype || (T && T->scalar_type() != dtype) ||
            dY->size(0) != M || dY->size(1) != m || B->size(0) != r || B->size(1) != cols || (T && (T->size(0) != M || T->size(1) != r)))
            Py_RETURN_NONE;
        const int64_t shape[3][2] = {{M, cols}, {m, r}, {r, cols}};
        const auto opt = X->options().requires_grad(false);
        for (int i = 0; i < 3; ++i) {
            PyObject* given = args[8 + i];
            if (given != Py_None) {
                const at::Tensor* g = plain(given);
                if (!g || g->scalar_type() != (i == 0 ? dtype : at::kFloat) || g->size(0) != shape[i][0] || g->size(1) != shape[i][1]) Py_RETURN_NONE;
                if (flag[i]) out[i] = *g;
            } else if (flag[i] && flag[3] && i > 0) {
                Py_RETURN_NONE;                          // accumulate needs them
            }
        }
        if (!current_stream(&stream)) return nullptr;
        for (int i = 0; i < 3; ++i)
            if (flag[i] && !out[i].defined()) out[i] = at::empty({shape[i][0], shape[i][1]}, i == 0 ? opt : opt.dtype(at::kFloat));
        dt = f32 ? 0 : 1;
        const size_t bytes = bytes_fn(M, m, cols, r, dt);
        size = bytes < 256 ? 256 : bytes;
        ws = at::empty({(int64_t)size}, opt.dtype(at::kByte));
        space = ws.data_ptr();
        const at::Tensor* operands[5] = {dY, X, T, A, B};
        for (int i = 0; i < 5; ++i) in[i] = operands[i] ? operands[i]->data_ptr() : nullptr;
        for (int i = 0; i < 3; ++i) to[i] = out[i].defined() ? out[i].data_ptr() : nullptr;
        PyObject* res[3];
        for (int i = 0; i < 3; ++i) {
            if (flag[i] && args[8 + i] != Py_None) { Py_INCREF(args[8 + i]); res[i] = args[8 + i]; }
            else res[i] = wrap_or_none(out[i]);
        }
        results = Py_BuildValue("(NNN)", res[0], res[1], res[2]);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (!results) return nullptr;
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = bwd_fn(in[0], in[1], in[2], in[3], in[4], to[0], to[1], to[2], M, m, cols, r, dt, flag[3], space, size, stream);
    Py_END_ALLOW_THREADS
    return finished(results, code, "lr_linear_bwd");
}

// (addresses of lr_linear_fwd, lr_linear_fwd_wants_T, lr_linear_bwd, lr_linear_bwd_workspace_bytes, the three callables)
PyObject* setup(PyObject*, PyObject* args) {
    unsigned long long a, b, c, d;
    if (!PyArg_ParseTuple(args, "KKKKOOO", &a, &b, &c, &d, &get_device, &get_stream, &check)) return nullptr;
    Py_INCREF(get_device); Py_INCREF(get_stream); Py_INCREF(check);
    fwd_fn = reinterpret_cast<FwdFn>(a); wants_fn = reinterpret_cast<WantsFn>(b);
    bwd_fn = reinterpret_cast<BwdFn>(c); bytes_fn = reinterpret_cast<BytesFn>(d);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fwd)), METH_FASTCALL, nullptr},
                         {"bwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bwd)), METH_FASTCALL, nullptr},
                         {"setup", setup, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "layer_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_layer_call() { return PyModule_Create(&module); }
