// The Python entry points' calls on plain torch tensors, without the Python in between: checks, outputs, stream and the call into the C ABI.
//
// approx(x, k, b, k_b, assignment) and exact(x, k) return (vals, idx), the library's status where it is not 0, or None for whatever is
// not a plain call - a tensor subclass, a function or dispatch mode, a trace, a tensor without memory of its own, arguments that are no integers, x
// not on the current device or not what the library takes - which binding.py then does, or refuses, as it does all calls with `out`.
//
// A call of a few microseconds on the GPU waits for its host side: of 8.4 us for 4 x 4096 f32, k = b = 64, the two outputs took 3.1 through torch's
// Python interface, the launch 3.2, ctypes 0.5 and the Python around them 1.1.  Here it takes 5.3.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/version.h>

#include "../../include/approx_topk.h"

namespace {

decltype(&approx_topk) approx_fn;         // of the library that binding.py has loaded
decltype(&approx_topk_assign) assign_fn;
decltype(&exact_topk) exact_fn;

bool integer(PyObject *o, int64_t *out) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *out = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0;
}

// None: not a plain call
template <typename CALL>
PyObject *plain_call(PyObject *obj, int64_t k, CALL call) {
    try {
        if (!THPVariable_CheckExact(obj) || k < 1 || at::impl::torch_function_mode_enabled() ||
            c10::impl::TorchDispatchModeTLS::any_modes_set() || torch::jit::tracer::isTracing())
            Py_RETURN_NONE;
        const at::Tensor &x = THPVariable_Unpack(obj);
        const at::ScalarType type = x.scalar_type();
        if (!x.is_cuda() || x.layout() != at::kStrided || !x.has_storage() || x.dim() != 2 || !x.is_contiguous() ||
            (type != at::kFloat && type != at::kBFloat16) || x.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Python,
            c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize})))
            Py_RETURN_NONE;
        const int64_t m = x.size(0), n = x.size(1);
        const c10::DeviceIndex device = x.get_device();
        if (device != c10::hip::current_device() || k > n) Py_RETURN_NONE;
        at::Tensor vals = at::empty({m, k}, x.options());
        at::Tensor idx = at::empty({m, k}, x.options().dtype(at::kInt));
        void *stream = c10::hip::getCurrentHIPStream(device).stream();
        void *const xp = x.data_ptr(), *const vp = vals.data_ptr(), *const ip = idx.data_ptr();
        int code;
        Py_BEGIN_ALLOW_THREADS
        code = call(xp, m, n, type == at::kFloat ? ATK_F32 : ATK_BF16, vp, (int32_t *)ip, stream);
        Py_END_ALLOW_THREADS
        if (code != ATK_OK) return PyLong_FromLong(code);
        PyObject *v = THPVariable_Wrap(std::move(vals));
        if (!v) return nullptr;
        PyObject *i = THPVariable_Wrap(std::move(idx));
        if (!i) {
            Py_DECREF(v);
            return nullptr;
        }
        PyObject *both = PyTuple_New(2);
        if (!both) {
            Py_DECREF(v);
            Py_DECREF(i);
            return nullptr;
        }
        PyTuple_SET_ITEM(both, 0, v);
        PyTuple_SET_ITEM(both, 1, i);
        return both;
    } catch (...) {  // (no memory, say: the Python path meets the same and says so in torch's words)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyObject *approx(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    int64_t k, b, k_b, assignment = 0;
    if (n_args != 5 || !approx_fn || !integer(args[1], &k) || !integer(args[2], &b) || !integer(args[3], &k_b) ||
        (args[4] != Py_None && (!integer(args[4], &assignment) || (assignment != ATK_INTERLEAVED && assignment != ATK_CONTIGUOUS))))
        Py_RETURN_NONE;
    if (args[4] == Py_None)
        return plain_call(args[0], k, [=](void *x, int64_t m, int64_t n, int type, void *v, int32_t *i, void *s) {
            return approx_fn(x, m, n, k, b, k_b, type, v, i, s);
        });
    return plain_call(args[0], k, [=](void *x, int64_t m, int64_t n, int type, void *v, int32_t *i, void *s) {
        return assign_fn(x, m, n, k, b, k_b, type, (int)assignment, v, i, s);
    });
}

PyObject *exact(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    int64_t k;
    if (n_args != 2 || !exact_fn || !integer(args[1], &k)) Py_RETURN_NONE;
    return plain_call(args[0], k, [=](void *x, int64_t m, int64_t n, int type, void *v, int32_t *i, void *s) {
        return exact_fn(x, m, n, k, type, v, i, s);
    });
}

// use(approx_topk, approx_topk_assign, exact_topk): the addresses of the C ABI's functions
PyObject *use(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    if (n_args != 3) {
        PyErr_SetString(PyExc_TypeError, "three addresses");
        return nullptr;
    }
    void *at[3];
    for (int i = 0; i < 3; ++i) {
        at[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    approx_fn = (decltype(approx_fn))at[0];
    assign_fn = (decltype(assign_fn))at[1];
    exact_fn = (decltype(exact_fn))at[2];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"approx", (PyCFunction)(void (*)())approx, METH_FASTCALL, nullptr},
    {"exact", (PyCFunction)(void (*)())exact, METH_FASTCALL, nullptr},
    {"use", (PyCFunction)(void (*)())use, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_atk_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__atk_torch() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {  // (this file knows torch's own structures: for that release alone)
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
