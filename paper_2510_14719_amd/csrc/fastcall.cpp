// The calls of binding.py without the interpreter's share: a Python extension that reads addresses, element types and the
// current stream from torch's own objects and calls the C ABI of the library.
//
// What bounds a small call is the host: on MI355X the launch itself takes 3 us and the kernel of 2 heads of 128 tokens 5.1; looking up
// torch's current stream from Python takes 2.8 us, the five tensors 0.9, the ctypes call 0.7.
// Back to back, us per call before / after: attn_fwd (1, 2, 128, 64) 8.2 / 5.2; gemm_nt (64, 64, 64) 7.4 / 3.5.
//
// Every function returns NotImplemented, having done nothing, for arguments that it does not take: then binding.py goes on
// with its own general code, which accepts, converts or refuses them.  Taken are exact tensors (no subclass, no wrapper without
// memory, no mode that wants to see the accesses) that are on the device and contiguous, or addresses as int; sizes as int in
// the range of a C int; scale as float or int; causal as bool or int; a stream as None or int; a type code as None or int.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "attn_fwd.h"
#include "gemm_nt.h"

namespace {

typedef decltype(&::attn_fwd) attn_fn;
typedef decltype(&::gemm_nt) gemm_fn;
static_assert(std::is_same<attn_fn, decltype(&::attn_fwd_fp8)>::value && std::is_same<gemm_fn, decltype(&::gemm_nt_fp8)>::value, "pairs of calls");

attn_fn attn_calls[2];          // attn_fwd, attn_fwd_fp8
gemm_fn gemm_calls[2];          // gemm_nt, gemm_nt_fp8
bool enabled = false;

PyObject* not_taken()
{
    Py_RETURN_NOTIMPLEMENTED;
}

// Address of a tensor (or an int), and the tensor itself where it is one.
bool address(PyObject* x, void*& p, const at::Tensor*& t)
{
    t = nullptr;
    if (THPVariable_CheckExact(x)) {
        const at::Tensor& a = THPVariable_Unpack(x);
        const c10::DispatchKeySet keys = a.key_set();
        if (!a.defined() || !a.is_cuda() || a.layout() != at::kStrided || !a.has_storage() || keys.has(c10::DispatchKey::Functionalize) ||
            keys.has(c10::DispatchKey::Python) || keys.has(c10::DispatchKey::FuncTorchGradWrapper) ||
            keys.has(c10::DispatchKey::FuncTorchBatched) || !a.is_contiguous())
            return false;
        p = a.data_ptr();
        t = &a;
        return true;
    }
    if (!PyLong_CheckExact(x)) return false;
    p = reinterpret_cast<void*>(PyLong_AsUnsignedLongLong(x));
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool c_int(PyObject* x, int& v)
{
    if (!PyLong_CheckExact(x)) return false;
    int overflow = 0;
    const long long l = PyLong_AsLongLongAndOverflow(x, &overflow);
    if (overflow || l < INT_MIN || l > INT_MAX) return false;
    v = (int)l;
    return true;
}

// The stream to launch on: the one given, or torch's current one (some tensor is on the device, so torch has initialised it).
bool stream_of(PyObject* x, bool have_tensor, void*& s)
{
    if (x == Py_None) {
        if (!have_tensor) return false;
        s = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (!PyLong_CheckExact(x)) return false;
    s = reinterpret_cast<void*>(PyLong_AsUnsignedLongLong(x));
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// The type code given, or that of the tensor's 16-bit elements.
bool code_of(PyObject* x, const at::Tensor* t, int& code)
{
    if (x != Py_None) return c_int(x, code);
    if (!t) return false;
    if (t->scalar_type() == at::kHalf) code = 0;
    else if (t->scalar_type() == at::kBFloat16) code = 1;
    else return false;
    return true;
}

// (q, k, v, o, lse, B, H, N, d, scale, causal, stream, type code)
template <int WHICH>            // 0: 16-bit inputs, whose type is the code; 1: E4M3 inputs, the code is the type of o
PyObject* attn(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 13 || !enabled || at::impl::torch_function_mode_enabled()) return not_taken();
    try {
        void* p[5];
        const at::Tensor* t[5];
        bool tensors = false;
        for (int i = 0; i < 5; ++i) {
            if (!address(args[i], p[i], t[i])) return not_taken();
            tensors |= t[i] != nullptr;
        }
        int size[4], code;
        for (int i = 0; i < 4; ++i)
            if (!c_int(args[5 + i], size[i])) return not_taken();
        if (!PyFloat_CheckExact(args[9]) && !PyLong_CheckExact(args[9])) return not_taken();
        const double scale = PyFloat_AsDouble(args[9]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return not_taken();
        }
        if (!PyBool_Check(args[10]) && !PyLong_CheckExact(args[10])) return not_taken();
        const int causal = PyObject_IsTrue(args[10]);
        void* stream;
        if (!stream_of(args[11], tensors, stream) || !code_of(args[12], t[WHICH == 0 ? 0 : 3], code)) return not_taken();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = attn_calls[WHICH](p[0], p[1], p[2], p[3], (float*)p[4], size[0], size[1], size[2], size[3], (float)scale, causal, stream, code);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (...) {             // (torch's: the general code meets the same and reports it)
        return not_taken();
    }
}

// (a, b, c, M, N, K, stream, type code)
template <int WHICH>
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 8 || !enabled || at::impl::torch_function_mode_enabled()) return not_taken();
    try {
        void* p[3];
        const at::Tensor* t[3];
        bool tensors = false;
        for (int i = 0; i < 3; ++i) {
            if (!address(args[i], p[i], t[i])) return not_taken();
            tensors |= t[i] != nullptr;
        }
        int size[3], code;
        for (int i = 0; i < 3; ++i)
            if (!c_int(args[3 + i], size[i])) return not_taken();
        void* stream;
        if (!stream_of(args[6], tensors, stream) || !code_of(args[7], WHICH == 0 ? t[0] : nullptr, code)) return not_taken();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = gemm_calls[WHICH](p[0], p[1], p[2], size[0], size[1], size[2], stream, code);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (...) {
        return not_taken();
    }
}

// bind(attn_fwd, attn_fwd_fp8, gemm_nt, gemm_nt_fp8): addresses of the functions of the loaded library
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    void* f[4];
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "bind takes four addresses");
        return nullptr;
    }
    for (int i = 0; i < 4; ++i) {
        f[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
        if (!f[i]) {
            PyErr_SetString(PyExc_ValueError, "bind takes four addresses");
            return nullptr;
        }
    }
    attn_calls[0] = (attn_fn)f[0];
    attn_calls[1] = (attn_fn)f[1];
    gemm_calls[0] = (gemm_fn)f[2];
    gemm_calls[1] = (gemm_fn)f[3];
    enabled = true;
    Py_RETURN_NONE;
}

// disable(): from here on nothing is taken (a forked child: torch refuses its device there, in the general code)
PyObject* disable(PyObject*, PyObject*)
{
    enabled = false;
    Py_RETURN_NONE;
}

template <typename F> PyCFunction fast(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef methods[] = {
    {"attn_fwd", fast(attn<0>), METH_FASTCALL, nullptr},
    {"attn_fwd_fp8", fast(attn<1>), METH_FASTCALL, nullptr},
    {"gemm_nt", fast(gemm<0>), METH_FASTCALL, nullptr},
    {"gemm_nt_fp8", fast(gemm<1>), METH_FASTCALL, nullptr},
    {"bind", fast(bind), METH_FASTCALL, nullptr},
    {"disable", disable, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch that the extension was compiled against, whose object layouts it knows (binding.py compares).
PyMODINIT_FUNC PyInit__fastcall(void)
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", FASTCALL_TORCH) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
