// mttkrp_dense() of the Python binding without ctypes: reads the tensors of one call through PyTorch's C++ interface and calls the C entry
// point.  Arguments of any other kind, or that the entry point's checks would refuse, are left to the Python code, which then says what is
// wrong with them; so is every call under a torch-function or dispatch mode, and every tensor subclass.
//
// A small call was bound by its caller: 64^3 at R = 16 took 7.1 us a call on the host with one launch and 10.4 with two (4 us of ctypes and
// Python), while a graph of the same launches runs the three modes in 14.2 us; now 2.9 and 6.1, the three modes 26.1 -> 15.6.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mttkrp.h"

namespace {

// the library's entry points, as the binding has loaded them
struct Entries {
    decltype(&mttkrp_dense_f64) f64;
    decltype(&mttkrp_dense_f32) f32;
    decltype(&mttkrp_dense_f64_ws) f64_ws;
    decltype(&mttkrp_dense_f32_ws) f32_ws;
    decltype(&mttkrp_dense_f64_ex) f64_ex;
    decltype(&mttkrp_dense_f32_ex) f32_ex;
} entries;
PyObject* current_stream = nullptr;      // torch's function from a device's index to the raw stream

// The plain tensor behind an object, or null.
const at::Tensor* plain(PyObject* o)
{
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.has_storage() && t.layout() == at::kStrided && t.is_cuda() ? &t : nullptr;
}

// The element of a list or tuple, borrowed, or null.
PyObject* element(PyObject* seq, Py_ssize_t i) { return PyTuple_Check(seq) ? PyTuple_GET_ITEM(seq, i) : PyList_GET_ITEM(seq, i); }
bool is_sequence(PyObject* o) { return PyTuple_Check(o) || PyList_Check(o); }

bool whole_number(PyObject* o, int64_t& v)
{
    if (!PyLong_CheckExact(o))
        return false;
    int over = 0;
    v = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0;
}

// dense(X, dims, factors, k, M, workspace, stream, lam, beta): M, a status other than 0, or None for a call that is left to the caller
PyObject* dense(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 9 || !entries.f64 || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set())
        Py_RETURN_NONE;
    const at::Tensor* const X = plain(a[0]);
    if (!X || !is_sequence(a[1]) || !is_sequence(a[2]))
        Py_RETURN_NONE;
    const at::ScalarType type = X->scalar_type();
    const bool f64 = type == at::kDouble;
    const auto dev = X->get_device();
    const Py_ssize_t d = Py_SIZE(a[1]);
    if ((!f64 && type != at::kFloat) || d < 1 || d > MTTKRP_MAX_NDIM || Py_SIZE(a[2]) != d || !X->is_contiguous())
        Py_RETURN_NONE;
    auto like_X = [&](const at::Tensor& t) { return t.scalar_type() == type && t.get_device() == dev && t.is_contiguous(); };
    int64_t dims[MTTKRP_MAX_NDIM], values = 1, k = 0, R = -1;
    for (Py_ssize_t m = 0; m < d; ++m) {
        if (!whole_number(element(a[1], m), dims[m]) || dims[m] < 1 || values > (int64_t)1 << 57 || dims[m] > (int64_t)1 << 57)
            Py_RETURN_NONE;
        if (__builtin_mul_overflow(values, dims[m], &values))
            Py_RETURN_NONE;
    }
    if (values != X->numel() || !whole_number(a[3], k) || k < 0 || k >= d)
        Py_RETURN_NONE;
    const void* factors[MTTKRP_MAX_NDIM];
    for (Py_ssize_t m = 0; m < d; ++m) {
        PyObject* const o = element(a[2], m);
        factors[m] = nullptr;
        if (o == Py_None)
            continue;
        const at::Tensor* const A = plain(o);
        if (!A || !like_X(*A) || A->dim() != 2 || A->size(0) != dims[m] || (R >= 0 && A->size(1) != R))
            Py_RETURN_NONE;
        R = A->size(1);
        factors[m] = A->data_ptr();
    }
    if (R < 0 || R > 0x7fffffff)
        Py_RETURN_NONE;
    const at::Tensor* ws = nullptr;
    const at::Tensor* lam = nullptr;
    if (a[5] != Py_None && !(ws = plain(a[5])))
        Py_RETURN_NONE;
    if (a[7] != Py_None && (!(lam = plain(a[7])) || !like_X(*lam) || lam->numel() != R))
        Py_RETURN_NONE;
    if (a[8] != Py_None && !PyFloat_CheckExact(a[8]))
        Py_RETURN_NONE;
    if (c10::impl::getDeviceGuardImpl(c10::DeviceType::CUDA)->getDevice().index() != dev)
        Py_RETURN_NONE;
    at::Tensor own;
    const at::Tensor* M = &own;
    if (a[4] == Py_None) {
        own = at::empty({dims[k], R}, X->options());
    } else {
        M = plain(a[4]);
        if (!M || !like_X(*M) || M->dim() != 2 || M->size(0) != dims[k] || M->size(1) != R)
            Py_RETURN_NONE;
    }
    void* stream = nullptr;
    if (a[6] == Py_None) {
        PyObject* const index = PyLong_FromLong((long)dev);
        PyObject* const raw = index ? PyObject_CallOneArg(current_stream, index) : nullptr;
        Py_XDECREF(index);
        if (!raw)
            return nullptr;
        stream = PyLong_AsVoidPtr(raw);
        Py_DECREF(raw);
        if (PyErr_Occurred())
            return nullptr;
    } else {
        if (!PyLong_CheckExact(a[6]))
            Py_RETURN_NONE;
        stream = PyLong_AsVoidPtr(a[6]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
    }
    void* const x = X->data_ptr();
    void* const m = M->data_ptr();
    void* const w = ws ? ws->data_ptr() : nullptr;
    const size_t w_bytes = ws ? ws->nbytes() : 0;
    const void* const l = lam ? lam->data_ptr() : nullptr;
    const double beta = a[8] != Py_None ? PyFloat_AS_DOUBLE(a[8]) : 0.0;
    const bool ex = lam || a[8] != Py_None;
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    if (f64) {
        const double* const* const f = (const double* const*)factors;
        rc = ex ? entries.f64_ex((int)d, dims, (const double*)x, f, (int)R, (int)k, (const double*)l, beta, (double*)m, w, w_bytes, stream)
             : ws ? entries.f64_ws((int)d, dims, (const double*)x, f, (int)R, (int)k, (double*)m, w, w_bytes, stream)
                  : entries.f64((int)d, dims, (const double*)x, f, (int)R, (int)k, (double*)m, stream);
    } else {
        const float* const* const f = (const float* const*)factors;
        rc = ex ? entries.f32_ex((int)d, dims, (const float*)x, f, (int)R, (int)k, (const float*)l, (float)beta, (float*)m, w, w_bytes, stream)
             : ws ? entries.f32_ws((int)d, dims, (const float*)x, f, (int)R, (int)k, (float*)m, w, w_bytes, stream)
                  : entries.f32((int)d, dims, (const float*)x, f, (int)R, (int)k, (float*)m, stream);
    }
    Py_END_ALLOW_THREADS;
    if (rc != MTTKRP_OK)
        return PyLong_FromLong(rc);
    if (a[4] == Py_None)
        return THPVariable_Wrap(std::move(own));
    Py_INCREF(a[4]);
    return a[4];
}

// (C++ exceptions, as of an allocation that fails, become Python's)
PyObject* dense_guarded(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    try {
        return dense(self, a, n);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// bind(f64, f32, f64_ws, f32_ws, f64_ex, f32_ex, current_stream): addresses of the C entry points, torch's function
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void* p[6];
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "bind() takes six addresses and a function");
        return nullptr;
    }
    for (int i = 0; i < 6; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred())
            return nullptr;
    }
    Py_INCREF(a[6]);
    Py_XSETREF(current_stream, a[6]);
    entries = {(decltype(entries.f64))p[0],    (decltype(entries.f32))p[1],    (decltype(entries.f64_ws))p[2],
               (decltype(entries.f32_ws))p[3], (decltype(entries.f64_ex))p[4], (decltype(entries.f32_ex))p[5]};
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"dense", (PyCFunction)(void (*)(void))dense_guarded, METH_FASTCALL, nullptr},
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_dense_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dense_call() { return PyModule_Create(&module); }
