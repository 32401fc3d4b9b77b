// The calls of binding.py whose arguments are in order, without Python's attribute look-ups: a small layer takes the GPU 3 us, and the checks and the
// conversion of its arguments in Python took the host as long.  Whatever is not in order returns -1 and is looked at again there, for the message.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/qfc.h"

namespace {

decltype(&qfc_forward) g_forward = nullptr;
decltype(&qfc_forward_fused) g_forward_fused = nullptr;
PyObject *g_stream = nullptr;  // torch's current stream, asked for once the arguments are in order

// Pointer of a contiguous binary16 matrix on a GPU with `cols` columns and (if rows >= 0) that many rows, which are returned; null: something else.
// Plain tensors with memory of their own only: subclasses and wrappers (tracing, vmap) go the other way.
void *matrix(PyObject *o, int64_t &rows, int64_t cols) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || !t.is_cuda() || t.scalar_type() != at::kHalf || t.dim() != 2 || !t.is_contiguous()) return nullptr;
    const auto sizes = t.sizes();
    if (sizes[1] != cols || (rows >= 0 && sizes[0] != rows)) return nullptr;
    rows = sizes[0];
    return t.mutable_data_ptr();
}

void *vector(PyObject *o, int64_t size) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || !t.is_cuda() || t.scalar_type() != at::kHalf || t.dim() != 1 || t.sizes()[0] != size || !t.is_contiguous()) return nullptr;
    return t.mutable_data_ptr();
}

// False with Python's error set where there is none
bool current_stream(void *&stream) {
    PyObject *s = PyObject_CallNoArgs(g_stream);
    if (!s) return false;
    stream = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !PyErr_Occurred();
}

// bind(address of qfc_forward, address of qfc_forward_fused, function that returns the current stream)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 3) return PyErr_Format(PyExc_TypeError, "two addresses and a function");
    void *f = PyLong_AsVoidPtr(a[0]), *g = PyLong_AsVoidPtr(a[1]);
    if (PyErr_Occurred()) return nullptr;
    g_forward = reinterpret_cast<decltype(g_forward)>(f);
    g_forward_fused = reinterpret_cast<decltype(g_forward_fused)>(g);
    Py_INCREF(a[2]);
    Py_XSETREF(g_stream, a[2]);
    Py_RETURN_NONE;
}

// forward(handle, x, y, N, K) -> status, or -1
PyObject *forward(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 5 || !g_forward) return PyLong_FromLong(-1);
    void *h = PyLong_AsVoidPtr(a[0]);
    const long N = PyLong_AsLong(a[3]), K = PyLong_AsLong(a[4]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return PyLong_FromLong(-1);
    }
    int64_t M = -1;
    void *x = nullptr, *y = nullptr;
    try {
        x = matrix(a[1], M, K);
        if (x) y = matrix(a[2], M, N);
    } catch (...) {
        y = nullptr;
    }
    if (!x || !y || M < 1 || M > INT32_MAX) return PyLong_FromLong(-1);
    void *stream;
    if (!current_stream(stream)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = g_forward(static_cast<qfc_handle_t>(h), x, (int32_t)M, y, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// forward_fused(handle, x, y, N, K, gate, activation, residual, gated_output, norm_gamma, norm_eps, norm_offset) -> status, or -1
PyObject *forward_fused(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 12 || !g_forward_fused) return PyLong_FromLong(-1);
    void *h = PyLong_AsVoidPtr(a[0]);
    const long N = PyLong_AsLong(a[3]), K = PyLong_AsLong(a[4]), activation = PyLong_AsLong(a[6]);
    const int gated = PyObject_IsTrue(a[8]);
    qfc_fusion_t f = {};
    f.norm_eps = (float)PyFloat_AsDouble(a[10]);
    f.norm_offset = (float)PyFloat_AsDouble(a[11]);
    if (PyErr_Occurred()) {
        PyErr_Clear();  // (an argument of another type: as the other way takes it)
        return PyLong_FromLong(-1);
    }
    if (activation < INT32_MIN || activation > INT32_MAX || (gated && a[7] != Py_None)) return PyLong_FromLong(-1);
    f.activation = (int32_t)activation;
    f.gated_output = gated;
    int64_t M = -1;
    void *x = nullptr, *y = nullptr;
    bool ok = false;
    try {
        x = matrix(a[1], M, K);
        if (x) y = matrix(a[2], M, gated ? N / 2 : N);
        ok = x && y;
        if (ok && a[5] != Py_None) ok = (f.gate = matrix(a[5], M, K)) != nullptr;
        if (ok && a[7] != Py_None) ok = (f.residual = matrix(a[7], M, N)) != nullptr;
        if (ok && a[9] != Py_None) ok = (f.norm_gamma = vector(a[9], K)) != nullptr;
    } catch (...) {
        ok = false;
    }
    if (!ok || M < 1 || M > INT32_MAX) return PyLong_FromLong(-1);
    void *stream;
    if (!current_stream(stream)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = g_forward_fused(static_cast<qfc_handle_t>(h), x, (int32_t)M, y, &f, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(bind), METH_FASTCALL, nullptr},
    {"forward", reinterpret_cast<PyCFunction>(forward), METH_FASTCALL, nullptr},
    {"forward_fused", reinterpret_cast<PyCFunction>(forward_fused), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", QFC_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
