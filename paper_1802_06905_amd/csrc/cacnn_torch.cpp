// The usual call of the binding in native code: contiguous device tensors of the right element sizes.  Asking a tensor for its address, length,
// element size and layout, and torch for its current stream, through the interpreter took 1.1 of a small call's 5.2 us; the launch itself
// takes 2.9.  Everything else (other operands, wrong sizes, errors) is left to the binding: -1 says that nothing was tried.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "cacnn_internal.h"

namespace {

using ConvFn = int (*)(const void* problem, int dtype, const void* image, int64_t image_elems, const void* filter, int64_t filter_elems,
                       void* out, int64_t out_elems, void* stream);
using PoolFn = int (*)(const void* problem, int dtype, int mode, const void* image, int64_t image_elems, void* out, int64_t out_elems, void* stream);

constexpr Py_ssize_t kProblemBytes = 9 * 8;
PyTypeObject* g_problem = nullptr;   // the binding's Problem, a ctypes structure
ConvFn g_conv = nullptr;
PoolFn g_pool = nullptr;

PyObject* not_tried() { return PyLong_FromLong(-1); }

bool small_int(PyObject* o, int* value) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    *value = (int)v;
    return !overflow && v == (long)*value;
}

// None: torch's current stream of the current device; else a raw handle
bool stream_of(PyObject* o, void** stream) {
    if (o == Py_None) {
        *stream = (void*)c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    *stream = PyLong_AsVoidPtr(o);
    if (*stream || !PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

// a contiguous device tensor of torch's own class with elements of `size` bytes
const at::Tensor* usual(PyObject* o, int64_t size) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.is_cuda() && t.element_size() == size && t.is_contiguous() ? &t : nullptr;
}

// the structure's bytes (they belong to the object, which the caller's arguments keep)
const void* problem_of(PyObject* o) {
    if (Py_TYPE(o) != g_problem) return nullptr;
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return nullptr;
    }
    const void* p = view.len == kProblemBytes ? view.buf : nullptr;
    PyBuffer_Release(&view);
    return p;
}

// conv(problem, dtype, image, filter, out, stream)
PyObject* conv(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int dtype = 0;
    void* stream = nullptr;
    if (n != 6 || !g_conv || !small_int(args[1], &dtype) || (dtype != 0 && dtype != 1)) return not_tried();
    const int64_t size = dtype == 0 ? 4 : 2;
    const void* const problem = problem_of(args[0]);
    const at::Tensor* const image = usual(args[2], size);
    const at::Tensor* const filter = usual(args[3], size);
    const at::Tensor* const out = usual(args[4], 4);
    if (!problem || !image || !filter || !out || out->scalar_type() != at::kFloat || !stream_of(args[5], &stream)) return not_tried();
    const void *pi = image->data_ptr(), *pf = filter->data_ptr();
    void* const po = out->data_ptr();
    const int64_t ni = image->numel(), nf = filter->numel(), no = out->numel();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_conv(problem, dtype, pi, ni, pf, nf, po, no, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// pool(problem, dtype, mode, image, out, stream)
PyObject* pool(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int dtype = 0, mode = 0;
    void* stream = nullptr;
    if (n != 6 || !g_pool || !small_int(args[1], &dtype) || !small_int(args[2], &mode) || (dtype != 0 && dtype != 1)) return not_tried();
    const void* const problem = problem_of(args[0]);
    const at::Tensor* const image = usual(args[3], dtype == 0 ? 4 : 2);
    const at::Tensor* const out = usual(args[4], 4);
    if (!problem || !image || !out || out->scalar_type() != at::kFloat || !stream_of(args[5], &stream)) return not_tried();
    const void* const pi = image->data_ptr();
    void* const po = out->data_ptr();
    const int64_t ni = image->numel(), no = out->numel();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_pool(problem, dtype, mode, pi, ni, po, no, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// setup(cacnn_internal_sized_interface(), size of Problem, Problem, address of cacnn_internal_conv_forward_sized, of cacnn_internal_pool_forward_sized);
// ImportError where the first two are not what this module was compiled for
PyObject* setup(PyObject*, PyObject* args) {
    PyObject *problem, *conv_at, *pool_at;
    int interface = 0;
    Py_ssize_t size = 0;
    if (!PyArg_ParseTuple(args, "inO!OO", &interface, &size, &PyType_Type, &problem, &conv_at, &pool_at)) return nullptr;
    if (interface != cacnn::kSizedInterface || size != kProblemBytes) {
        PyErr_SetString(PyExc_ImportError, "_cacnn_torch was compiled for another version of the library");
        return nullptr;
    }
    void* const c = PyLong_AsVoidPtr(conv_at);
    void* const p = PyLong_AsVoidPtr(pool_at);
    if (PyErr_Occurred()) return nullptr;
    Py_INCREF(problem);
    Py_XDECREF((PyObject*)g_problem);
    g_problem = (PyTypeObject*)problem;
    g_conv = (ConvFn)c;
    g_pool = (PoolFn)p;
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"conv", (PyCFunction)(void (*)(void))conv, METH_FASTCALL, nullptr},
    {"pool", (PyCFunction)(void (*)(void))pool, METH_FASTCALL, nullptr},
    {"setup", setup, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_cacnn_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__cacnn_torch() { return PyModule_Create(&g_module); }
