// The calls a learner and a server make on every step (ParameterServer.push,
// pull_many, apply_pull) from Python tensors to the C ABI in one native call:
// the checks of the binding, the arrays of ids and pointers, the call (with
// the interpreter's lock released), and the record of the streams that use the
// tensors. Through ctypes and torch's Python methods these took 1.4 us a push and
// 4.4 us a pull of one replica beside its launch.
//
// Each function returns the status, or None, with nothing done, for arguments
// it does not take (tensor subclasses, wrong sizes or types, objects that are
// not tensors): the Python binding then makes the call itself and raises what is
// to be raised.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ps.h"

namespace {

using PushFn = int (*)(ps_server *, int, const void *, int);
using PullsFn = int (*)(ps_server *, int, const int *, void *const *, int);

// Data pointer and dtype of an ordinary device tensor of n contiguous values;
// null for anything else.
void *plain(PyObject *o, int64_t n, int *dtype, at::Tensor *out) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    try {
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || t.layout() != at::kStrided || t.numel() != n || !t.is_contiguous())
            return nullptr;
        if (t.scalar_type() == at::kFloat) *dtype = PS_F32;
        else if (t.scalar_type() == at::kBFloat16) *dtype = PS_BF16;
        else return nullptr;
        *out = t;
        return t.data_ptr();
    } catch (...) {   // a functorch wrapper has no storage of its own
        return nullptr;
    }
}

// Mark t as used on the streams packed in `streams` (stream id, device index,
// device type; 64-bit each). False with a Python error set on failure.
bool used_on(const at::Tensor &t, const int64_t *streams, Py_ssize_t count) {
    try {
        for (Py_ssize_t i = 0; i < count; ++i)
            t.record_stream(c10::Stream::unpack3(
                streams[3 * i], static_cast<c10::DeviceIndex>(streams[3 * i + 1]),
                static_cast<c10::DeviceType>(streams[3 * i + 2])));
        return true;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "record_stream failed");
    }
    return false;
}

// Arguments every call starts with: the function's address, the handle, and
// at the end n and the packed streams.
struct Call {
    void *fn;
    ps_server *ps;
    int64_t n;
    const int64_t *streams;
    Py_ssize_t stream_count;
};

bool parse(Call &c, PyObject *fn, PyObject *h, PyObject *n, PyObject *streams) {
    c.fn = PyLong_AsVoidPtr(fn);
    c.ps = static_cast<ps_server *>(PyLong_AsVoidPtr(h));
    c.n = PyLong_AsLongLong(n);
    if (PyErr_Occurred()) return false;
    if (!PyBytes_Check(streams) || PyBytes_GET_SIZE(streams) % 24 != 0) {
        PyErr_SetString(PyExc_TypeError, "streams: packed bytes expected");
        return false;
    }
    c.streams = reinterpret_cast<const int64_t *>(PyBytes_AS_STRING(streams));
    c.stream_count = PyBytes_GET_SIZE(streams) / 24;
    return true;
}

// A C int from a Python int; false (no error set) for anything else.
bool small_int(PyObject *o, int *out) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < INT32_MIN || v > INT32_MAX) return false;
    *out = static_cast<int>(v);
    return true;
}

// push(ps_push_dtype, handle, learner, gradient, n, streams)
PyObject *push(PyObject *, PyObject *const *a, Py_ssize_t count) {
    Call c;
    if (count != 6) return PyErr_Format(PyExc_TypeError, "push takes 6 arguments");
    if (!parse(c, a[0], a[1], a[4], a[5])) return nullptr;
    int learner, dtype;
    at::Tensor t;
    if (!small_int(a[2], &learner)) Py_RETURN_NONE;
    void *grad = plain(a[3], c.n, &dtype, &t);
    if (grad == nullptr) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = reinterpret_cast<PushFn>(c.fn)(c.ps, learner, grad, dtype);
    Py_END_ALLOW_THREADS
    if (rc == PS_OK && !used_on(t, c.streams, c.stream_count)) return nullptr;
    return PyLong_FromLong(rc);
}

// pulls(ps_pull_many or ps_apply_pull, handle, learners, replicas, n, streams)
PyObject *pulls(PyObject *, PyObject *const *a, Py_ssize_t count) {
    Call c;
    if (count != 6) return PyErr_Format(PyExc_TypeError, "pulls takes 6 arguments");
    if (!parse(c, a[0], a[1], a[4], a[5])) return nullptr;
    if (!PyList_CheckExact(a[3]) && !PyTuple_CheckExact(a[3])) Py_RETURN_NONE;
    if (!PyList_CheckExact(a[2]) && !PyTuple_CheckExact(a[2]) && !PyRange_Check(a[2]))
        Py_RETURN_NONE;
    PyObject *ids = PySequence_Fast(a[2], "learners");
    if (ids == nullptr) return nullptr;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(a[3]);
    int learners[PS_MAX_REPLICAS], code = PS_F32;
    void *dsts[PS_MAX_REPLICAS];
    at::Tensor t[PS_MAX_REPLICAS];
    bool ok = n <= PS_MAX_REPLICAS && PySequence_Fast_GET_SIZE(ids) == n;
    for (Py_ssize_t i = 0; ok && i < n; ++i) {
        int dtype;
        dsts[i] = plain(PySequence_Fast_GET_ITEM(a[3], i), c.n, &dtype, &t[i]);
        ok = dsts[i] != nullptr && (i == 0 || dtype == code) &&
             small_int(PySequence_Fast_GET_ITEM(ids, i), &learners[i]);
        if (ok) code = dtype;
    }
    Py_DECREF(ids);
    if (!ok) Py_RETURN_NONE;
    // before the call, as the binding does: a refused pull marks them too
    for (Py_ssize_t i = 0; i < n; ++i)
        if (!used_on(t[i], c.streams, c.stream_count)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = reinterpret_cast<PullsFn>(c.fn)(c.ps, static_cast<int>(n), learners, dsts, code);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"push", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(push)), METH_FASTCALL,
     "push(function, handle, learner, gradient, n, streams) -> status or None"},
    {"pulls", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pulls)), METH_FASTCALL,
     "pulls(function, handle, learners, replicas, n, streams) -> status or None"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
