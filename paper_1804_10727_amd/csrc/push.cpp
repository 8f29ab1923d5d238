// The way of a push from Python into the library: the tensor's address and sizes are read, and the library called, without a step
// through the interpreter.  What waits for the host is pushes that are held back: 37 audio streams, 501 pushes in 32 launches, 574 us by
// ctypes, 514 so.  A launch per push mostly waits for the GPU, or for the launch itself (one sensor, 4,096 pushes, by the speed of the
// launches in a process 14,020 : 13,750 and 18,690 : 17,010; 64 audio streams 5,578 : 5,593).
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>
#include <cstring>
#include <vector>

namespace {

typedef int (*PushFn)(void *streams, const int32_t *stream_ids, int n_ids, const void *dev_rows, int n_rows);
PushFn push_fn = nullptr;

PyObject *bind(PyObject *, PyObject *address)
{
    void *p = PyLong_AsVoidPtr(address);
    if (PyErr_Occurred()) return nullptr;
    push_fn = reinterpret_cast<PushFn>(p);
    Py_RETURN_NONE;
}

struct Ids {                                       // a copy: other threads run while the library does
    int32_t few[64];
    std::vector<int32_t> many;
    const int32_t *at = nullptr;
    int n = 0;
    // One axis of int32 values; anything else is for the caller to convert.
    bool take(PyObject *o)
    {
        Py_buffer b;
        if (!PyObject_CheckBuffer(o)) return false;
        if (PyObject_GetBuffer(o, &b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) { PyErr_Clear(); return false; }
        const bool ok = b.ndim == 1 && b.itemsize == 4 && b.format && strcmp(b.format, "i") == 0 && b.len / 4 <= INT_MAX;
        if (ok) {
            n = (int)(b.len / 4);
            int32_t *to = few;
            try {
                if (n > 64) { many.resize(n); to = many.data(); }
            } catch (...) { PyBuffer_Release(&b); return false; }
            if (n > 0) memcpy(to, b.buf, (size_t)b.len);
            at = to;
        }
        PyBuffer_Release(&b);
        return ok;
    }
};

// push(streams, rows, stream_ids or None, n_rows or None): what idf_push_segment returned, or None where the arguments are not plain
// tensors and arrays of the usual kinds, or are wrong: those go the long way round, which converts them or raises.
PyObject *push(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    if (n_args != 4 || !push_fn) { PyErr_SetString(PyExc_TypeError, "push(streams, rows, stream_ids, n_rows)"); return nullptr; }
    if (!THPVariable_CheckExact(args[1])) Py_RETURN_NONE;
    void *streams = PyLong_AsVoidPtr(args[0]);
    if (PyErr_Occurred()) return nullptr;
    int64_t n_ids = 0, n_rows = 0;
    const void *rows = nullptr;
    Ids ids;
    try {
        const at::Tensor &t = THPVariable_Unpack(args[1]);
        if (!t.is_cuda() || !t.is_contiguous() || t.dim() < 2) Py_RETURN_NONE;
        n_ids = t.size(0);
        n_rows = t.size(1);
        rows = t.data_ptr();
    } catch (...) { Py_RETURN_NONE; }              // (tensors without memory of their own)
    if (args[2] != Py_None) {
        if (!ids.take(args[2])) Py_RETURN_NONE;
        n_ids = ids.n;
    }
    if (args[3] != Py_None) {
        if (!PyLong_CheckExact(args[3])) Py_RETURN_NONE;
        n_rows = PyLong_AsLongLong(args[3]);
        if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    }
    if (n_ids > INT_MAX || n_rows > INT_MAX || n_rows < INT_MIN) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = push_fn(streams, ids.at, (int)n_ids, rows, (int)n_rows);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"bind", bind, METH_O, "the address of idf_push_segment"},
    {"push", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(push)), METH_FASTCALL, "idf_push_segment on a tensor"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_push", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__push() { return PyModule_Create(&module); }
