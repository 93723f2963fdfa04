// The binding's way from lists of torch tensors to one call of the C ABI: checks
// every buffer as binding.py's _pointers does, collects the device pointers and
// makes the call, in one step.  In Python the same took 5 to 6 us a call, more
// than the launch (about 3.5 us) and, for small plans, than the kernel.
//
// call(fn, plan, desc, kind_a, list_a, kind_b, list_b, stream) -> the call's return
// code, or None for anything that is not plainly in order: the caller then goes
// the way through Python, which reports what is wrong (or copes with objects that
// are no plain tensors).  Nothing is kept from one call to the next.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "hp.h"

namespace {

// Filled in once per plan by binding.py (Plan._desc); the same layout there.
struct Desc {
    int64_t n_src, n_dst, dst_rows, hidden, elem_bytes;
    const int64_t *src_rows;
};

enum Kind { kSrc = 0, kDst = 1, kAccum = 2 };     // kAccum: binary32 accumulators in the place of source buffers

typedef int (*Call)(const void *plan, const void *const *a, void *const *b, void *stream);

// The device pointers of a list (or tuple) of tensors; false if any of it is not plainly in order.
bool pointers(PyObject *list, Kind kind, const Desc &d, void **out) {
    const bool is_list = PyList_CheckExact(list);
    if (!is_list && !PyTuple_CheckExact(list)) return false;
    const int64_t n = is_list ? PyList_GET_SIZE(list) : PyTuple_GET_SIZE(list);
    if (n != (kind == kDst ? d.n_dst : d.n_src) || n > HP_MAX_BUFFERS) return false;
    const int64_t elem = kind == kAccum ? 4 : d.elem_bytes;
    for (int64_t i = 0; i < n; ++i) {
        PyObject *o = is_list ? PyList_GET_ITEM(list, i) : PyTuple_GET_ITEM(list, i);
        if (o == Py_None) {
            out[i] = nullptr;
            continue;
        }
        if (!THPVariable_CheckExact(o)) return false;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (t.unsafeGetTensorImpl()->is_python_dispatch() || !t.has_storage()) return false;
        const int64_t rows = kind == kDst ? d.dst_rows : d.src_rows[i];
        if (!t.is_cuda() || !t.is_contiguous() || (int64_t)t.element_size() != elem || t.numel() < rows * d.hidden) return false;
        out[i] = t.numel() ? t.data_ptr() : nullptr;
    }
    return true;
}

// A stream argument: None, an object with a cuda_stream, or a number.
bool stream_of(PyObject *o, void **out) {
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    PyObject *v = PyLong_CheckExact(o) ? Py_NewRef(o) : PyObject_GetAttrString(o, "cuda_stream");
    if (v) {
        *out = PyLong_AsVoidPtr(v);
        Py_DECREF(v);
    }
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    if (n_args != 8) {
        PyErr_SetString(PyExc_TypeError, "call takes 8 arguments");
        return nullptr;
    }
    const Call fn = (Call)PyLong_AsVoidPtr(args[0]);
    const void *plan = PyLong_AsVoidPtr(args[1]);
    const Desc *desc = (const Desc *)PyLong_AsVoidPtr(args[2]);
    const long kind_a = PyLong_AsLong(args[3]), kind_b = PyLong_AsLong(args[5]);
    if (PyErr_Occurred()) return nullptr;
    if (!fn || !plan || !desc) Py_RETURN_NONE;
    void *a[HP_MAX_BUFFERS], *b[HP_MAX_BUFFERS], *stream = nullptr;
    try {
        if (!pointers(args[4], (Kind)kind_a, *desc, a) || !pointers(args[6], (Kind)kind_b, *desc, b) ||
            !stream_of(args[7], &stream))
            Py_RETURN_NONE;
    } catch (const std::exception &) {
        Py_RETURN_NONE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(plan, a, b, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "hp_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_hp_marshal(void) {
    PyObject *m = PyModule_Create(&module);
    // a tensor's layout is that of the torch it was compiled against: the binding compares
    if (m && PyModule_AddStringConstant(m, "torch_version", HP_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
