// _tq_marshal: the per-tensor part of the Python binding.  A batched call takes up to four lists of tensors, of each of
// which the binding wants to know that it is a contiguous device tensor of the right size, and its address; in Python
// that is five attribute calls a tensor and, for small tensors, as long as the launches themselves.
//
// Both functions look at plain tensors (torch.Tensor, nn.Parameter) in a list or tuple and at nothing else: anything
// they do not know, or that raises, is left to the caller's own Python code, which raises the error.
#include <cstdint>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

// Not their subclasses: what one of those hands out may differ from what it stores.
bool plain_sequence(PyObject* seq) { return PyList_CheckExact(seq) || PyTuple_CheckExact(seq); }

// pointers(tensors) -> bytes: the addresses, 8 bytes each; None unless all are contiguous device tensors.
PyObject* pointers(PyObject*, PyObject* seq)
{
    if (!plain_sequence(seq)) Py_RETURN_NONE;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    PyObject* out = PyBytes_FromStringAndSize(nullptr, n * (Py_ssize_t)sizeof(void*));
    if (!out) return nullptr;
    void** p = reinterpret_cast<void**>(PyBytes_AS_STRING(out));
    try {
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject* o = PySequence_Fast_GET_ITEM(seq, i);
            bool usable = THPVariable_CheckExact(o);
            if (usable) {
                const at::Tensor& t = THPVariable_Unpack(o);
                usable = t.is_cuda() && t.is_contiguous();
                if (usable) p[i] = t.data_ptr();
            }
            if (!usable) {
                Py_DECREF(out);
                Py_RETURN_NONE;
            }
        }
    } catch (...) {
        Py_DECREF(out);
        Py_RETURN_NONE;
    }
    return out;
}

// sized(tensors, count, low, high, dtype or None) -> bool: whether there are `count` tensors, each of low .. high elements
// and of that dtype.
PyObject* sized(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "sized takes five arguments");
        return nullptr;
    }
    PyObject* seq = args[0];
    const long long count = PyLong_AsLongLong(args[1]), low = PyLong_AsLongLong(args[2]), high = PyLong_AsLongLong(args[3]);
    if (PyErr_Occurred()) return nullptr;
    if (!plain_sequence(seq) || PySequence_Fast_GET_SIZE(seq) != count) Py_RETURN_FALSE;
    if (args[4] != Py_None && !THPDtype_Check(args[4])) Py_RETURN_FALSE;
    try {
        for (Py_ssize_t i = 0; i < count; ++i) {
            PyObject* o = PySequence_Fast_GET_ITEM(seq, i);
            if (!THPVariable_CheckExact(o)) Py_RETURN_FALSE;
            const at::Tensor& t = THPVariable_Unpack(o);
            const long long n = t.numel();
            if (n < low || n > high) Py_RETURN_FALSE;
            if (args[4] != Py_None && t.scalar_type() != reinterpret_cast<THPDtype*>(args[4])->scalar_type) Py_RETURN_FALSE;
        }
    } catch (...) {
        Py_RETURN_FALSE;
    }
    Py_RETURN_TRUE;
}

PyMethodDef methods[] = {
    {"pointers", pointers, METH_O, nullptr},
    {"sized", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(sized)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tq_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tq_marshal() { return PyModule_Create(&module); }
