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

// What is asked of the tensors of a list: how many there are (any number where count < 0), their elements and type.
struct Wanted {
    long long count = -1, low = 0, high = INT64_MAX;
    PyObject* dtype = Py_None;
};

// Fills `w` from (count, low, high, dtype); false with an exception set.
bool wanted(PyObject* const* args, Wanted& w)
{
    w.count = PyLong_AsLongLong(args[0]);
    w.low = PyLong_AsLongLong(args[1]);
    w.high = PyLong_AsLongLong(args[2]);
    w.dtype = args[3];
    return !PyErr_Occurred();
}

// Whether `seq` is a list or tuple of as many tensors as are wanted, each of which is as wanted and `use` takes it.
template <typename Use>
bool all_as_wanted(PyObject* seq, const Wanted& w, Use use)
{
    if (!plain_sequence(seq)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    if ((w.count >= 0 && n != w.count) || (w.dtype != Py_None && !THPDtype_Check(w.dtype))) return false;
    try {
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject* o = PySequence_Fast_GET_ITEM(seq, i);
            if (!THPVariable_CheckExact(o)) return false;
            const at::Tensor& t = THPVariable_Unpack(o);
            const long long elems = t.numel();
            if (elems < w.low || elems > w.high) return false;
            if (w.dtype != Py_None && t.scalar_type() != reinterpret_cast<THPDtype*>(w.dtype)->scalar_type) return false;
            if (!use(i, t)) return false;
        }
    } catch (...) {
        return false;
    }
    return true;
}

// pointers(tensors[, count, low, high, dtype or None]) -> bytes: the addresses, 8 bytes each; None unless all are
// contiguous device tensors and, where that is asked, as `sized` wants them.
PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    Wanted w;
    if (nargs != 1 && nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "pointers takes one argument or five");
        return nullptr;
    }
    if (nargs == 5 && !wanted(args + 1, w)) return nullptr;
    if (!plain_sequence(args[0])) Py_RETURN_NONE;
    PyObject* out = PyBytes_FromStringAndSize(nullptr, PySequence_Fast_GET_SIZE(args[0]) * (Py_ssize_t)sizeof(void*));
    if (!out) return nullptr;
    void** p = reinterpret_cast<void**>(PyBytes_AS_STRING(out));
    const bool usable = all_as_wanted(args[0], w, [&](Py_ssize_t i, const at::Tensor& t) {
        if (!t.is_cuda() || !t.is_contiguous()) return false;
        p[i] = t.data_ptr();
        return true;
    });
    if (usable) return out;
    Py_DECREF(out);
    Py_RETURN_NONE;
}

// sized(tensors, count, low, high, dtype or None) -> bool: whether there are `count` tensors, each of low .. high elements
// and of that dtype.
PyObject* sized(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    Wanted w;
    if (nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "sized takes five arguments");
        return nullptr;
    }
    if (!wanted(args + 1, w)) return nullptr;
    if (w.count < 0) Py_RETURN_FALSE;
    return PyBool_FromLong(all_as_wanted(args[0], w, [](Py_ssize_t, const at::Tensor&) { return true; }));
}

PyMethodDef methods[] = {
    {"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pointers)), METH_FASTCALL, nullptr},
    {"sized", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(sized)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tq_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tq_marshal() { return PyModule_Create(&module); }
