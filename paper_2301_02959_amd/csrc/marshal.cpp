// The binding's per-tensor check and pointer, in native code: device_pointer(tensor, dtypes=None) returns the data pointer
// of a contiguous CUDA tensor whose dtype is in the tuple `dtypes` (None: any), None for None, and hands whatever else,
// a tensor subclass or wrapper included, to the function given to set_fallback, which looks at it in Python and raises.
// A call of the router passes nine tensors; four attribute reads and a call each in Python are 0.31 us a tensor, this is 0.07.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

static PyObject* fallback = nullptr;

static PyObject* set_fallback(PyObject*, PyObject* fn)
{
    Py_INCREF(fn);
    Py_XDECREF(fallback);
    fallback = fn;
    Py_RETURN_NONE;
}

// The pointer as a Python integer, or null (and no Python error) where the fallback has to look.
static PyObject* plain_pointer(PyObject* obj, PyObject* dtypes)
{
    if (!THPVariable_CheckExact(obj) || (dtypes != Py_None && !PyTuple_CheckExact(dtypes))) return nullptr;
    try {
        const at::Tensor& t = THPVariable_Unpack(obj);
        if (!t.is_cuda() || !t.is_contiguous()) return nullptr;
        if (dtypes != Py_None) {
            const at::ScalarType have = t.scalar_type();
            bool found = false;
            for (Py_ssize_t k = 0; k < PyTuple_GET_SIZE(dtypes) && !found; ++k) {
                PyObject* const want = PyTuple_GET_ITEM(dtypes, k);
                found = THPDtype_Check(want) && reinterpret_cast<THPDtype*>(want)->scalar_type == have;
            }
            if (!found) return nullptr;
        }
        return PyLong_FromUnsignedLongLong(reinterpret_cast<unsigned long long>(t.data_ptr()));
    } catch (...) {                               // a wrapper without storage: Python says so
        PyErr_Clear();
        return nullptr;
    }
}

static PyObject* device_pointer(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (nargs < 1 || nargs > 2 || fallback == nullptr) {
        PyErr_SetString(PyExc_TypeError, "device_pointer(tensor, dtypes=None), after set_fallback");
        return nullptr;
    }
    if (args[0] == Py_None) Py_RETURN_NONE;
    PyObject* const pointer = plain_pointer(args[0], nargs == 2 ? args[1] : Py_None);
    if (pointer != nullptr || PyErr_Occurred()) return pointer;
    return PyObject_Vectorcall(fallback, args, (size_t)nargs, nullptr);
}

static PyMethodDef methods[] = {
    {"device_pointer", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(device_pointer)), METH_FASTCALL,
     "device_pointer(tensor, dtypes=None): data pointer of a contiguous CUDA tensor"},
    {"set_fallback", set_fallback, METH_O, "set_fallback(function): what device_pointer calls for anything but such a tensor"},
    {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

// built_for: the torch whose headers this was compiled with.  Its objects' layouts are compiled in, so the binding takes no
// other's.
PyMODINIT_FUNC PyInit__marshal()
{
    PyObject* const m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", FS_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
