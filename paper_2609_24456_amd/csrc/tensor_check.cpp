// The Python binding's check of one tensor argument, natively: type, dtype,
// size, contiguity and device in one call (about 0.1 us; the same checks through
// torch's Python attributes take 0.75 us, and a delivery step makes fifteen of
// them, which kept the GPU waiting on small batches).  It only ever says yes:
// whatever it does not accept, the binding checks again in Python, which raises
// the error or knows better.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

bool dtype_is(PyObject* want, at::ScalarType have) {
    return THPDtype_Check(want) && reinterpret_cast<THPDtype*>(want)->scalar_type == have;
}

// A size in bytes or elements: None (no requirement, 0) or an int; false on anything else
bool read_size(PyObject* o, long long* n) {
    if (o == Py_None) {
        *n = 0;
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    *n = PyLong_AsLongLong(o);
    if (*n == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// address(t, dtype, nbytes, numel): the device address of a plain contiguous
// tensor on a HIP device, of dtype `dtype` (a dtype, a tuple of them or None)
// and holding at least `nbytes` bytes and `numel` elements (None: any); None if
// it is anything else.
PyObject* address(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 4) {
        PyErr_SetString(PyExc_TypeError, "address takes (tensor, dtype, nbytes, numel)");
        return nullptr;
    }
    long long nbytes = 0, numel = 0;
    if (!THPVariable_CheckExact(args[0]) || !read_size(args[2], &nbytes) || !read_size(args[3], &numel)) Py_RETURN_NONE;
    uintptr_t p = 0;
    try {
        const at::Tensor& t = THPVariable_Unpack(args[0]);
        PyObject* want = args[1];
        if (want != Py_None) {
            bool ok = false;
            if (PyTuple_CheckExact(want)) {
                for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(want) && !ok; ++i)
                    ok = dtype_is(PyTuple_GET_ITEM(want, i), t.scalar_type());
            } else {
                ok = dtype_is(want, t.scalar_type());
            }
            if (!ok) Py_RETURN_NONE;
        }
        const long long n = t.numel();
        if (!t.is_cuda() || n * (long long)t.element_size() < nbytes || n < numel || !t.is_contiguous()) Py_RETURN_NONE;
        p = reinterpret_cast<uintptr_t>(t.data_ptr());
    } catch (...) {  // a wrapper without storage, a symbolic size: the Python path says so
        Py_RETURN_NONE;
    }
    return PyLong_FromUnsignedLongLong((unsigned long long)p);
}

PyMethodDef methods[] = {
    {"address", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(address)), METH_FASTCALL,
     "device address of a checked tensor argument, or None"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tensor_check", "checks of the binding's tensor arguments", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tensor_check(void) {
    PyObject* m = PyModule_Create(&module);
    // the layouts read above are this torch's: the binding uses no other's
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION_BUILT) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
