// Arguments of the library's calls from Python: device addresses of checked tensors, and whole job arrays.
//
// A call of the library is one or two launches of a few microseconds, and what its caller in Python does beforehand
// is checks of up to twelve tensors (of dozens for a batch): four attributes of each and an object for its
// address, 0.26 to 0.34 us apiece in Python, 0.06 here.  An iteration's mark of eight tables 19 us a call with the checks in
// Python, small checkpoints 50 us.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

namespace {

constexpr Py_ssize_t kJobFields = 16;  // of cnr_table_job, each 64 bits

PyObject *general = nullptr;  // address() of anything but plain tensors and parameters

// Device address of a contiguous GPU tensor of the given dtype (None: any); 0 for None.  False: a Python error is set.
bool address_of(PyObject *t, PyObject *dtype, PyObject *name, unsigned long long &out) {
    out = 0;
    if (t == Py_None) return true;
    if (!THPVariable_CheckExact(t)) {  // subclasses answer for themselves; the rest is refused there
        THPObjectPtr r(PyObject_CallFunctionObjArgs(general, t, dtype, name, nullptr));
        if (!r) return false;
        out = PyLong_AsUnsignedLongLong(r.get());
        return !PyErr_Occurred();
    }
    const at::Tensor &v = THPVariable_Unpack(t);
    if (!v.is_cuda()) {
        PyErr_Format(PyExc_TypeError, "%S must be a tensor on the GPU", name);
        return false;
    }
    if (dtype != Py_None) {
        if (!THPDtype_Check(dtype)) {
            PyErr_SetString(PyExc_TypeError, "dtype must be a torch.dtype or None");
            return false;
        }
        if (v.scalar_type() != reinterpret_cast<THPDtype *>(dtype)->scalar_type) {
            PyObject *got = PyObject_GetAttrString(t, "dtype");
            if (got) PyErr_Format(PyExc_TypeError, "%S must be %S, got %S", name, dtype, got);
            Py_XDECREF(got);
            return false;
        }
    }
    if (!v.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%S must be contiguous", name);
        return false;
    }
    out = (unsigned long long)(uintptr_t)v.data_ptr();
    return true;
}

PyObject *address(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "address(tensor, dtype, name)");
        return nullptr;
    }
    unsigned long long p;
    return address_of(args[0], args[1], args[2], p) ? PyLong_FromUnsignedLongLong(p) : nullptr;
    END_HANDLE_TH_ERRORS
}

// A field of a job: a number where `kind` is the type int (anything with __index__), else an address, of a tensor of dtype `kind` or for
// None or the number 0, a field that the call does not read.
bool field(PyObject *v, PyObject *kind, PyObject *name, unsigned long long &out) {
    if (kind == reinterpret_cast<PyObject *>(&PyLong_Type)) {
        if (PyLong_CheckExact(v)) {
            out = PyLong_AsUnsignedLongLong(v);
        } else {
            THPObjectPtr index(PyNumber_Index(v));
            if (!index) return false;
            out = PyLong_AsUnsignedLongLong(index.get());
        }
        return out != ~0ull || !PyErr_Occurred();
    }
    out = 0;
    if (v == Py_None) return true;
    if (PyLong_CheckExact(v)) {
        int overflow;
        if (PyLong_AsLongLongAndOverflow(v, &overflow) == 0 && !overflow) return true;
    }
    return address_of(v, kind, name, out);
}

// pack_jobs(rows, kinds, names): rows of sixteen fields, the struct's in order; the bytes of the array.
PyObject *pack_jobs(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 3 || !PyList_Check(args[0]) || !PyTuple_Check(args[1]) || !PyTuple_Check(args[2]) ||
        PyTuple_GET_SIZE(args[1]) != kJobFields || PyTuple_GET_SIZE(args[2]) != kJobFields) {
        PyErr_SetString(PyExc_TypeError, "pack_jobs(list of rows, kinds, names)");
        return nullptr;
    }
    const Py_ssize_t rows = PyList_GET_SIZE(args[0]);
    THPObjectPtr bytes(PyBytes_FromStringAndSize(nullptr, rows * kJobFields * 8));  // given back if a tensor throws, too
    if (!bytes) return nullptr;
    for (Py_ssize_t i = 0; i < rows; ++i) {
        // the list can change hands while a subclass answers: its length is looked at again, the row is held
        PyObject *at = i < PyList_GET_SIZE(args[0]) ? PyList_GET_ITEM(args[0], i) : nullptr;
        if (!at || !PyTuple_Check(at) || PyTuple_GET_SIZE(at) != kJobFields) {
            PyErr_SetString(PyExc_TypeError, "a job has sixteen fields");
            return nullptr;
        }
        Py_INCREF(at);
        THPObjectPtr row(at);
        for (Py_ssize_t f = 0; f < kJobFields; ++f) {
            unsigned long long x;
            if (!field(PyTuple_GET_ITEM(at, f), PyTuple_GET_ITEM(args[1], f), PyTuple_GET_ITEM(args[2], f), x)) return nullptr;
            memcpy(PyBytes_AS_STRING(bytes.get()) + (i * kJobFields + f) * 8, &x, 8);
        }
    }
    return bytes.release();
    END_HANDLE_TH_ERRORS
}

PyObject *set_general(PyObject *, PyObject *f) {
    Py_INCREF(f);
    Py_XSETREF(general, f);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"address", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(address)), METH_FASTCALL,
     "address(tensor, dtype, name): device address of a contiguous GPU tensor, 0 for None"},
    {"pack_jobs", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(pack_jobs)), METH_FASTCALL,
     "pack_jobs(rows, kinds, names): the bytes of an array of cnr_table_job"},
    {"set_general", set_general, METH_O, "set_general(f): what answers for tensors of other types"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
