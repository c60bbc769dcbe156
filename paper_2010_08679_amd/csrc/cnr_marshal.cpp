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

// ---- the calls of a BatchCheckpointer ------------------------------------------------------------------
// batch_jobs(checkpointers, stage, tensors, outputs): the bytes of the job array of one stage of a batch, in one step from the objects that own
// the buffers; for the mark (bytes, index type).  Only what is in order in every respect is taken here: None is returned for anything else,
// and the caller's general way answers or refuses it.  Nothing is kept from one call to the next.  (An iteration's mark of eight tables as
// called 8.7 -> 6.9 us, of which the GPU is busy for 6.5; the five calls of a small checkpoint 26 -> 23 us on the host, fifteen of them the launches.)
enum Stage { kClear, kMark, kCompact, kRows };
const char *const kNames[] = {"n_rows", "dim", "capacity", "bitmap", "mark_scratch", "row_ids", "n_dirty", "scratch", "scale", "bias", "packed", "bits", "row_min", "row_max"};
enum Name { kNRows, kDim, kCapacity, kBitmap, kMarkScratch, kRowIds, kNDirty, kScratch, kScale, kBias, kPacked, kBits, kRowMin, kRowMax, kNameCount };
PyObject *names[kNameCount];

// The fields of cnr_table_job, in order.
enum Field { fTable, fNRows, fBitmap, fIndices, fNIndices, fMarkScratch, fRowIds, fCapacity, fNDirty, fScratch, fScale, fBias, fRowMin, fRowMax, fCodes, fPacked };

bool number(PyObject *owner, Name name, unsigned long long &out) {
    THPObjectPtr v(PyObject_GetAttr(owner, names[name]));
    if (!v || !PyLong_CheckExact(v.get())) return false;
    int overflow;
    const long long x = PyLong_AsLongLongAndOverflow(v.get(), &overflow);
    out = (unsigned long long)x;
    return !overflow && x >= 0;
}
// Address of a plain contiguous GPU tensor of this type (Undefined: any) with at least `least` elements.
bool plain(PyObject *v, at::ScalarType type, unsigned long long least, unsigned long long &out, unsigned long long *count = nullptr) {
    if (!THPVariable_CheckExact(v)) return false;
    const at::Tensor &t = THPVariable_Unpack(v);
    if (!t.is_cuda() || (type != at::ScalarType::Undefined && t.scalar_type() != type) || !t.is_contiguous()) return false;
    const unsigned long long n = (unsigned long long)t.numel();
    if (n < least) return false;
    if (count) *count = n;
    out = (unsigned long long)(uintptr_t)t.data_ptr();
    return true;
}
bool tensor(PyObject *owner, Name name, at::ScalarType type, bool may_be_none, unsigned long long least, unsigned long long &out) {
    THPObjectPtr v(PyObject_GetAttr(owner, names[name]));
    if (!v) return false;
    if (v.get() == Py_None) return may_be_none;  // out stays 0
    return plain(v.get(), type, least, out);
}
PyObject *item(PyObject *seq, Py_ssize_t i) {  // borrowed, of a list or a tuple
    if (PyList_CheckExact(seq)) return i < PyList_GET_SIZE(seq) ? PyList_GET_ITEM(seq, i) : nullptr;
    if (PyTuple_CheckExact(seq)) return i < PyTuple_GET_SIZE(seq) ? PyTuple_GET_ITEM(seq, i) : nullptr;
    return nullptr;
}
bool job(PyObject *owner, long stage, PyObject *t, PyObject *o, unsigned long long (&f)[kJobFields], at::ScalarType &index_type) {
    constexpr at::ScalarType i32 = at::kInt, i64 = at::kLong, f32 = at::kFloat, u8 = at::kByte, any = at::ScalarType::Undefined;
    if (!number(owner, kNRows, f[fNRows])) return false;
    if (stage != kRows && !tensor(owner, kBitmap, i32, false, 0, f[fBitmap])) return false;
    if (stage == kMark) {
        if (!tensor(owner, kMarkScratch, any, true, 0, f[fMarkScratch])) return false;
        if (t == Py_None) return true;
        if (!plain(t, any, 0, f[fIndices], &f[fNIndices])) return false;
        const at::ScalarType type = THPVariable_Unpack(t).scalar_type();
        if ((type != i32 && type != i64) || (index_type != any && index_type != type)) return false;
        index_type = type;
        return true;
    }
    if (stage == kClear) return true;
    if (!tensor(owner, kRowIds, i32, false, 0, f[fRowIds]) || !number(owner, kCapacity, f[fCapacity]) || !tensor(owner, kNDirty, i64, false, 0, f[fNDirty])) return false;
    if (stage == kCompact) return tensor(owner, kScratch, any, false, 0, f[fScratch]);
    unsigned long long dim, bits;
    if (!number(owner, kDim, dim) || !number(o, kBits, bits)) return false;
    if ((bits != 2 && bits != 3 && bits != 4 && bits != 8) || dim == 0 || dim > 1u << 20 || dim * bits % 8 || f[fNRows] >> 32 || f[fCapacity] >> 32) return false;
    const unsigned long long cap = f[fCapacity] ? f[fCapacity] : 1;
    return plain(t, f32, f[fNRows] * dim, f[fTable]) && tensor(o, kScale, f32, false, cap, f[fScale]) && tensor(o, kBias, f32, false, cap, f[fBias]) &&
           tensor(o, kRowMin, f32, true, 0, f[fRowMin]) && tensor(o, kRowMax, f32, true, 0, f[fRowMax]) &&
           tensor(o, kPacked, u8, false, cap * (dim * bits / 8), f[fPacked]);
}
PyObject *batch_jobs(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 4 || !PyList_CheckExact(args[0]) || !PyLong_CheckExact(args[1])) Py_RETURN_NONE;
    const long stage = PyLong_AsLong(args[1]);
    const Py_ssize_t rows = PyList_GET_SIZE(args[0]);
    THPObjectPtr bytes(PyBytes_FromStringAndSize(nullptr, rows * kJobFields * 8));
    if (!bytes) return nullptr;
    at::ScalarType index_type = at::ScalarType::Undefined;
    bool good = stage >= kClear && stage <= kRows;
    try {
        for (Py_ssize_t i = 0; i < rows && good; ++i) {
            // held: an attribute of an unusual object can run code that takes them out of their lists
            PyObject *owner = item(args[0], i), *t = stage == kMark || stage == kRows ? item(args[2], i) : Py_None, *o = stage == kRows ? item(args[3], i) : Py_None;
            if (!owner || !t || !o) {
                good = false;
                break;
            }
            Py_INCREF(owner);
            Py_INCREF(t);
            Py_INCREF(o);
            THPObjectPtr hold_owner(owner), hold_t(t), hold_o(o);
            unsigned long long f[kJobFields] = {};
            good = job(owner, stage, t, o, f, index_type);
            memcpy(PyBytes_AS_STRING(bytes.get()) + i * kJobFields * 8, f, sizeof(f));
        }
        // look-ups beyond the last table are not marked, but none may be of another type
        if (stage == kMark)
            for (Py_ssize_t i = rows; good; ++i) {
                PyObject *t = item(args[2], i);
                if (!t) break;
                good = t == Py_None || (THPVariable_CheckExact(t) && THPVariable_Unpack(t).scalar_type() == index_type);
            }
    } catch (...) {  // a tensor that has no address; the general way meets and reports it
        good = false;
    }
    if (!good || (stage == kMark && index_type == at::ScalarType::Undefined)) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (stage != kMark) return bytes.release();
    return Py_BuildValue("(NO)", bytes.release(), index_type == at::kInt ? Py_False : Py_True);
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
    {"batch_jobs", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(batch_jobs)), METH_FASTCALL,
     "batch_jobs(checkpointers, stage, tensors, outputs): the bytes of a batch's job array, or None where the general way has to look"},
    {"set_general", set_general, METH_O, "set_general(f): what answers for tensors of other types"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    for (int i = 0; i < kNameCount; ++i)
        if (!names[i] && !(names[i] = PyUnicode_InternFromString(kNames[i]))) return nullptr;
    return PyModule_Create(&module);
}
