// The Python binding's tensor checks and pointers, natively: one call takes
// all tensors of an entry point.  In Python each tensor's type, device, dtype,
// layout, size and address cost about a microsecond, so that a receive of 64
// sources spent longer on its 128 small tensors than the GPU on the pass.
//
// A check that fails, or a tensor this file does not know to treat (a
// subclass, a wrapper without storage), is answered with None: the binding
// then runs its own checks, which raise the error or accept the tensor.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <vector>

namespace {

// dtypes an argument may have, as bits of a mask (kOptional: None may stand
// in the tensor's place)
enum : unsigned { kF32 = 1, kBF16 = 2, kI16 = 4, kU16 = 8, kI8 = 16, kU8 = 32, kOptional = 64 };

unsigned dtype_bit(at::ScalarType t) {
    switch (t) {
    case at::kFloat: return kF32;
    case at::kBFloat16: return kBF16;
    case at::kShort: return kI16;
    case at::kUInt16: return kU16;
    case at::kChar: return kI8;
    case at::kByte: return kU8;
    default: return 0;
    }
}

// The address of a contiguous tensor of device `device` with one of the
// dtypes of `mask` and at least `need` elements.
bool address(PyObject *o, long device, unsigned mask, long long need, void **out) {
    if (!THPVariable_CheckExact(o))
        return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.device().index() != device || !(dtype_bit(t.scalar_type()) & mask) ||
        !t.is_contiguous() || t.numel() < need)
        return false;
    *out = t.data_ptr();
    return true;
}

// addresses(device, tensor, mask, need, tensor, mask, need, ...): a tuple of
// addresses (None for an optional tensor that is not given), or None.
PyObject *addresses(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n < 1 || (n - 1) % 3) {
        PyErr_SetString(PyExc_TypeError, "addresses(device, (tensor, mask, need)...)");
        return nullptr;
    }
    const long device = PyLong_AsLong(args[0]);
    const Py_ssize_t count = (n - 1) / 3;
    PyObject *result = PyTuple_New(count);
    if (!result)
        return nullptr;
    try {
        for (Py_ssize_t i = 0; i < count; ++i) {
            PyObject *const *a = args + 1 + 3 * i;
            PyObject *value = Py_None;
            const unsigned mask = (unsigned)PyLong_AsUnsignedLong(a[1]);
            if (a[0] != Py_None || !(mask & kOptional)) {
                void *p = nullptr;
                const long long need = PyLong_AsLongLong(a[2]);
                if (PyErr_Occurred() || !address(a[0], device, mask, need, &p)) {
                    Py_DECREF(result);
                    PyErr_Clear();
                    Py_RETURN_NONE;
                }
                value = PyLong_FromVoidPtr(p);
                if (!value) {
                    Py_DECREF(result);
                    return nullptr;
                }
            } else {
                Py_INCREF(value);
            }
            PyTuple_SET_ITEM(result, i, value);
        }
    } catch (const std::exception &) {
        Py_DECREF(result);
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return result;
}

// address_array(device, tensors, mask, need): the addresses of a list or tuple
// of tensors as the bytes of a C array of pointers, or None.
PyObject *address_array(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "address_array(device, tensors, mask, need)");
        return nullptr;
    }
    if (!PyList_CheckExact(args[1]) && !PyTuple_CheckExact(args[1]))
        Py_RETURN_NONE;
    const long device = PyLong_AsLong(args[0]);
    const unsigned mask = (unsigned)PyLong_AsUnsignedLong(args[2]);
    const long long need = PyLong_AsLongLong(args[3]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const Py_ssize_t count = PySequence_Fast_GET_SIZE(args[1]);
    PyObject *const *items = PySequence_Fast_ITEMS(args[1]);
    try {
        std::vector<void *> p((size_t)count);
        for (Py_ssize_t i = 0; i < count; ++i)
            if (!address(items[i], device, mask, need, &p[(size_t)i]))
                Py_RETURN_NONE;
        return PyBytes_FromStringAndSize(reinterpret_cast<const char *>(p.data()),
                                         count * (Py_ssize_t)sizeof(void *));
    } catch (const std::exception &) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyMethodDef methods[] = {
    {"addresses", (PyCFunction)(void (*)(void))addresses, METH_FASTCALL,
     "addresses(device, tensor, mask, need, ...) -> tuple or None"},
    {"address_array", (PyCFunction)(void (*)(void))address_array, METH_FASTCALL,
     "address_array(device, tensors, mask, need) -> bytes or None"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    PyObject *m = PyModule_Create(&module);
    if (m && (PyModule_AddIntConstant(m, "F32", kF32) || PyModule_AddIntConstant(m, "BF16", kBF16) ||
              PyModule_AddIntConstant(m, "I16", kI16) || PyModule_AddIntConstant(m, "U16", kU16) ||
              PyModule_AddIntConstant(m, "I8", kI8) || PyModule_AddIntConstant(m, "U8", kU8) ||
              PyModule_AddIntConstant(m, "OPTIONAL", kOptional))) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
