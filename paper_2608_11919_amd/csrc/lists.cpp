// lists.cpp -- the binding's tensor lists in native code.
//
// A step over a few hundred small tensors spent its time on the host: reading device,
// dtype, contiguity, size and address of six lists of 288 adapter tensors in Python took
// about 0.5 ms a step, against some 60 us of kernels.  take() does the reading for one
// list: 3.7 us for 288 tensors, 202 in Python (the whole step of 288 adapter tensors
// 570 -> 59 us, of four tensors 43 -> 30 us).
//
// It only ever says "this list is in order, here are its addresses and sizes"; for
// anything else (another device or dtype, a strided tensor, a tensor subclass, a torch
// function mode, an object that is no tensor) it returns None, and the binding's own
// checks run and raise.  Nothing is kept between calls.

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <exception>

namespace {

// take(tensors, device, dtype) -> (addresses, sizes, type) or None.
//   tensors  list or tuple of tensors, all contiguous and on `device`
//   dtype    the dtype they must have, or None: any one dtype, the same for all
// addresses and sizes are bytes objects of one 64-bit word per tensor; type is the
// tensors' torch.dtype (None for an empty list).
PyObject* take(PyObject*, PyObject* const* args, Py_ssize_t n_args)
{
    if (n_args != 3) {
        PyErr_SetString(PyExc_TypeError, "take(tensors, device, dtype)");
        return nullptr;
    }
    PyObject* list = args[0];
    const bool is_list = PyList_CheckExact(list);
    if (!(is_list || PyTuple_CheckExact(list)) || !THPDevice_Check(args[1]) ||
        !(args[2] == Py_None || THPDtype_Check(args[2])) ||
        at::impl::torch_function_mode_enabled())
        Py_RETURN_NONE;
    const Py_ssize_t n = is_list ? PyList_GET_SIZE(list) : PyTuple_GET_SIZE(list);
    const c10::Device device = reinterpret_cast<THPDevice*>(args[1])->device;

    PyObject* ptrs = PyBytes_FromStringAndSize(nullptr, 8 * n);
    PyObject* sizes = ptrs ? PyBytes_FromStringAndSize(nullptr, 8 * n) : nullptr;
    if (!sizes) {
        Py_XDECREF(ptrs);
        return nullptr;
    }
    bool in_order = true;
    PyObject* type = Py_None;
    try {
        c10::ScalarType want = c10::ScalarType::Undefined;
        if (args[2] != Py_None)
            want = reinterpret_cast<THPDtype*>(args[2])->scalar_type;
        char* p = PyBytes_AS_STRING(ptrs);
        char* s = PyBytes_AS_STRING(sizes);
        for (Py_ssize_t i = 0; i < n && in_order; ++i) {
            PyObject* o = is_list ? PyList_GET_ITEM(list, i) : PyTuple_GET_ITEM(list, i);
            if (!THPVariable_CheckExact(o)) {
                in_order = false;
                break;
            }
            const at::Tensor& t = THPVariable_Unpack(o);
            if (i == 0 && args[2] == Py_None)
                want = t.scalar_type();
            if (t.device() != device || t.scalar_type() != want || !t.is_contiguous()) {
                in_order = false;
                break;
            }
            const int64_t numel = t.numel();
            const uint64_t at = reinterpret_cast<uint64_t>(t.data_ptr());
            std::memcpy(p + 8 * i, &at, 8);
            std::memcpy(s + 8 * i, &numel, 8);
        }
        if (in_order && n > 0)
            type = reinterpret_cast<PyObject*>(torch::getTHPDtype(want));
    } catch (const std::exception&) {
        in_order = false;  // a tensor without storage, say: the binding's checks report it
    }
    PyObject* out = nullptr;
    if (in_order) {
        out = PyTuple_Pack(3, ptrs, sizes, type);
    } else {
        PyErr_Clear();
        out = Py_None;
        Py_INCREF(out);
    }
    Py_DECREF(ptrs);
    Py_DECREF(sizes);
    return out;
}

// covers(sizes, have, block): every have[i] >= ceil(sizes[i] / block) (block >= 1).
PyObject* covers(PyObject*, PyObject* const* args, Py_ssize_t n_args)
{
    if (n_args != 3 || !PyBytes_CheckExact(args[0]) || !PyBytes_CheckExact(args[1])) {
        PyErr_SetString(PyExc_TypeError, "covers(sizes, have, block)");
        return nullptr;
    }
    const int64_t block = PyLong_AsLongLong(args[2]);
    if (block == -1 && PyErr_Occurred())
        return nullptr;
    const Py_ssize_t bytes = PyBytes_GET_SIZE(args[0]);
    if (block < 1 || bytes % 8 != 0 || PyBytes_GET_SIZE(args[1]) != bytes)
        Py_RETURN_FALSE;
    for (Py_ssize_t i = 0; i < bytes; i += 8) {
        int64_t n, have;
        std::memcpy(&n, PyBytes_AS_STRING(args[0]) + i, 8);
        std::memcpy(&have, PyBytes_AS_STRING(args[1]) + i, 8);
        if (have < n / block + (n % block != 0))
            Py_RETURN_FALSE;
    }
    Py_RETURN_TRUE;
}

PyMethodDef methods[] = {
    {"take", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(take)), METH_FASTCALL,
     "Addresses, sizes and dtype of a list of contiguous tensors on one device, or None."},
    {"covers", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(covers)), METH_FASTCALL,
     "Whether every have[i] holds ceil(sizes[i] / block) entries."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lists", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lists() { return PyModule_Create(&module); }
