// The binding's tensor checks: address(t, device, dtype, shape) is t's data
// address when t is a contiguous tensor on `device`, of `dtype` (None: any) and
// of `shape` (None: any), 0 when it is all that and empty, and -1 otherwise
// (the caller then finds out what is wrong and says so).  A layer call checks
// eight tensors: about 1 us each as Python attribute reads, 0.1 us here.
// built_for is the torch it was compiled against (its C++ objects' layout): the
// binding uses the module with that torch only.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

PyObject* address(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 4) {
    PyErr_SetString(PyExc_TypeError, "address(tensor, device, dtype, shape)");
    return nullptr;
  }
  PyObject *to = args[0], *dev = args[1], *dt = args[2], *shape = args[3];
  if (!THPVariable_Check(to) || !THPDevice_Check(dev)) return PyLong_FromLong(-1);
  try {
    const at::Tensor& t = THPVariable_Unpack(to);
    if (t.layout() != c10::kStrided || t.device() != reinterpret_cast<THPDevice*>(dev)->device)
      return PyLong_FromLong(-1);
    if (dt != Py_None &&
        (!THPDtype_Check(dt) || t.scalar_type() != reinterpret_cast<THPDtype*>(dt)->scalar_type))
      return PyLong_FromLong(-1);
    if (shape != Py_None) {
      if (!PyTuple_Check(shape) || PyTuple_GET_SIZE(shape) != t.dim()) return PyLong_FromLong(-1);
      for (Py_ssize_t i = 0; i < t.dim(); ++i) {
        const long long v = PyLong_AsLongLong(PyTuple_GET_ITEM(shape, i));
        if (v == -1 && PyErr_Occurred()) return nullptr;
        if (t.size(i) != v) return PyLong_FromLong(-1);
      }
    }
    if (!t.is_contiguous()) return PyLong_FromLong(-1);
    if (t.numel() == 0) return PyLong_FromLong(0);
    return PyLong_FromUnsignedLongLong(reinterpret_cast<uintptr_t>(t.data_ptr()));
  } catch (const std::exception&) {      // a tensor without storage, or one that only stands for another
    PyErr_Clear();                       // (a Python error of its own comes again with the caller's checks)
    return PyLong_FromLong(-1);
  }
}

PyMethodDef methods[] = {
    {"address", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(address)), METH_FASTCALL,
     "address(tensor, device, dtype or None, shape or None)"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "built_for", CTS_TORCH_VERSION) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
