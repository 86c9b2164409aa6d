// Output tensors of a call, made in one step: most of the binding's own time was torch.empty from Python, 1.3 us
// each, and a call returns up to seven with its workspace.  Candidate lists with keys, 1024 rows of 50, us a call: 15.5 from
// Python, 13.3 with one tensor after the other made and wrapped, 11.0 with all made before any is wrapped.
// They are what torch.empty gives: separate tensors from torch's allocator, through its dispatcher, with its errors, and
// without Python's lock while they are allocated (the allocator may wait for the device, or for a thread that wants the lock).
// (The binding calls torch.empty itself under a mode that overrides torch's functions, which sees nothing of this.)
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/util/SmallVector.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>
#include <torch/csrc/utils/pybind.h>

namespace {

constexpr Py_ssize_t kMostDims = 4;

struct Spec {
  at::ScalarType type;
  Py_ssize_t dims;
  int64_t sizes[kMostDims];
};

// empties(device index, (dtype, size, ...), ...) -> tuple of uninitialised tensors
PyObject *empties(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  const long index = n_args > 0 ? PyLong_AsLong(args[0]) : -1;
  if (PyErr_Occurred()) return nullptr;
  TORCH_CHECK_VALUE(index >= 0 && index < 128, "empties: a device index, then (dtype, size, ...) tuples");
  const c10::Device device(c10::DeviceType::CUDA, (c10::DeviceIndex)index);
  c10::SmallVector<Spec, 8> specs;
  for (Py_ssize_t a = 1; a < n_args; ++a) {
    PyObject *spec = args[a];
    const Py_ssize_t dims = PyTuple_Check(spec) ? PyTuple_GET_SIZE(spec) - 1 : -1;
    TORCH_CHECK_TYPE(dims >= 0 && dims <= kMostDims && THPDtype_Check(PyTuple_GET_ITEM(spec, 0)),
                     "empties: a device index, then (dtype, size, ...) tuples");
    Spec s = {reinterpret_cast<THPDtype *>(PyTuple_GET_ITEM(spec, 0))->scalar_type, dims, {}};
    for (Py_ssize_t d = 0; d < dims; ++d) {
      s.sizes[d] = PyLong_AsLongLong(PyTuple_GET_ITEM(spec, d + 1));
      if (s.sizes[d] == -1 && PyErr_Occurred()) return nullptr;
    }
    specs.push_back(s);
  }
  c10::SmallVector<at::Tensor, 8> made;
  {
    pybind11::gil_scoped_release unlocked;
    for (const Spec &s : specs)
      made.push_back(at::empty(at::IntArrayRef(s.sizes, (size_t)s.dims), at::TensorOptions().dtype(s.type).device(device)));
  }
  THPObjectPtr out(PyTuple_New(n_args - 1));
  if (!out) return nullptr;
  for (Py_ssize_t a = 0; a + 1 < n_args; ++a) {
    PyObject *t = THPVariable_Wrap(std::move(made[(size_t)a]));
    if (t == nullptr) return nullptr;
    PyTuple_SET_ITEM(out.get(), a, t);
  }
  return out.release();
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"empties", (PyCFunction)(void (*)())empties, METH_FASTCALL, "uninitialised device tensors, one per (dtype, size, ...)"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_outputs", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__outputs() { return PyModule_Create(&module); }
