// Python extension of the binding: the checks of a call's tensors and their
// addresses, without a Python call per tensor (a serving rank has hundreds of
// local tensors, and the checks run on every call). It answers only for plain
// torch tensors that pass every check; for anything else it says no and the
// binding's own Python checks decide, with their messages.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

// One local tensor of a plan: its element count and the library's dtype code.
struct Expect {
  int64_t numel;
  int64_t dtype;
};

bool holds(at::ScalarType t, int64_t code) {
  switch (code) {
    case 0: return t == at::kFloat || t == at::kInt || t == at::kUInt32;
    case 1: return t == at::kBFloat16 || t == at::kShort || t == at::kUInt16;
    case 2: return t == at::kFloat8_e4m3fn || t == at::kByte || t == at::kChar;
    default: return false;
  }
}

// The tensor behind an object of exactly torch.Tensor or torch.nn.Parameter
// in GPU memory and contiguous; null otherwise.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() ? &t : nullptr;
}

// pointers(sequence, expect, out): the tensors' addresses into the array of
// 8-byte words at address out, if every one is as expected (bytes of Expect
// records); False (the array then holds nothing of use) otherwise.
PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 3 || !PyBytes_CheckExact(args[1])) {
    PyErr_SetString(PyExc_TypeError, "pointers(sequence, bytes, address)");
    return nullptr;
  }
  uint64_t* out = static_cast<uint64_t*>(PyLong_AsVoidPtr(args[2]));
  if (PyErr_Occurred()) return nullptr;
  if (!PyList_CheckExact(args[0]) && !PyTuple_CheckExact(args[0])) Py_RETURN_FALSE;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(args[0]);
  const auto* want = reinterpret_cast<const Expect*>(PyBytes_AS_STRING(args[1]));
  if (PyBytes_GET_SIZE(args[1]) != n * Py_ssize_t(sizeof(Expect))) Py_RETURN_FALSE;
  PyObject** items = PySequence_Fast_ITEMS(args[0]);
  try {
    for (Py_ssize_t i = 0; i < n; ++i) {
      const at::Tensor* t = plain(items[i]);
      if (!t || t->numel() != want[i].numel || !holds(t->scalar_type(), want[i].dtype)) Py_RETURN_FALSE;
      out[i] = reinterpret_cast<uint64_t>(t->data_ptr());
    }
  } catch (const std::exception&) {
    Py_RETURN_FALSE;
  }
  Py_RETURN_TRUE;
}

// address(tensor, nbytes): the address of a plain tensor of at least nbytes
// bytes; None otherwise.
PyObject* address(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 2) {
    PyErr_SetString(PyExc_TypeError, "address(tensor, nbytes)");
    return nullptr;
  }
  const long long nbytes = PyLong_AsLongLong(args[1]);
  if (nbytes == -1 && PyErr_Occurred()) return nullptr;
  try {
    const at::Tensor* t = plain(args[0]);
    if (!t || t->numel() * int64_t(t->element_size()) < nbytes) Py_RETURN_NONE;
    return PyLong_FromVoidPtr(t->data_ptr());
  } catch (const std::exception&) {
    Py_RETURN_NONE;
  }
}

PyMethodDef methods[] = {
    {"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(pointers)), METH_FASTCALL, nullptr},
    {"address", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(address)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_args", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__args() { return PyModule_Create(&module); }
