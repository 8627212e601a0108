// What a CPU test of the binding's native calls needs: tensors that say they are on a GPU while their memory is the host's, and an
// entry point that notes whether its caller holds the interpreter's lock.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/core/TensorImpl.h>

#include <vector>

namespace {

int calls = 0, locked = 0;

int noting_entry() {  // (called with any entry point's arguments, which it does not look at)
  calls++;
  locked += PyGILState_Check();
  return 0;
}

PyObject* entry(PyObject*, PyObject*) { return PyLong_FromVoidPtr(reinterpret_cast<void*>(noting_entry)); }

// ("f", "i" or "b", extents...): a dense tensor of floats, 32-bit integers or bytes
PyObject* tensor(PyObject*, PyObject* args) {
  const char kind = *PyUnicode_AsUTF8(PyTuple_GetItem(args, 0));
  const auto type = kind == 'f' ? c10::kFloat : kind == 'i' ? c10::kInt : c10::kByte;
  std::vector<int64_t> sizes;
  size_t bytes = kind == 'b' ? 1 : 4;
  for (Py_ssize_t i = 1; i < PyTuple_Size(args); i++) {
    sizes.push_back(PyLong_AsLongLong(PyTuple_GetItem(args, i)));
    bytes *= (size_t)sizes.back();
  }
  alignas(16) static char memory[1 << 16];
  if (bytes > sizeof memory) return PyErr_NoMemory();
  c10::Storage storage(c10::Storage::use_byte_size_t(), bytes, c10::DataPtr(memory, c10::Device(c10::kCUDA, 0)), nullptr, false);
  auto impl = c10::make_intrusive<c10::TensorImpl>(std::move(storage), c10::DispatchKeySet(c10::DispatchKey::CUDA), c10::scalarTypeToTypeMeta(type));
  impl->set_sizes_contiguous(sizes);
  return THPVariable_Wrap(at::Tensor(std::move(impl)));
}

PyObject* count(PyObject*, PyObject*) { return Py_BuildValue("(ii)", calls, locked); }

PyMethodDef methods[] = {{"entry", entry, METH_NOARGS, nullptr}, {"tensor", tensor, METH_VARARGS, nullptr}, {"count", count, METH_NOARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "fast_call_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_fast_call_host(void) { return PyModule_Create(&module); }
