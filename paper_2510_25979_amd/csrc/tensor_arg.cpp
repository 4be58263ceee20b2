// What the ctypes binding asks of every tensor argument, in one native call: is it a plain GPU tensor,
// contiguous, of the expected type and shape, and where does it start?  In Python these are six attribute look-ups and
// two tuples, 0.5 us a tensor (0.1 here).  attention_exact with five tensors takes 5.2 us of the host's time a call, 7.0 to
// 8.1 in Python; that is what small calls cost, and nothing where the kernel takes longer (64 x 12 heads of 64 x 64: 7.6 either way).
//
// Only the answer "yes" is given here.  Anything else -- a subclass, a tensor without storage, a wrong shape -- is None,
// and the Python code behind it decides and says what is wrong.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

bool has_shape(const at::Tensor& t, PyObject* shape) {
  if (!PyTuple_CheckExact(shape)) return false;
  const c10::IntArrayRef sizes = t.sizes();
  if (PyTuple_GET_SIZE(shape) != (Py_ssize_t)sizes.size()) return false;
  for (size_t i = 0; i < sizes.size(); ++i) {
    PyObject* n = PyTuple_GET_ITEM(shape, (Py_ssize_t)i);
    if (!PyLong_CheckExact(n)) return false;
    int overflow = 0;
    if (PyLong_AsLongLongAndOverflow(n, &overflow) != sizes[i] || overflow) return false;
  }
  return true;
}

// address(tensor, dtype or None, shape or None) -> int or None
PyObject* address(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) {
    PyErr_SetString(PyExc_TypeError, "address(tensor, dtype, shape)");
    return nullptr;
  }
  try {
    if (THPVariable_CheckExact(args[0])) {
      const at::Tensor& t = THPVariable_Unpack(args[0]);
      if (t.is_cuda() && t.is_contiguous() &&
          (args[1] == Py_None || (THPDtype_Check(args[1]) &&
                                  reinterpret_cast<THPDtype*>(args[1])->scalar_type == t.scalar_type())) &&
          (args[2] == Py_None || has_shape(t, args[2])))
        return PyLong_FromVoidPtr(t.data_ptr());
    }
  } catch (...) {   // (what Python raises for the same question, it raises itself)
  }
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"address", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(address)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tensor_arg", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tensor_arg() { return PyModule_Create(&module); }
