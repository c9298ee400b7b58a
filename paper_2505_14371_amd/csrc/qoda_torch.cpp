// The torch-facing loop's look at its K x L gradients, in native code: every tensor is looked at in every round, and in a small model
// that was most of the host's time (four lists of 17 tensors: 20 us in Python, under 2 here).  A module of the interpreter, not part of
// libqoda's C ABI.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

// A plain tensor or parameter; anything else (a subclass may answer for itself) is left to the caller's own look.
const at::Tensor *plain_tensor(PyObject *o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

// gather(node_grads, params, nodes, out): whether node_grads is a list or tuple of `nodes` lists or tuples of contiguous fp32 CUDA tensors with the
// parameters' numbers of elements; if so, their addresses are stored at out, node by node.  False also where that cannot be told here.
PyObject *gather(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
  if (nargs != 4) {
    PyErr_SetString(PyExc_TypeError, "gather(node_grads, params, nodes, out)");
    return nullptr;
  }
  PyObject *lists = args[0], *params = args[1];
  const Py_ssize_t nodes = PyLong_AsSsize_t(args[2]);
  uint64_t *out = static_cast<uint64_t *>(PyLong_AsVoidPtr(args[3]));
  if (PyErr_Occurred()) return nullptr;
  const auto plain = [](PyObject *o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); };
  if (!plain(lists) || !plain(params) || PySequence_Fast_GET_SIZE(lists) != nodes) Py_RETURN_FALSE;
  const Py_ssize_t L = PySequence_Fast_GET_SIZE(params);
  try {
    for (Py_ssize_t k = 0; k < nodes; ++k) {
      PyObject *g = PySequence_Fast_GET_ITEM(lists, k);
      if (!plain(g) || PySequence_Fast_GET_SIZE(g) != L) Py_RETURN_FALSE;
      for (Py_ssize_t l = 0; l < L; ++l) {
        const at::Tensor *t = plain_tensor(PySequence_Fast_GET_ITEM(g, l)), *p = plain_tensor(PySequence_Fast_GET_ITEM(params, l));
        if (!t || !p || !t->is_cuda() || t->scalar_type() != at::kFloat || !t->is_contiguous() || t->numel() != p->numel()) Py_RETURN_FALSE;
        out[k * L + l] = reinterpret_cast<uint64_t>(t->data_ptr());
      }
    }
  } catch (...) {   // a tensor without memory of its own, say: the caller's look reports it
    Py_RETURN_FALSE;
  }
  Py_RETURN_TRUE;
}

PyMethodDef methods[] = {{"gather", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gather)), METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qoda_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__qoda_torch() {
  PyObject *m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "built_for", QODA_BUILT_FOR) != 0) {   // the caller compares it with what is running
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
