// Python extension: muon_adamw_step for a list of (p, g, m, v) torch tensors without a Python call per tensor and attribute.
// A list of small tensors is bound by that marshalling: a step of 25 gains of 1024 elements took 33.9 us in Python, 4 of them
// on the device, and takes 8.6 like this.  It takes the ordinary case only - plain contiguous tensors of the types the step knows - and answers None
// to everything else, which the binding then handles (and refuses, where it has to) in Python.
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/PyInterpreter.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "../../include/muon.h"

namespace {

// float32, bfloat16: the library's codes; -1: anything else
int dtype_code(const at::Tensor& t) {
  const auto s = t.scalar_type();
  return s == at::kFloat ? (int)MUON_F32 : s == at::kBFloat16 ? (int)MUON_BF16 : -1;
}

// One record from a (p, g, m, v) tuple; false: not the ordinary case.  May throw what the tensors' methods throw.
bool record_of(PyObject* quad, muon_adamw_param* out) {
  if (!PyTuple_CheckExact(quad) || PyTuple_GET_SIZE(quad) != 4) return false;
  const at::Tensor* t[4];
  for (int i = 0; i < 4; ++i) {
    PyObject* o = PyTuple_GET_ITEM(quad, i);
    if (!THPVariable_CheckExact(o)) return false;          // subclasses see the calls of the Python path
    t[i] = &THPVariable_Unpack(o);
    if (!t[i]->is_contiguous() || t[i]->numel() != t[0]->numel()) return false;
  }
  const int pc = dtype_code(*t[0]), gc = dtype_code(*t[1]);
  if (pc < 0 || gc < 0 || dtype_code(*t[2]) != MUON_F32 || dtype_code(*t[3]) != MUON_F32) return false;
  *out = muon_adamw_param{t[0]->data_ptr(), t[1]->data_ptr(), static_cast<float*>(t[2]->data_ptr()),
                          static_cast<float*>(t[3]->data_ptr()), t[0]->numel(), pc, gc};
  return true;
}

PyObject* g_device_context = nullptr;            // torch.utils._device.DeviceContext, for as long as the process runs

// Function modes see every call of the Python path, so a mode leaves the work to that, with one exception: the mode behind
// torch.set_default_device and `with torch.device(..)` changes calls that make tensors and hands every other one through.
bool modes_see_calls() {
  using at::impl::PythonTorchFunctionTLS;
  if (!at::impl::torch_function_mode_enabled()) return false;
  for (int64_t i = 0, n = PythonTorchFunctionTLS::stack_len(); i < n; ++i)
    if ((PyObject*)Py_TYPE(PythonTorchFunctionTLS::get_stack_at(i)->ptr(getPyInterpreter())) != g_device_context) return true;
  return false;
}

// step(list of tuples, address of a muon_adamw_hparams, stream) -> status of muon_adamw_step, or None
PyObject* step(PyObject*, PyObject* args) {
  PyObject* list = nullptr;
  unsigned long long hp = 0, stream = 0;
  if (!PyArg_ParseTuple(args, "O!KK", &PyList_Type, &list, &hp, &stream)) return nullptr;
  try {
    if (modes_see_calls()) Py_RETURN_NONE;
    const Py_ssize_t n = PyList_GET_SIZE(list);
    std::vector<muon_adamw_param> records((size_t)n);
    for (Py_ssize_t i = 0; i < n; ++i)
      if (!record_of(PyList_GET_ITEM(list, i), &records[(size_t)i])) Py_RETURN_NONE;
    if (n > INT32_MAX) Py_RETURN_NONE;
    int status = 0;
    Py_BEGIN_ALLOW_THREADS                       // the caller's list keeps the tensors alive
    status = muon_adamw_step(records.data(), (int32_t)n, reinterpret_cast<const muon_adamw_hparams*>((uintptr_t)hp),
                             reinterpret_cast<void*>((uintptr_t)stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
  } catch (...) {                                // a tensor without storage, say: the Python path raises it
    Py_RETURN_NONE;
  }
}

PyMethodDef methods[] = {{"step", step, METH_VARARGS, "muon_adamw_step on a list of (p, g, m, v) tuples of plain tensors"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_adamw_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// Reading a tensor is inlined code for one layout, so the module says which torch it was compiled for and how large the
// library's records were; the binding does not use it with another.
PyMODINIT_FUNC PyInit__adamw_marshal() {
  PyObject* m = PyModule_Create(&module);
  if (!m) return nullptr;
  if (PyObject* device = PyImport_ImportModule("torch.utils._device")) {
    g_device_context = PyObject_GetAttrString(device, "DeviceContext");
    Py_DECREF(device);
  }
  PyErr_Clear();                                 // (without it, modes of any kind go to Python)
  PyObject* sizes = Py_BuildValue("(nn)", (Py_ssize_t)sizeof(muon_adamw_param), (Py_ssize_t)sizeof(muon_adamw_hparams));
  if (!sizes || PyModule_AddStringConstant(m, "built_for", MUON_BUILT_FOR) < 0 || PyModule_AddObject(m, "record_sizes", sizes) < 0) {
    Py_XDECREF(sizes);
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
