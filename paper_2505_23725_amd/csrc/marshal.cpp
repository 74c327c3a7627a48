// Addresses of tensors for the C entry points (binding.py).  A call of the library names up to a few hundred tensors,
// and reading type, device, layout and address of each from Python takes longer than the kernels of a small step:
// 3.4 us for the four tensors of an AdamW parameter.
//
// Only what is plainly in order is answered here: a torch.Tensor or Parameter, contiguous, on the current device (and, for
// adamw_groups, of a type that the library takes; who asks for a single address looks at the type itself).  For anything else the
// answer is None, and the caller's own checks say what is wrong with it (or, for a subclass, ask its own methods).  Nothing is
// kept from one call to the next.
#include <torch/csrc/python_headers.h>

#include <ATen/core/Tensor.h>
#include <c10/core/impl/DeviceGuardImplInterface.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <cstdint>
#include <cstring>

#include "muloco.h"

namespace {

// The tensor, where its address may be read without further questions.  `device` is the current one, asked for with the first
// tensor on a GPU (there may be none).
const at::Tensor* plain(PyObject* o, int& device) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !t.has_storage() || !t.is_contiguous()) return nullptr;
  if (device < 0) device = c10::impl::getDeviceGuardImpl(c10::kCUDA)->getDevice().index();
  return t.get_device() == device ? &t : nullptr;
}

int type_code(const at::Tensor& t) {
  return t.scalar_type() == at::kFloat ? MLC_F32 : t.scalar_type() == at::kBFloat16 ? MLC_BF16 : -1;
}

// pointer(tensor) -> address or None
PyObject* pointer(PyObject*, PyObject* arg) {
  HANDLE_TH_ERRORS
  int device = -1;
  const at::Tensor* t = plain(arg, device);
  if (!t) Py_RETURN_NONE;
  return PyLong_FromUnsignedLongLong((unsigned long long)(uintptr_t)t->data_ptr());
  END_HANDLE_TH_ERRORS
}

// adamw_groups([(param, grad, exp_avg, exp_avg_sq), ...]) -> their mlc_adamw_group entries as bytes, or None
PyObject* adamw_groups(PyObject*, PyObject* arg) {
  HANDLE_TH_ERRORS
  if (!PyList_CheckExact(arg)) Py_RETURN_NONE;
  const Py_ssize_t n = PyList_GET_SIZE(arg);
  int device = -1;
  PyObject* out = PyBytes_FromStringAndSize(nullptr, n * (Py_ssize_t)sizeof(mlc_adamw_group));
  if (!out) return nullptr;
  THPObjectPtr held(out);
  char* at = PyBytes_AS_STRING(out);
  for (Py_ssize_t i = 0; i < n; ++i, at += sizeof(mlc_adamw_group)) {
    PyObject* four = PyList_GET_ITEM(arg, i);
    if (!PyTuple_CheckExact(four) || PyTuple_GET_SIZE(four) != 4) Py_RETURN_NONE;
    const at::Tensor* t[4];
    for (int k = 0; k < 4; ++k) {
      t[k] = plain(PyTuple_GET_ITEM(four, k), device);
      if (!t[k] || t[k]->numel() != t[0]->numel()) Py_RETURN_NONE;
    }
    const int param = type_code(*t[0]), grad = type_code(*t[1]);
    if (param < 0 || grad < 0 || type_code(*t[2]) != MLC_F32 || type_code(*t[3]) != MLC_F32) Py_RETURN_NONE;
    mlc_adamw_group g;
    std::memset(&g, 0, sizeof g);
    g.count = t[0]->numel();
    g.param = t[0]->data_ptr();
    g.param_dtype = param;
    g.grad = t[1]->data_ptr();
    g.grad_dtype = grad;
    g.exp_avg = (float*)t[2]->data_ptr();
    g.exp_avg_sq = (float*)t[3]->data_ptr();
    std::memcpy(at, &g, sizeof g);
  }
  return held.release();
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"pointer", pointer, METH_O, nullptr},
    {"adamw_groups", adamw_groups, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  PyObject* m = PyModule_Create(&module);
  // the torch whose structures this was compiled for; the binding asks for the same
  if (m && PyModule_AddStringConstant(m, "torch_version", MLC_TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
