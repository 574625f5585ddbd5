// Argument marshalling of Shampoo.step in native code: checks the parameter and gradient
// tensors of a step (device, dtype, contiguity, shape) and hands their addresses to
// shampoo_step on the current stream.  Ten attribute look-ups per tensor cost a millisecond in
// Python on a few hundred parameters, more than the step itself; here they cost some tens of
// nanoseconds per tensor.  What the tensor library throws (a tensor without storage, no device, no memory) leaves here
// as the Python exception that the same call raises from Python.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <pybind11/pybind11.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <cstdint>
#include <memory>
#include <vector>

namespace {

using StepFn = int (*)(void *, void *const *, const void *const *, float, int64_t, void *);

struct Stepper {
  StepFn fn;
  void *handle;
  c10::Device device{c10::DeviceType::CUDA, 0};
  at::ScalarType grad_dtype;
  std::vector<std::vector<int64_t>> shapes;
  std::vector<void *> w;
  std::vector<const void *> g;
};

constexpr const char *CAPSULE = "shampoo.stepper";

void stepper_free(PyObject *cap) { delete static_cast<Stepper *>(PyCapsule_GetPointer(cap, CAPSULE)); }

// make(address of shampoo_step, handle, device index, gradients are bf16, [shape tuples])
PyObject *make(PyObject *, PyObject *args) {
  HANDLE_TH_ERRORS
  unsigned long long fn, handle;
  int device, bf16;
  PyObject *shapes;
  if (!PyArg_ParseTuple(args, "KKipO!", &fn, &handle, &device, &bf16, &PyList_Type, &shapes)) return nullptr;
  auto s = std::make_unique<Stepper>();
  s->fn = reinterpret_cast<StepFn>(fn);
  s->handle = reinterpret_cast<void *>(handle);
  s->device = c10::Device(c10::DeviceType::CUDA, static_cast<c10::DeviceIndex>(device));
  s->grad_dtype = bf16 ? at::kBFloat16 : at::kFloat;
  for (Py_ssize_t i = 0; i < PyList_GET_SIZE(shapes); ++i) {
    PyObject *t = PyList_GET_ITEM(shapes, i);
    std::vector<int64_t> dims;
    for (Py_ssize_t k = 0; PyTuple_Check(t) && k < PyTuple_GET_SIZE(t); ++k) dims.push_back(PyLong_AsLongLong(PyTuple_GET_ITEM(t, k)));
    if (!PyTuple_Check(t) || PyErr_Occurred()) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "shapes are tuples of integers");
      return nullptr;
    }
    s->shapes.push_back(std::move(dims));
  }
  s->w.resize(s->shapes.size());
  s->g.resize(s->shapes.size());
  PyObject *cap = PyCapsule_New(s.get(), CAPSULE, stepper_free);
  if (cap) (void)s.release();
  return cap;
  END_HANDLE_TH_ERRORS
}

// step(stepper, params, grads, lr, step number) -> return code of shampoo_step
PyObject *step(PyObject *, PyObject *args) {
  HANDLE_TH_ERRORS
  PyObject *cap, *params, *grads;
  float lr;
  long long t;
  if (!PyArg_ParseTuple(args, "OOOfL", &cap, &params, &grads, &lr, &t)) return nullptr;
  auto *s = static_cast<Stepper *>(PyCapsule_GetPointer(cap, CAPSULE));
  if (!s) return nullptr;
  THPObjectPtr ps(PySequence_Fast(params, "params is a sequence of tensors"));
  if (!ps) return nullptr;
  THPObjectPtr gs(PySequence_Fast(grads, "grads is a sequence of tensors"));
  if (!gs) return nullptr;
  const Py_ssize_t n = static_cast<Py_ssize_t>(s->shapes.size());
  if (PySequence_Fast_GET_SIZE(ps.get()) != n || PySequence_Fast_GET_SIZE(gs.get()) != n) {
    PyErr_SetString(PyExc_ValueError, "one parameter and one gradient tensor per declared parameter");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject *po = PySequence_Fast_GET_ITEM(ps.get(), i), *go = PySequence_Fast_GET_ITEM(gs.get(), i);
    const char *bad = nullptr;
    if (!THPVariable_Check(po) || !THPVariable_Check(go)) {
      bad = "parameters and gradients are tensors";
    } else {
      const at::Tensor &w = THPVariable_Unpack(po), &g = THPVariable_Unpack(go);
      const c10::IntArrayRef shape(s->shapes[i]);
      if (w.device() != s->device || g.device() != s->device) bad = "tensors must live on the optimizer's device";
      else if (w.scalar_type() != at::kFloat || g.scalar_type() != s->grad_dtype)
        bad = s->grad_dtype == at::kFloat ? "parameters are float32, gradients torch.float32" : "parameters are float32, gradients torch.bfloat16";
      else if (!w.is_contiguous() || !g.is_contiguous()) bad = "tensors must be contiguous";
      else if (w.sizes() != shape || g.sizes() != shape) bad = "shape differs from the one given at creation";
      else { s->w[i] = w.data_ptr(); s->g[i] = g.data_ptr(); }
    }
    if (bad) { PyErr_Format(PyExc_ValueError, "parameter %zd: %s", i, bad); return nullptr; }
  }
  void *stream = c10::hip::getCurrentHIPStream().stream();
  int rc;
  {
    pybind11::gil_scoped_release no_gil;
    rc = s->fn(s->handle, s->w.data(), s->g.data(), lr, static_cast<int64_t>(t), stream);
  }
  return PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"make", make, METH_VARARGS, nullptr}, {"step", step, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
