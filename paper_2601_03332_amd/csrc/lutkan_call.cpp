// The forward calls of the binding as one native function each: what a program pays on the host for a call whose kernel runs 4 us.
// Through ctypes a call of one small layer took the host 5.7 - 6.6 us (checks 0.6 - 0.75, the output 1.1 - 1.4, ctypes 0.5, the launch 2.4);
// here 4.4, of which the kernel's own 4.0 are the limit: 10 -> 8 at 1024 rows 6.0 -> 5.2 us a call, 256 -> 256 at 16 rows 6.0 -> 5.3,
// 78 -> 16 -> 2 at 256 rows 7.2 -> 6.5.
//
// A function takes the layer object(s) and x, makes the checks of binding._check_io, allocates y (and the workspace, if the call
// needs one) with torch's allocator and calls the library on the current stream, both without the interpreter's lock, as torch's own
// functions and ctypes do: an allocation may wait for the device, and the device for a thread that needs the lock.
// It returns None, having done nothing, for anything but the plain case -- a strided CUDA tensor of torch's own class with no
// dispatch or function mode active, a layer of the binding's own struct -- and for whatever the library refuses: the binding then
// takes the general path, which serves it or says what is wrong.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <vector>

#include "lutkan.h"

namespace {

// Handed over by the binding (init): the library's entry points, the ctypes classes of the two layer structs, and torch's function
// that returns the handle of the current stream.
struct {
  decltype(&lutkan_forward_or_workspace) forward_or_workspace;
  decltype(&lutkan_forward) forward;
  decltype(&lutkan_model_forward_or_workspace) model_or_workspace;
  decltype(&lutkan_model_forward) model;
  decltype(&bspline_forward_workspace_bytes) spline_workspace_bytes;
  decltype(&bspline_kan_forward) spline;
  PyObject *lut_struct, *spline_struct, *current_stream;
} g;

PyObject *s_c, *s_d, *s_m, *s_device;      // attribute names of a layer object

// A layer object's fields.  `c` holds the ctypes struct's memory for as long as this lives.
struct Layer {
  Py_buffer c{};
  long d = 0, m = 0;
  c10::Device device{c10::kCPU};
  ~Layer() { if (c.obj) PyBuffer_Release(&c); }
  Layer() = default;
  Layer(const Layer &) = delete;
  Layer &operator=(const Layer &) = delete;

  bool read(PyObject *layer, PyObject *struct_type, size_t bytes) {
    PyObject *held = PyObject_GetAttr(layer, s_c);
    bool ok = held && (PyObject *)Py_TYPE(held) == struct_type && PyObject_GetBuffer(held, &c, PyBUF_SIMPLE) == 0 && (size_t)c.len == bytes;
    Py_XDECREF(held);
    ok = ok && number(layer, s_d, &d) && number(layer, s_m, &m);
    if (!ok) return false;
    PyObject *dev = PyObject_GetAttr(layer, s_device);
    ok = dev && THPDevice_Check(dev);
    if (ok) device = reinterpret_cast<THPDevice *>(dev)->device;
    Py_XDECREF(dev);
    return ok;
  }

 private:
  static bool number(PyObject *layer, PyObject *name, long *out) {
    PyObject *v = PyObject_GetAttr(layer, name);
    const bool ok = v && PyLong_CheckExact(v);
    if (ok) *out = PyLong_AsLong(v);
    Py_XDECREF(v);
    return ok && !(*out == -1 && PyErr_Occurred());
  }
};

// x as the kernels take it: [B][d] contiguous fp32 on the layer's GPU, and nothing that would intercept or defer an operator on it.
const at::Tensor *plain_input(PyObject *x, long d, c10::Device device) {
  if (!THPVariable_CheckExact(x)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(x);
  const c10::DispatchKeySet plain({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA});
  if (!t.defined() || (t.key_set().raw_repr() & ~plain.raw_repr()) != 0 || t.layout() != c10::kStrided || t.scalar_type() != at::kFloat) return nullptr;
  if (t.device() != device || !device.is_cuda() || !device.has_index() || t.dim() != 2 || t.size(1) != d || !t.is_contiguous()) return nullptr;
  if (c10::impl::dispatch_mode_enabled() || at::impl::torch_function_mode_enabled()) return nullptr;
  if (c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Tracer) || c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Functionalize) ||
      c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode))
    return nullptr;
  return &t;
}

bool stream_of(c10::Device device, void **out) {
  PyObject *index = PyLong_FromLong(device.index());
  PyObject *handle = index ? PyObject_CallOneArg(g.current_stream, index) : nullptr;
  Py_XDECREF(index);
  if (!handle) return false;
  *out = PyLong_AsVoidPtr(handle);
  Py_DECREF(handle);
  return !PyErr_Occurred();
}

at::Tensor workspace_of(size_t bytes, c10::Device device) {
  return at::empty({(int64_t)std::max<size_t>(bytes, 256)}, at::TensorOptions().dtype(at::kByte).device(device));
}

PyObject *not_taken() {
  PyErr_Clear();
  Py_RETURN_NONE;
}

struct WithoutLock {
  PyThreadState *state = PyEval_SaveThread();
  ~WithoutLock() { PyEval_RestoreThread(state); }
};

// once(needed): the call that runs without a workspace or says how much one takes; again(workspace, bytes): the call with one.
template <typename Once, typename Again>
PyObject *forward(const at::Tensor &x, long m, c10::Device device, const Once &once, const Again &again) {
  try {
    void *stream = nullptr;
    if (!stream_of(device, &stream)) return not_taken();
    at::Tensor y;
    int rc;
    {
      const WithoutLock unlocked;
      y = at::empty({x.size(0), m}, x.options().requires_grad(false));
      const float *in = x.const_data_ptr<float>();
      float *out = y.mutable_data_ptr<float>();
      const int64_t B = x.size(0);
      size_t needed = 0;
      rc = once(in, B, out, &needed, stream);
      if (rc == LUTKAN_OK && needed != 0) {
        const at::Tensor workspace = workspace_of(needed, device);
        rc = again(in, B, out, workspace.mutable_data_ptr(), (size_t)workspace.numel(), stream);
      }
    }
    if (rc != LUTKAN_OK) return not_taken();
    return THPVariable_Wrap(y);
  } catch (...) {                                          // no exception crosses into the interpreter: the general path reports it
    return not_taken();
  }
}

PyObject *lut_forward(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Layer layer;
  if (n != 2 || !layer.read(args[0], g.lut_struct, sizeof(lutkan_dev_layer))) return not_taken();
  const at::Tensor *x = plain_input(args[1], layer.d, layer.device);
  if (!x) return not_taken();
  const auto *l = static_cast<const lutkan_dev_layer *>(layer.c.buf);
  return forward(*x, layer.m, layer.device,
                 [&](const float *in, int64_t B, float *out, size_t *needed, void *stream) { return g.forward_or_workspace(l, in, B, out, nullptr, needed, stream); },
                 [&](const float *in, int64_t B, float *out, void *ws, size_t bytes, void *stream) { return g.forward(l, in, B, out, nullptr, ws, bytes, stream); });
}

PyObject *lut_model_forward(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 2 || !(PyList_CheckExact(args[0]) || PyTuple_CheckExact(args[0]))) return not_taken();
  const Py_ssize_t count = PySequence_Fast_GET_SIZE(args[0]);
  if (count < 1 || count > LUTKAN_MAX_LAYERS) return not_taken();
  lutkan_dev_layer layers[LUTKAN_MAX_LAYERS];
  long d = 0, m = 0;
  c10::Device device(c10::kCPU);
  for (Py_ssize_t i = 0; i < count; ++i) {
    if (i >= PySequence_Fast_GET_SIZE(args[0])) return not_taken();                  // reading an attribute may run code that changes the list
    PyObject *const item = PySequence_Fast_GET_ITEM(args[0], i);
    Py_INCREF(item);
    Layer layer;
    const bool ok = layer.read(item, g.lut_struct, sizeof(lutkan_dev_layer));
    Py_DECREF(item);
    if (!ok) return not_taken();
    if (i == 0) { d = layer.d; device = layer.device; }
    if (layer.device != device) return not_taken();
    m = layer.m;
    std::memcpy(&layers[i], layer.c.buf, sizeof(lutkan_dev_layer));
  }
  const at::Tensor *x = plain_input(args[1], d, device);
  if (!x) return not_taken();
  const int32_t n_layers = (int32_t)count;
  return forward(*x, m, device,
                 [&](const float *in, int64_t B, float *out, size_t *needed, void *stream) { return g.model_or_workspace(layers, n_layers, in, B, out, nullptr, needed, stream); },
                 [&](const float *in, int64_t B, float *out, void *ws, size_t bytes, void *stream) { return g.model(layers, n_layers, in, B, out, nullptr, ws, bytes, stream); });
}

PyObject *spline_forward(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Layer layer;
  if (n != 2 || !layer.read(args[0], g.spline_struct, sizeof(bspline_dev_layer))) return not_taken();
  const at::Tensor *x = plain_input(args[1], layer.d, layer.device);
  if (!x) return not_taken();
  const auto *l = static_cast<const bspline_dev_layer *>(layer.c.buf);
  return forward(*x, layer.m, layer.device,
                 [&](const float *, int64_t B, float *, size_t *needed, void *) { *needed = std::max<size_t>(g.spline_workspace_bytes(l, B), 256); return LUTKAN_OK; },
                 [&](const float *in, int64_t B, float *out, void *ws, size_t bytes, void *stream) { return g.spline(l, in, B, out, ws, bytes, stream); });
}

// init(addresses of the six entry points, the two struct classes, the stream function)
PyObject *init(PyObject *, PyObject *args) {
  unsigned long long p[6];
  PyObject *lut_struct, *spline_struct, *current_stream;
  if (!PyArg_ParseTuple(args, "KKKKKKOOO", &p[0], &p[1], &p[2], &p[3], &p[4], &p[5], &lut_struct, &spline_struct, &current_stream)) return nullptr;
  g.forward_or_workspace = reinterpret_cast<decltype(g.forward_or_workspace)>(p[0]);
  g.forward = reinterpret_cast<decltype(g.forward)>(p[1]);
  g.model_or_workspace = reinterpret_cast<decltype(g.model_or_workspace)>(p[2]);
  g.model = reinterpret_cast<decltype(g.model)>(p[3]);
  g.spline_workspace_bytes = reinterpret_cast<decltype(g.spline_workspace_bytes)>(p[4]);
  g.spline = reinterpret_cast<decltype(g.spline)>(p[5]);
  Py_INCREF(lut_struct); Py_INCREF(spline_struct); Py_INCREF(current_stream);
  g.lut_struct = lut_struct; g.spline_struct = spline_struct; g.current_stream = current_stream;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"init", init, METH_VARARGS, nullptr},
                         {"lut_forward", (PyCFunction)(void (*)())lut_forward, METH_FASTCALL, nullptr},
                         {"lut_model_forward", (PyCFunction)(void (*)())lut_model_forward, METH_FASTCALL, nullptr},
                         {"spline_forward", (PyCFunction)(void (*)())spline_forward, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lutkan_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lutkan_call() {
  s_c = PyUnicode_InternFromString("c");
  s_d = PyUnicode_InternFromString("d");
  s_m = PyUnicode_InternFromString("m");
  s_device = PyUnicode_InternFromString("device");
  return (s_c && s_d && s_m && s_device) ? PyModule_Create(&module) : nullptr;
}
