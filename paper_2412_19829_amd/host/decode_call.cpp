// The host side of one decode step, for binding.gformer_attn_decode: a step of a few users takes 4 to 5 us on the
// device, and checking and marshalling its seven tensors in Python took 8 (1 x 12 heads, d = 64: 8.2 us a step among
// others, 4.3 with this, which is the kernel).
//
// decode(address, q, k, v, out, kcache, vcache, state, window, n_sparse_heads, t, phi, softmax_scale, eps, stream)
// returns the gf_status of the call at `address` (gformer_attn_decode), or None for anything that is not the plain,
// well-formed call: wrapped or traced tensors, shapes or types that do not fit, numbers out of range.  The
// binding's own code then does or refuses the call, with its own messages.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/core/DispatchKeySet.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstring>

#include "../../include/gformer.h"

namespace {

using Decode = decltype(&gformer_attn_decode);

// A dense tensor and nothing else: a wrapper's data pointer is not what the caller means.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.layout() != at::kStrided || t.is_nested() || !t.has_storage() ||
      t.unsafeGetTensorImpl()->has_symbolic_sizes_strides() || !t.is_contiguous())
    return nullptr;
  constexpr c10::DispatchKeySet wrapped({
      c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::Functionalize,
      c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Conjugate,
      c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
  return t.key_set().has_any(wrapped) ? nullptr : &t;
}

bool to_long(PyObject* o, int64_t lo, int64_t hi, int64_t& x) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  x = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0 && x >= lo && x <= hi;
}
bool to_float(PyObject* o, float& x) {
  if (!PyFloat_CheckExact(o)) return false;
  x = (float)PyFloat_AS_DOUBLE(o);
  return true;
}

PyObject* raw_stream_getter = nullptr;   // torch._C._cuda_getCurrentRawStream, where torch has it

// What the call takes from its arguments; the stream only where it was named.
struct Step {
  gformer_params p;
  void* at[7];   // q, k, v, out, kcache, vcache, state
  int64_t B, H, d, window, t, device, stream;
};

// False for anything but the plain call.  Asking a tensor may throw.
bool gather(PyObject* const* a, Step& s) {
  const at::Tensor* x[7];
  for (int i = 0; i < 7; ++i) {
    x[i] = nullptr;
    if (i >= 4 && a[1 + i] == Py_None) continue;
    if (!(x[i] = plain(a[1 + i]))) return false;
  }
  int64_t h0, phi;
  std::memset(&s, 0, sizeof(s));
  if (!to_long(a[8], INT_MIN, INT_MAX, s.window) || !to_long(a[9], 0, INT_MAX, h0) || !to_long(a[10], LLONG_MIN, LLONG_MAX, s.t) ||
      !to_long(a[11], INT_MIN, INT_MAX, phi) || !to_float(a[12], s.p.softmax_scale) || !to_float(a[13], s.p.eps) ||
      (a[14] != Py_None && !to_long(a[14], 0, LLONG_MAX, s.stream)))
    return false;
  const at::Tensor& q = *x[0];
  const auto type = q.scalar_type();
  if ((type != at::kBFloat16 && type != at::kFloat) || q.dim() != 3) return false;
  for (int i = 1; i < 4; ++i)
    if (x[i]->scalar_type() != type || x[i]->sizes() != q.sizes()) return false;
  s.B = q.size(0);
  s.H = q.size(1);
  s.d = q.size(2);
  if (s.B > INT_MAX || s.H > INT_MAX || s.d > INT_MAX || h0 > s.H) return false;
  if (h0 > 0) {
    const int64_t ring[4] = {s.B, h0, s.window, s.d};
    for (int i = 4; i < 6; ++i)
      if (!x[i] || x[i]->scalar_type() != type || x[i]->sizes() != at::IntArrayRef(ring, 4)) return false;
  }
  if (h0 < s.H) {
    const int64_t sums[3] = {s.B, s.H - h0, s.d * s.d + s.d};
    if (!x[6] || x[6]->scalar_type() != at::kFloat || x[6]->sizes() != at::IntArrayRef(sums, 3)) return false;
  }
  // the device is asked last, so that host tensors go through all of the above, which a process without a device can run
  s.device = q.get_device();
  for (int i = 0; i < 7; ++i)
    if (x[i] && (!x[i]->is_cuda() || x[i]->get_device() != s.device)) return false;
  for (int i = 0; i < 7; ++i) s.at[i] = x[i] ? x[i]->data_ptr() : nullptr;
  s.p.struct_size = sizeof(s.p);
  s.p.dtype = type == at::kBFloat16 ? GF_BF16 : GF_F32;
  s.p.phi = (int32_t)phi;
  s.p.n_sparse_heads = (int32_t)h0;
  return true;
}

PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 15) {
    PyErr_SetString(PyExc_TypeError, "decode takes 15 arguments");
    return nullptr;
  }
  Step s;
  try {   // no C++ exception may leave a function that the interpreter called
    if (!gather(a, s)) Py_RETURN_NONE;
  } catch (...) {
    Py_RETURN_NONE;   // the binding's code raises it, or says what is missing
  }
  if (a[14] == Py_None) {
    if (!raw_stream_getter) Py_RETURN_NONE;   // the binding knows another way
    PyObject* index = PyLong_FromLong((long)s.device);
    PyObject* handle = index ? PyObject_CallOneArg(raw_stream_getter, index) : nullptr;
    Py_XDECREF(index);
    if (!handle) return nullptr;
    s.stream = (int64_t)PyLong_AsUnsignedLongLongMask(handle);
    Py_DECREF(handle);
  }
  const Decode call = reinterpret_cast<Decode>(PyLong_AsVoidPtr(a[0]));
  if (!call) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no function address");
    return nullptr;
  }
  gf_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call(s.at[0], s.at[1], s.at[2], s.at[3], s.at[4], s.at[5], static_cast<float*>(s.at[6]), (int)s.B, (int)s.H,
            (int)s.d, (int)s.window, s.t, &s.p, reinterpret_cast<void*>(s.stream));
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)st);
}

PyMethodDef methods[] = {
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(decode)), METH_FASTCALL, "one decode step"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_decode_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__decode_call() {
  PyObject* torch_c = PyImport_ImportModule("torch._C");
  if (!torch_c) return nullptr;
  raw_stream_getter = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
  Py_DECREF(torch_c);
  if (!raw_stream_getter) PyErr_Clear();
  return PyModule_Create(&module);
}
