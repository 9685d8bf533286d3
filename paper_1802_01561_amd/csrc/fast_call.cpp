// Argument marshalling of the ordinary call, without Python objects per argument:
// plain contiguous device tensors of the expected types and shapes, preallocated
// outputs, a workspace and the current stream.  Each function checks exactly that
// and calls the C entry point it is given (include/vtrace.h); on anything else it
// returns None, having done nothing, and binding.py's own path, which allocates
// and reports errors, takes the call.
//
// In Python the checks and conversions of a loss call take about 9 us, more than
// the kernel of a 32-lane batch.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include <initializer_list>

#include "vtrace.h"

namespace {

using at::ScalarType;

// An ordinary dense device tensor: no subclass, no functional transform, nothing
// that gives its storage another meaning.
const at::Tensor* plain_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  static const c10::DispatchKeySet special(
      {c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::Functionalize,
       c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::BatchedNestedTensor,
       c10::DispatchKey::Conjugate, c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.is_quantized() ||
      t.key_set().has_any(special) || !t.is_contiguous())
    return nullptr;
  return &t;
}

// Collects pointers while everything is as expected.
struct Args {
  bool ok = true;
  c10::Device device{c10::DeviceType::CUDA, -1};

  const at::Tensor* first(PyObject* o, size_t dims) {
    const at::Tensor* t = plain_tensor(o);
    if (t == nullptr || static_cast<size_t>(t->dim()) != dims) {
      ok = false;
      return nullptr;
    }
    device = t->device();
    return t;
  }
  void* tensor(PyObject* o, std::initializer_list<int64_t> shape, ScalarType type) {
    const at::Tensor* t = ok ? plain_tensor(o) : nullptr;
    if (t == nullptr || t->scalar_type() != type || t->device() != device ||
        t->sizes() != c10::IntArrayRef(shape.begin(), shape.size())) {
      ok = false;
      return nullptr;
    }
    return t->data_ptr();
  }
  void* optional(PyObject* o, std::initializer_list<int64_t> shape, ScalarType type) {
    return o == Py_None ? nullptr : tensor(o, shape, type);
  }
  // The workspace's bytes (as many as `bytes` says, which the library checks).
  void* workspace(PyObject* o) {
    const at::Tensor* t = ok ? plain_tensor(o) : nullptr;
    if (t == nullptr) {
      ok = false;
      return nullptr;
    }
    return t->data_ptr();
  }
  float number(PyObject* o) {
    if (!PyFloat_CheckExact(o)) {
      ok = false;
      return 0.0f;
    }
    return static_cast<float>(PyFloat_AS_DOUBLE(o));
  }
  size_t integer(PyObject* o) {
    if (!PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    const size_t v = PyLong_AsSize_t(o);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return v;
  }
  template <typename T>
  T address(PyObject* o) {
    return reinterpret_cast<T>(integer(o));
  }
};

// Modes that watch tensor operations see the call through binding.py's path.
bool watched() {
  return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}

constexpr ScalarType F32 = ScalarType::Float, BF16 = ScalarType::BFloat16, I32 = ScalarType::Int;

bool logits_type(const at::Tensor& t, vtrace_dtype* code) {
  *code = t.scalar_type() == BF16 ? VTRACE_BF16 : VTRACE_F32;
  return t.scalar_type() == BF16 || t.scalar_type() == F32;
}

// targets(fn, target, behaviour, actions, rewards, discounts, values, bootstrap,
//         rho_bar, c_bar, lambda, variant, log_probs, vs, pg, workspace, bytes, stream)
PyObject* targets(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n != 18 || watched()) Py_RETURN_NONE;
  Args a;
  const at::Tensor* z = a.first(v[1], 3);
  vtrace_dtype dt;
  if (!a.ok || !logits_type(*z, &dt)) Py_RETURN_NONE;
  const int64_t T = z->size(0), B = z->size(1), A = z->size(2);
  const auto fn = a.address<decltype(&vtrace_targets_ex)>(v[0]);
  void* const y = v[12] == Py_True ? a.tensor(v[2], {T, B}, F32) : a.tensor(v[2], {T, B, A}, z->scalar_type());
  void* const act = a.tensor(v[3], {T, B}, I32);
  void* const r = a.tensor(v[4], {T, B}, F32);
  void* const g = a.tensor(v[5], {T, B}, F32);
  void* const val = a.tensor(v[6], {T, B}, F32);
  void* const boot = a.tensor(v[7], {B}, F32);
  const float rho = a.number(v[8]), c = a.number(v[9]), lam = a.number(v[10]);
  const auto variant = a.address<const vtrace_variant*>(v[11]);
  void* const vs = a.tensor(v[13], {T, B}, F32);
  void* const pg = a.tensor(v[14], {T, B}, F32);
  void* const ws = v[15] == Py_None ? nullptr : a.workspace(v[15]);
  const size_t bytes = a.integer(v[16]);
  const auto stream = a.address<vtrace_stream_t>(v[17]);
  if (!a.ok) Py_RETURN_NONE;
  vtrace_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = fn(T, B, A, dt, z->data_ptr(), y, static_cast<const int32_t*>(act), static_cast<const float*>(r),
          static_cast<const float*>(g), static_cast<const float*>(val), static_cast<const float*>(boot), rho, c, lam,
          variant, static_cast<float*>(vs), static_cast<float*>(pg), ws, bytes, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(st);
}

// loss(fn, target, behaviour, actions, rewards, discounts, values, bootstrap, rho_bar,
//      c_bar, lambda, baseline_cost, entropy_cost, variant, log_probs, bf16_grad, losses,
//      d_logits, d_values, vs, pg, lane_losses, workspace, bytes, stream)
PyObject* loss(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n != 25 || watched()) Py_RETURN_NONE;
  Args a;
  const at::Tensor* z = a.first(v[1], 3);
  vtrace_dtype dt;
  if (!a.ok || !logits_type(*z, &dt)) Py_RETURN_NONE;
  const int64_t T = z->size(0), B = z->size(1), A = z->size(2);
  const auto fn = a.address<decltype(&vtrace_loss_grad_ex)>(v[0]);
  void* const y = v[14] == Py_True ? a.tensor(v[2], {T, B}, F32) : a.tensor(v[2], {T, B, A}, z->scalar_type());
  void* const act = a.tensor(v[3], {T, B}, I32);
  void* const r = a.tensor(v[4], {T, B}, F32);
  void* const g = a.tensor(v[5], {T, B}, F32);
  void* const val = a.tensor(v[6], {T, B}, F32);
  void* const boot = a.tensor(v[7], {B}, F32);
  const float rho = a.number(v[8]), c = a.number(v[9]), lam = a.number(v[10]);
  const float bc = a.number(v[11]), ec = a.number(v[12]);
  const auto variant = a.address<const vtrace_variant*>(v[13]);
  void* const losses = a.tensor(v[16], {4}, F32);
  void* const dl = a.tensor(v[17], {T, B, A}, v[15] == Py_True ? BF16 : F32);
  void* const dv = a.tensor(v[18], {T, B}, F32);
  void* const vs = a.optional(v[19], {T, B}, F32);
  void* const pg = a.optional(v[20], {T, B}, F32);
  void* const lane = a.optional(v[21], {B, 3}, F32);
  void* const ws = a.workspace(v[22]);
  const size_t bytes = a.integer(v[23]);
  const auto stream = a.address<vtrace_stream_t>(v[24]);
  if (!a.ok) Py_RETURN_NONE;
  vtrace_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = fn(T, B, A, dt, z->data_ptr(), y, static_cast<const int32_t*>(act), static_cast<const float*>(r),
          static_cast<const float*>(g), static_cast<const float*>(val), static_cast<const float*>(boot), rho, c, lam,
          bc, ec, variant, static_cast<float*>(losses), dl, static_cast<float*>(dv), static_cast<float*>(vs),
          static_cast<float*>(pg), static_cast<float*>(lane), ws, bytes, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(st);
}

// head(fn, hidden, weight, bias, behaviour, actions, rewards, discounts, bootstrap, rho_bar,
//      c_bar, lambda, baseline_cost, entropy_cost, variant, log_probs, bf16_grad, losses,
//      d_hidden, d_weight, d_bias, vs, pg, lane_losses, outputs, workspace, bytes, stream)
PyObject* head(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n != 28 || watched()) Py_RETURN_NONE;
  Args a;
  const at::Tensor* h = a.first(v[1], 3);
  const at::Tensor* w = a.ok ? plain_tensor(v[2]) : nullptr;
  if (h == nullptr || w == nullptr || h->scalar_type() != BF16 || w->dim() != 2) Py_RETURN_NONE;
  const int64_t T = h->size(0), B = h->size(1), H = h->size(2), A = w->size(1) - 1;
  const auto fn = a.address<decltype(&vtrace_head_loss_grad)>(v[0]);
  void* const weight = a.tensor(v[2], {H, A + 1}, BF16);
  void* const bias = a.tensor(v[3], {A + 1}, F32);
  vtrace_dtype dt = VTRACE_F32;
  void* y = nullptr;
  if (v[15] == Py_True) {
    y = a.tensor(v[4], {T, B}, F32);
  } else {
    const at::Tensor* b = plain_tensor(v[4]);
    if (b == nullptr || !logits_type(*b, &dt)) Py_RETURN_NONE;
    y = a.tensor(v[4], {T, B, A}, b->scalar_type());
  }
  void* const act = a.tensor(v[5], {T, B}, I32);
  void* const r = a.tensor(v[6], {T, B}, F32);
  void* const g = a.tensor(v[7], {T, B}, F32);
  void* const boot = a.tensor(v[8], {B}, F32);
  const float rho = a.number(v[9]), c = a.number(v[10]), lam = a.number(v[11]);
  const float bc = a.number(v[12]), ec = a.number(v[13]);
  const auto variant = a.address<const vtrace_variant*>(v[14]);
  void* const losses = a.tensor(v[17], {4}, F32);
  void* const dh = a.tensor(v[18], {T, B, H}, v[16] == Py_True ? BF16 : F32);
  void* const dw = a.tensor(v[19], {H, A + 1}, F32);
  void* const db = a.tensor(v[20], {A + 1}, F32);
  void* const vs = a.optional(v[21], {T, B}, F32);
  void* const pg = a.optional(v[22], {T, B}, F32);
  void* const lane = a.optional(v[23], {B, 3}, F32);
  void* const outs = a.optional(v[24], {T, B, A + 1}, F32);
  void* const ws = a.workspace(v[25]);
  const size_t bytes = a.integer(v[26]);
  const auto stream = a.address<vtrace_stream_t>(v[27]);
  if (!a.ok) Py_RETURN_NONE;
  vtrace_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = fn(T, B, A, H, dt, h->data_ptr(), weight, static_cast<const float*>(bias), y, static_cast<const int32_t*>(act),
          static_cast<const float*>(r), static_cast<const float*>(g), static_cast<const float*>(boot), rho, c, lam, bc,
          ec, variant, static_cast<float*>(losses), dh, static_cast<float*>(dw), static_cast<float*>(db),
          static_cast<float*>(vs), static_cast<float*>(pg), static_cast<float*>(lane), static_cast<float*>(outs), ws,
          bytes, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(st);
}

// A C++ exception (none is expected: every access is checked first) leaves the
// call to binding.py's path.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* v, Py_ssize_t n) {
  try {
    return F(self, v, n);
  } catch (...) {
    Py_RETURN_NONE;
  }
}

#define METHOD(name) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(targets), METHOD(loss), METHOD(head), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast_call(void) { return PyModule_Create(&module); }
