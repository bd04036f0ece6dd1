// The calls of api.py in native code, for arguments that are plainly valid: the same checks as there, the output
// and workspace allocations, and the C-ABI call.  Every function here takes api.py's arguments in order and
// returns what that function returns -- or None where anything is missing, of another type, shape or device, or
// not an ordinary tensor; api.py then looks at the arguments one by one, for its message or for the forms only
// it takes.  An error status goes to api.py's exception.
//
// What it is for: a call is one to five launches of a few microseconds each, and checking and marshalling its
// operands in Python took longer (host time per call: forward of one token 15 us, forward and backward of 64
// tokens 56 us for 38 us on the GPU, AdamW over 14 tensors 31 for 20).
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/Functions.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include <algorithm>
#include <cstring>
#include <utility>

#include "../../include/qalora.h"

namespace {

// Entry points of the C-ABI library api.py has loaded.
struct Library {
#define QALORA_ENTRIES(X)                                                                                            \
  X(qalora_check_desc) X(qalora_packed_bytes) X(qalora_workspace_bytes) X(qalora_quantize) X(qalora_forward)          \
  X(qalora_kept_bytes) X(qalora_forward_keep) X(qalora_backward) X(qalora_backward_kept) X(qalora_deployed_bytes)     \
  X(qalora_forward_deployed) X(qalora_forward_factors16) X(qalora_adamw_step) X(qalora_shared_kept_bytes)             \
  X(qalora_shared_workspace_bytes) X(qalora_forward_shared) X(qalora_backward_shared) X(qalora_swiglu_forward_wide)   \
  X(qalora_swiglu_backward_wide)
#define QALORA_MEMBER(name) decltype(&::name) name = nullptr;
  QALORA_ENTRIES(QALORA_MEMBER)
} lib;
PyObject* raise_status = nullptr;  // api.py: (status, entry point) -> raises
PyObject *desc_type = nullptr, *adamw_type = nullptr;  // api.py's mirrors of qalora_desc and qalora_adamw
bool bound = false;

// The operands of one call, held until it returns (a list they came in can change while the interpreter lock is
// released).  Held by their Python objects: a tensor's own count is atomic (AdamW over 14 adapter tensors, host time a
// call: 7.7 us by tensors in a vector, 6.6 so).  `ok` falls once anything is not plainly right.
struct Call {
  static constexpr int kMostHeld = 4 * 32 + 16;  // an optimiser step's
  bool ok = true;
  int n_held = 0;
  PyObject* held[kMostHeld];
  qalora_desc desc{};
  c10::Device dev{c10::DeviceType::CPU};
  int64_t T = 0, L = 0;

  // (under a mode the allocations below would have to go through Python)
  Call() { ok = bound && !at::impl::torch_function_mode_enabled() && !c10::impl::dispatch_mode_enabled(); }
  ~Call() {
    while (n_held > 0) Py_DECREF(held[--n_held]);
  }
  Call(const Call&) = delete;
  void need(bool v) { ok = ok && v; }

  // an ordinary, contiguous tensor on a GPU, the call's from the first one on
  const at::Tensor* tensor(PyObject* o, bool first = false) {
    if (!ok || !THPVariable_CheckExact(o)) {
      ok = false;
      return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() ||
        t.unsafeGetTensorImpl()->is_python_dispatch() || !t.is_contiguous() || t.is_neg() || t.is_conj()) {
      ok = false;
      return nullptr;
    }
    if (first) dev = t.device();
    need(t.device() == dev);
    need(n_held < kMostHeld);
    if (!ok) return nullptr;
    Py_INCREF(o);
    held[n_held++] = o;
    return &t;
  }
  void* matrix(PyObject* o, at::ScalarType dtype, int64_t rows, int64_t cols) {
    const at::Tensor* t = tensor(o);
    need(t && t->scalar_type() == dtype && t->dim() == 2 && t->size(0) == rows && t->size(1) == cols);
    return ok ? t->data_ptr() : nullptr;
  }
  void* bytes(PyObject* o, size_t at_least) {
    const at::Tensor* t = tensor(o);
    need(t && (size_t)t->nbytes() >= at_least);
    return ok ? t->data_ptr() : nullptr;
  }
  // x or dy, from which the call takes its tokens and device
  void* activations(PyObject* o, int64_t width) {
    const at::Tensor* t = tensor(o, true);
    need(t && t->scalar_type() == at::kBFloat16 && t->dim() == 2 && t->size(1) == width && t->size(0) > 0 &&
         t->size(0) <= INT32_MAX);
    if (!ok) return nullptr;
    T = t->size(0);
    return t->data_ptr();
  }
  template <typename S>
  void read_struct(PyObject* o, PyObject* type, S& out) {  // a ctypes mirror
    Py_buffer b;
    if (!ok || !PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type)) || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
      PyErr_Clear();
      ok = false;
      return;
    }
    if (b.len == (Py_ssize_t)sizeof(S)) std::memcpy(&out, b.buf, sizeof(S));
    else ok = false;
    PyBuffer_Release(&b);
  }
  void layer(PyObject* d) {
    read_struct(d, desc_type, desc);
    need(ok && lib.qalora_check_desc(&desc) == QALORA_OK);
    if (ok) L = desc.d_in / desc.group;
  }
  int dtype_of(at::ScalarType t) {
    need(t == at::kFloat || t == at::kBFloat16);
    return t == at::kBFloat16 ? QALORA_BF16 : QALORA_F32;
  }
  // an output matrix: the caller's, or a new one of the given type
  at::Tensor out(PyObject* o, PyObject* dtype, int64_t rows, int64_t cols, int& code) {
    if (!ok) return {};
    if (o == Py_None) {
      if (!THPDtype_Check(dtype)) {
        ok = false;
        return {};
      }
      const at::ScalarType st = reinterpret_cast<THPDtype*>(dtype)->scalar_type;
      code = dtype_of(st);
      return ok ? at::empty({rows, cols}, at::TensorOptions().dtype(st).device(dev)) : at::Tensor();
    }
    const at::Tensor* t = tensor(o);
    need(t && t->dim() == 2 && t->size(0) == rows && t->size(1) == cols);
    if (!ok) return {};
    code = dtype_of(t->scalar_type());
    return *t;
  }
  at::Tensor scratch(PyObject* o, size_t size) {  // the caller's, or new
    if (!ok) return {};
    if (o == Py_None)
      return at::empty({(int64_t)std::max<size_t>(size, 16)}, at::TensorOptions().dtype(at::kByte).device(dev));
    const at::Tensor* t = tensor(o);
    return t ? *t : at::Tensor();
  }
  bool truth(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) {
      PyErr_Clear();
      ok = false;
    }
    return v > 0;
  }
};

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Runs the C call without the interpreter lock; false: a Python exception is set.  Its arguments are evaluated by
// the caller, under the lock: reading a tensor's address can allocate (a lazily cloned one is copied then) and throw.
template <typename... P, typename... A>
bool run(const char* name, int (*f)(P...), A... args) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f(args...);
  Py_END_ALLOW_THREADS
  if (rc == QALORA_OK) return true;
  PyObject* r = PyObject_CallFunction(raise_status, "is", rc, name);
  Py_XDECREF(r);
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, name);
  return false;
}

PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }
// what the caller gave, or the new tensor
PyObject* given_or(PyObject* o, const at::Tensor& t) {
  if (o == Py_None) return wrap(t);
  Py_INCREF(o);
  return o;
}
PyObject* tuple(std::initializer_list<PyObject*> items) {
  PyObject* r = PyTuple_New((Py_ssize_t)items.size());
  Py_ssize_t i = 0;
  for (PyObject* o : items) PyTuple_SET_ITEM(r, i++, o);
  return r;
}
float* f32(void* p) { return static_cast<float*>(p); }

struct Weights {
  void *packed = nullptr, *alpha = nullptr, *beta = nullptr, *A = nullptr, *B = nullptr;
};
Weights weights(Call& c, PyObject* packed, PyObject* alpha, PyObject* beta) {
  Weights w;
  if (!c.ok) return w;
  w.packed = c.bytes(packed, lib.qalora_packed_bytes(&c.desc));
  w.alpha = c.matrix(alpha, at::kFloat, c.L, c.desc.d_out);
  w.beta = c.matrix(beta, at::kFloat, c.L, c.desc.d_out);
  return w;
}
void adapter(Call& c, PyObject* A, PyObject* B, Weights& w) {
  c.need((A == Py_None) == (B == Py_None));
  if (!c.ok || A == Py_None) return;
  w.A = c.matrix(A, at::kFloat, c.L, c.desc.rank);
  w.B = c.matrix(B, at::kFloat, c.desc.rank, c.desc.d_out);
}

#define FASTCALL(name, count) \
  PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) { \
    HANDLE_TH_ERRORS \
    if (n != count) { PyErr_SetString(PyExc_TypeError, #name ": " #count " arguments"); return nullptr; }
#define FASTCALL_END END_HANDLE_TH_ERRORS }
#define PLAIN(c) if (!(c).ok) Py_RETURN_NONE

// desc, W
FASTCALL(quantize, 2)
  Call c;
  c.layer(a[0]);
  const at::Tensor* W = c.tensor(a[1], true);
  c.need(W && W->scalar_type() == at::kFloat && W->dim() == 2 && W->size(0) == c.desc.d_in && W->size(1) == c.desc.d_out);
  PLAIN(c);
  const auto opts = at::TensorOptions().device(c.dev);
  const at::Tensor packed = at::empty({(int64_t)lib.qalora_packed_bytes(&c.desc)}, opts.dtype(at::kByte));
  const at::Tensor alpha = at::empty({c.L, c.desc.d_out}, opts.dtype(at::kFloat)), beta = at::empty_like(alpha);
  void* st = stream();
  if (!run("qalora_quantize", lib.qalora_quantize, &c.desc, f32(W->data_ptr()), packed.data_ptr(), f32(alpha.data_ptr()),
           f32(beta.data_ptr()), nullptr, 0, st))
    return nullptr;
  return tuple({wrap(packed), wrap(alpha), wrap(beta)});
FASTCALL_END

// desc, x, packed, alpha, beta, A, B, out_dtype, ws, y
FASTCALL(forward, 10)
  Call c;
  c.layer(a[0]);
  void* x = c.activations(a[1], c.desc.d_in);
  Weights w = weights(c, a[2], a[3], a[4]);
  adapter(c, a[5], a[6], w);
  int code = 0;
  const at::Tensor y = c.out(a[9], a[7], c.T, c.desc.d_out, code);
  PLAIN(c);
  const at::Tensor ws = c.scratch(a[8], a[8] == Py_None ? lib.qalora_workspace_bytes(&c.desc, (int)c.T, QALORA_OP_FORWARD) : 0);
  PLAIN(c);
  void* st = stream();
  if (!run("qalora_forward", lib.qalora_forward, &c.desc, (int)c.T, x, w.packed, f32(w.alpha), f32(w.beta), f32(w.A),
           f32(w.B), y.data_ptr(), code, ws.data_ptr(), ws.nbytes(), st))
    return nullptr;
  return given_or(a[9], y);
FASTCALL_END

// desc, x, packed, alpha, beta, A, B, out_dtype, ws, y, kept
FASTCALL(forward_keep, 11)
  Call c;
  c.layer(a[0]);
  void* x = c.activations(a[1], c.desc.d_in);
  Weights w = weights(c, a[2], a[3], a[4]);
  c.need(a[5] != Py_None);
  adapter(c, a[5], a[6], w);
  int code = 0;
  const at::Tensor y = c.out(a[9], a[7], c.T, c.desc.d_out, code);
  PLAIN(c);
  const size_t keep = lib.qalora_kept_bytes(&c.desc, (int)c.T);
  const at::Tensor kept = c.scratch(a[10], keep);
  const at::Tensor ws = c.scratch(a[8], a[8] == Py_None ? lib.qalora_workspace_bytes(&c.desc, (int)c.T, QALORA_OP_FORWARD) : 0);
  c.need(c.ok && (size_t)kept.nbytes() >= keep);
  PLAIN(c);
  void* st = stream();
  if (!run("qalora_forward_keep", lib.qalora_forward_keep, &c.desc, (int)c.T, x, w.packed, f32(w.alpha), f32(w.beta),
           f32(w.A), f32(w.B), y.data_ptr(), code, kept.data_ptr(), ws.data_ptr(), ws.nbytes(), st))
    return nullptr;
  return tuple({given_or(a[9], y), given_or(a[10], kept)});
FASTCALL_END

// The backward of one layer: `x` or `kept` is null.
PyObject* backward_of(Call& c, void* dy, void* x, void* kept, const Weights& w, PyObject* want_dx, PyObject* dx_dtype,
                      PyObject* pA, PyObject* pB, PyObject* pdA, PyObject* pdB, PyObject* accumulate, PyObject* pws,
                      PyObject* pdx) {
  int code = 0;
  at::Tensor dx, dA, dB;
  if (c.ok && (pdx != Py_None || c.truth(want_dx))) dx = c.out(pdx, dx_dtype, c.T, c.desc.d_in, code);
  const bool acc = c.truth(accumulate);
  if (c.ok && w.A) {
    if (pdA != Py_None) c.matrix(pdA, at::kFloat, c.L, c.desc.rank);
    if (pdB != Py_None) c.matrix(pdB, at::kFloat, c.desc.rank, c.desc.d_out);
    if (c.ok) dA = pdA != Py_None ? THPVariable_Unpack(pdA) : at::zeros_like(THPVariable_Unpack(pA));
    if (c.ok) dB = pdB != Py_None ? THPVariable_Unpack(pdB) : at::zeros_like(THPVariable_Unpack(pB));
  } else {
    c.need(pdA == Py_None && pdB == Py_None);
  }
  PLAIN(c);
  const at::Tensor ws = c.scratch(pws, pws == Py_None ? lib.qalora_workspace_bytes(&c.desc, (int)c.T, QALORA_OP_BACKWARD) : 0);
  PLAIN(c);
  void* pdx_data = dx.defined() ? dx.data_ptr() : nullptr;
  float* gA = dA.defined() ? f32(dA.data_ptr()) : nullptr;
  float* gB = dB.defined() ? f32(dB.data_ptr()) : nullptr;
  void* st = stream();
  const bool done =
      kept ? run("qalora_backward_kept", lib.qalora_backward_kept, &c.desc, (int)c.T, dy, kept, w.packed, f32(w.alpha),
                 f32(w.beta), f32(w.A), f32(w.B), pdx_data, code, gA, gB, acc, ws.data_ptr(), ws.nbytes(), st)
           : run("qalora_backward", lib.qalora_backward, &c.desc, (int)c.T, dy, x, w.packed, f32(w.alpha), f32(w.beta),
                 f32(w.A), f32(w.B), pdx_data, code, gA, gB, acc, ws.data_ptr(), ws.nbytes(), st);
  if (!done) return nullptr;
  return tuple({dx.defined() ? given_or(pdx, dx) : Py_NewRef(Py_None), dA.defined() ? given_or(pdA, dA) : Py_NewRef(Py_None),
                dB.defined() ? given_or(pdB, dB) : Py_NewRef(Py_None)});
}

// desc, dy, x, packed, alpha, beta, A, B, want_dx, dx_dtype, dA, dB, accumulate, ws, dx
FASTCALL(backward, 15)
  Call c;
  c.layer(a[0]);
  void* dy = c.activations(a[1], c.desc.d_out);
  Weights w = weights(c, a[3], a[4], a[5]);
  adapter(c, a[6], a[7], w);
  void* x = nullptr;
  if (c.ok && (w.A || a[2] != Py_None)) x = c.matrix(a[2], at::kBFloat16, c.T, c.desc.d_in);
  return backward_of(c, dy, x, nullptr, w, a[8], a[9], a[6], a[7], a[10], a[11], a[12], a[13], a[14]);
FASTCALL_END

// desc, dy, kept, packed, alpha, beta, A, B, want_dx, dx_dtype, dA, dB, accumulate, ws, dx
FASTCALL(backward_kept, 15)
  Call c;
  c.layer(a[0]);
  void* dy = c.activations(a[1], c.desc.d_out);
  Weights w = weights(c, a[3], a[4], a[5]);
  c.need(a[6] != Py_None);
  adapter(c, a[6], a[7], w);
  void* kept = c.ok ? c.bytes(a[2], lib.qalora_kept_bytes(&c.desc, (int)c.T)) : nullptr;
  c.need(kept != nullptr);
  return backward_of(c, dy, nullptr, kept, w, a[8], a[9], a[6], a[7], a[10], a[11], a[12], a[13], a[14]);
FASTCALL_END

// desc, x, deployed, packed, out_dtype, ws, y
FASTCALL(forward_deployed, 7)
  Call c;
  c.layer(a[0]);
  void* x = c.activations(a[1], c.desc.d_in);
  PLAIN(c);
  const size_t need = lib.qalora_deployed_bytes(&c.desc);
  c.need(need > 0);
  void* deployed = c.bytes(a[2], need);
  void* packed = nullptr;
  if (c.ok && (a[3] != Py_None || c.T > QALORA_DEPLOYED_STREAM_TOKENS))
    packed = c.bytes(a[3], c.T > QALORA_DEPLOYED_STREAM_TOKENS ? lib.qalora_packed_bytes(&c.desc) : 0);
  int code = 0;
  const at::Tensor y = c.out(a[6], a[4], c.T, c.desc.d_out, code);
  PLAIN(c);
  const at::Tensor ws = c.scratch(a[5], a[5] == Py_None ? lib.qalora_workspace_bytes(&c.desc, (int)c.T, QALORA_OP_FORWARD) : 0);
  PLAIN(c);
  void* st = stream();
  if (!run("qalora_forward_deployed", lib.qalora_forward_deployed, &c.desc, (int)c.T, x, packed, deployed, y.data_ptr(),
           code, ws.data_ptr(), ws.nbytes(), st))
    return nullptr;
  return given_or(a[6], y);
FASTCALL_END

// desc, x, packed, factors16, out_dtype, ws, y
FASTCALL(forward_factors16, 7)
  Call c;
  c.layer(a[0]);
  void* x = c.activations(a[1], c.desc.d_in);
  PLAIN(c);
  void* packed = c.bytes(a[2], lib.qalora_packed_bytes(&c.desc));
  void* fac = c.bytes(a[3], (size_t)4 * c.L * c.desc.d_out);
  int code = 0;
  const at::Tensor y = c.out(a[6], a[4], c.T, c.desc.d_out, code);
  PLAIN(c);
  const at::Tensor ws =
      c.scratch(a[5], a[5] == Py_None ? lib.qalora_workspace_bytes(&c.desc, (int)c.T, QALORA_OP_FORWARD_FACTORS16) : 0);
  PLAIN(c);
  void* st = stream();
  if (!run("qalora_forward_factors16", lib.qalora_forward_factors16, &c.desc, (int)c.T, x, packed, fac, y.data_ptr(), code,
           ws.data_ptr(), ws.nbytes(), st))
    return nullptr;
  return given_or(a[6], y);
FASTCALL_END

// A list or tuple of `count` items, borrowed.
PyObject** items(Call& c, PyObject* o, Py_ssize_t count) {
  if (!c.ok || !(PyList_CheckExact(o) || PyTuple_CheckExact(o)) || PySequence_Fast_GET_SIZE(o) != count) {
    c.ok = false;
    return nullptr;
  }
  return PySequence_Fast_ITEMS(o);
}

// The adapters (A, B, s) of linears that share x, and where the backward puts their gradients.
struct Parts {
  int n = 0;
  qalora_part p[QALORA_MAX_PARTS] = {};
};
Parts parts(Call& c, PyObject* adapters, PyObject* grads) {
  Parts r;
  if (!c.ok || !(PyList_CheckExact(adapters) || PyTuple_CheckExact(adapters))) {
    c.ok = false;
    return r;
  }
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(adapters);
  c.need(n >= 1 && n <= QALORA_MAX_PARTS);
  PyObject** list = items(c, adapters, n);
  PyObject** glist = grads ? items(c, grads, n) : nullptr;
  int64_t width = 0;
  for (Py_ssize_t q = 0; c.ok && q < n; ++q) {
    PyObject** abs = items(c, list[q], 3);
    const at::Tensor* A = c.ok ? c.tensor(abs[0]) : nullptr;
    const at::Tensor* B = c.ok ? c.tensor(abs[1]) : nullptr;
    c.need(A && B && A->scalar_type() == at::kFloat && B->scalar_type() == at::kFloat && A->dim() == 2 && B->dim() == 2 &&
           A->size(0) == c.L && A->size(1) == B->size(0) && B->size(1) <= INT32_MAX && A->size(1) <= INT32_MAX &&
           (PyFloat_CheckExact(abs[2]) || PyLong_CheckExact(abs[2])));
    if (!c.ok) return r;
    const double s = PyFloat_AsDouble(abs[2]);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      c.ok = false;
      return r;
    }
    qalora_part& p = r.p[q];
    p.d_out = (int32_t)B->size(1);
    p.rank = (int32_t)A->size(1);
    p.s = (float)s;
    p.A = f32(A->data_ptr());
    p.B = f32(B->data_ptr());
    width += p.d_out;
    if (grads) {
      PyObject** g = items(c, glist[q], 2);
      if (!c.ok) return r;
      p.dA = f32(c.matrix(g[0], at::kFloat, A->size(0), A->size(1)));
      p.dB = f32(c.matrix(g[1], at::kFloat, B->size(0), B->size(1)));
    }
  }
  c.need(width == c.desc.d_out);
  r.n = (int)n;
  return r;
}

// desc, x, packed, alpha, beta, adapters, keep, out_dtype, ws, y, kept
FASTCALL(forward_shared, 11)
  Call c;
  c.layer(a[0]);
  void* x = c.activations(a[1], c.desc.d_in);
  Weights w = weights(c, a[2], a[3], a[4]);
  const Parts p = parts(c, a[5], nullptr);
  const bool keep = c.truth(a[6]);
  int code = 0;
  const at::Tensor y = c.out(a[9], a[7], c.T, c.desc.d_out, code);
  PLAIN(c);
  at::Tensor kept;
  if (keep) {
    const size_t kb = lib.qalora_shared_kept_bytes(&c.desc, (int)c.T, p.n, p.p);
    kept = c.scratch(a[10], kb);
    c.need(c.ok && (size_t)kept.nbytes() >= kb);
  }
  const at::Tensor ws = c.scratch(
      a[8], a[8] == Py_None ? lib.qalora_shared_workspace_bytes(&c.desc, (int)c.T, QALORA_OP_FORWARD, p.n, p.p) : 0);
  PLAIN(c);
  void* st = stream();
  if (!run("qalora_forward_shared", lib.qalora_forward_shared, &c.desc, (int)c.T, x, w.packed, f32(w.alpha), f32(w.beta),
           p.n, p.p, y.data_ptr(), code, keep ? kept.data_ptr() : nullptr, ws.data_ptr(), ws.nbytes(), st))
    return nullptr;
  if (!keep) return given_or(a[9], y);
  return tuple({given_or(a[9], y), given_or(a[10], kept)});
FASTCALL_END

// desc, dy, x, kept, packed, alpha, beta, adapters, want_dx, dx_dtype, grads, accumulate, ws, dx -> dx
FASTCALL(backward_shared, 14)
  Call c;
  c.layer(a[0]);
  void* dy = c.activations(a[1], c.desc.d_out);
  Weights w = weights(c, a[4], a[5], a[6]);
  c.need(a[10] != Py_None);
  const Parts p = parts(c, a[7], a[10]);
  PLAIN(c);
  void *x = nullptr, *kept = nullptr;
  if (a[3] == Py_None) x = c.matrix(a[2], at::kBFloat16, c.T, c.desc.d_in);
  else kept = c.bytes(a[3], lib.qalora_shared_kept_bytes(&c.desc, (int)c.T, p.n, p.p));
  int code = 0;
  at::Tensor dx;
  if (c.ok && (a[13] != Py_None || c.truth(a[8]))) dx = c.out(a[13], a[9], c.T, c.desc.d_in, code);
  const bool acc = c.truth(a[11]);
  PLAIN(c);
  const at::Tensor ws = c.scratch(
      a[12], a[12] == Py_None ? lib.qalora_shared_workspace_bytes(&c.desc, (int)c.T, QALORA_OP_BACKWARD, p.n, p.p) : 0);
  PLAIN(c);
  void* pdx = dx.defined() ? dx.data_ptr() : nullptr;
  void* st = stream();
  if (!run("qalora_backward_shared", lib.qalora_backward_shared, &c.desc, (int)c.T, dy, x, kept, w.packed, f32(w.alpha),
           f32(w.beta), p.n, p.p, pdx, code, acc, ws.data_ptr(), ws.nbytes(), st))
    return nullptr;
  return tuple({dx.defined() ? given_or(a[13], dx) : Py_NewRef(Py_None), Py_NewRef(a[10])});
FASTCALL_END

// gu, cols, out
FASTCALL(swiglu_forward_wide, 3)
  Call c;
  const at::Tensor* gu = c.tensor(a[0], true);
  c.need(PyLong_CheckExact(a[1]));
  PLAIN(c);
  const long long cols = PyLong_AsLongLong(a[1]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  c.need(cols > 0 && cols < (1ll << 40) && gu->scalar_type() == at::kBFloat16 && gu->dim() == 2 && gu->size(1) == 2 * cols);
  PLAIN(c);
  const int64_t rows = gu->size(0);
  at::Tensor out;
  if (a[2] == Py_None) {
    out = at::empty({rows, cols}, gu->options());
  } else {
    c.matrix(a[2], at::kBFloat16, rows, cols);
    PLAIN(c);
    out = THPVariable_Unpack(a[2]);
  }
  void* st = stream();
  if (!run("qalora_swiglu_forward_wide", lib.qalora_swiglu_forward_wide, gu->data_ptr(), out.data_ptr(), (size_t)rows,
           (size_t)cols, st))
    return nullptr;
  return given_or(a[2], out);
FASTCALL_END

// dh, gu, cols, out
FASTCALL(swiglu_backward_wide, 4)
  Call c;
  const at::Tensor* gu = c.tensor(a[1], true);
  c.need(PyLong_CheckExact(a[2]));
  PLAIN(c);
  const long long cols = PyLong_AsLongLong(a[2]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  c.need(cols > 0 && cols < (1ll << 40) && gu->scalar_type() == at::kBFloat16 && gu->dim() == 2 && gu->size(1) == 2 * cols);
  PLAIN(c);
  const int64_t rows = gu->size(0);
  void* dh = c.matrix(a[0], at::kBFloat16, rows, cols);
  PLAIN(c);
  at::Tensor out;
  if (a[3] == Py_None) {
    out = at::empty({rows, 2 * cols}, gu->options());
  } else {
    c.matrix(a[3], at::kBFloat16, rows, 2 * cols);
    PLAIN(c);
    out = THPVariable_Unpack(a[3]);
  }
  void* st = stream();
  if (!run("qalora_swiglu_backward_wide", lib.qalora_swiglu_backward_wide, dh, gu->data_ptr(), out.data_ptr(), (size_t)rows,
           (size_t)cols, st))
    return nullptr;
  return given_or(a[3], out);
FASTCALL_END

// hp, step, params, grads, exp_avg, exp_avg_sq, zero_grads, grad_norm, ws -> True
FASTCALL(adamw_step, 9)
  constexpr Py_ssize_t kMost = 32;
  Call c;
  qalora_adamw hp{};
  c.read_struct(a[0], adamw_type, hp);
  c.need(PyLong_CheckExact(a[1]) && (PyList_CheckExact(a[2]) || PyTuple_CheckExact(a[2])));
  PLAIN(c);
  const long step = PyLong_AsLong(a[1]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  const Py_ssize_t count = PySequence_Fast_GET_SIZE(a[2]);
  c.need(step >= 1 && step <= INT32_MAX && count >= 1 && count <= kMost);
  float* ptr[4][kMost];
  size_t numel[kMost];
  PyObject** first = items(c, a[2], count);
  for (int l = 0; c.ok && l < 4; ++l) {
    PyObject** list = items(c, a[2 + l], count);
    for (Py_ssize_t i = 0; c.ok && i < count; ++i) {
      const at::Tensor* t = c.tensor(list[i], l == 0 && i == 0);
      c.need(t && t->scalar_type() == at::kFloat && (l == 0 || t->sizes() == THPVariable_Unpack(first[i]).sizes()));
      if (!c.ok) break;
      ptr[l][i] = f32(t->data_ptr());
      numel[i] = (size_t)t->numel();
    }
  }
  c.need(a[8] != Py_None);
  const at::Tensor* ws = c.ok ? c.tensor(a[8]) : nullptr;
  float* norm = nullptr;
  if (c.ok && a[7] != Py_None) {
    const at::Tensor* t = c.tensor(a[7]);
    c.need(t && t->scalar_type() == at::kFloat && t->nbytes() >= 4);
    if (c.ok) norm = f32(t->data_ptr());
  }
  const bool zero = c.truth(a[6]);
  // (api.py passes the number of elements of ws for its size in bytes)
  PLAIN(c);
  void* st = stream();
  if (!run("qalora_adamw_step", lib.qalora_adamw_step, &hp, (int)step, (int)count, ptr[0], ptr[1], ptr[2], ptr[3], numel,
           zero, norm, ws->data_ptr(), (size_t)ws->numel(), st))
    return nullptr;
  Py_RETURN_TRUE;
FASTCALL_END

// bind({entry point: address}, raise_status, Desc, AdamW)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *table, *raiser, *desc, *adamw;
  if (!PyArg_ParseTuple(args, "O!OO!O!", &PyDict_Type, &table, &raiser, &PyType_Type, &desc, &PyType_Type, &adamw))
    return nullptr;
  Library next;
#define QALORA_BIND(name)                                                    \
  {                                                                          \
    PyObject* v = PyDict_GetItemString(table, #name);                        \
    void* p = v ? PyLong_AsVoidPtr(v) : nullptr;                             \
    if (!p) {                                                                \
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);         \
      return nullptr;                                                        \
    }                                                                        \
    next.name = reinterpret_cast<decltype(next.name)>(p);                    \
  }
  QALORA_ENTRIES(QALORA_BIND)
  lib = next;
  for (auto [to, from] : {std::pair{&raise_status, raiser}, {&desc_type, desc}, {&adamw_type, adamw}}) {
    Py_INCREF(from);
    Py_XSETREF(*to, from);
  }
  bound = true;
  Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, METHOD(quantize), METHOD(forward), METHOD(forward_keep),
                         METHOD(backward), METHOD(backward_kept), METHOD(forward_deployed), METHOD(forward_factors16),
                         METHOD(forward_shared), METHOD(backward_shared), METHOD(swiglu_forward_wide),
                         METHOD(swiglu_backward_wide), METHOD(adamw_step), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Native form of the binding's calls (see api.py).", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
