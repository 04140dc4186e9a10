// The calls of binding.py on ordinary tensors, in native code.
//
// A call of the library costs the host two to six microseconds of kernel launches; checking seven
// tensors and marshalling the arguments in Python cost ten more, which is what a short call (a
// decoding step, a small forward) waited for.  Each function here takes the arguments of its
// namesake in binding.py, makes the same checks, allocates the same outputs and calls the C ABI on
// the current stream of Q's device.  It returns None for anything but the plain, valid call - a
// tensor subclass, an argument of another type, any check that fails - with nothing launched: the
// Python code then takes the call and raises the error, if it is one.  A call that the library
// rejects returns its status as an int.
//
// Host time per call: forward 15 -> 5.5 us, decoding step 16 -> 6 us, write step 11 -> 3.6 us.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/moda.h"

namespace {

// The library's entry points, as loaded by binding.py.
decltype(&moda_attn_fwd) g_fwd;
decltype(&moda_attn_bwd) g_bwd;
decltype(&moda_attn_bwd_workspace_bytes) g_bwd_bytes;
decltype(&moda_attn_decode) g_decode;
decltype(&moda_attn_decode_workspace_bytes) g_decode_bytes;
decltype(&moda_depth_append) g_append;

// An argument that must be a plain strided tensor in device memory, or None.
struct Arg {
  const at::Tensor* t = nullptr;  // null: None
  bool ok = true;
  explicit Arg(PyObject* o) {
    if (o == Py_None) return;
    ok = THPVariable_CheckExact(o);
    if (!ok) return;
    t = &THPVariable_Unpack(o);
    ok = t->is_cuda() && t->layout() == at::kStrided && t->has_storage();
  }
  explicit operator bool() const { return t != nullptr; }
  const at::Tensor* operator->() const { return t; }
  // of type `dt` on device `dev`, contiguous, of this shape (None passes)
  bool is(at::ScalarType dt, c10::Device dev, at::IntArrayRef shape) const {
    return t == nullptr || (t->scalar_type() == dt && t->device() == dev && t->sizes() == shape && t->is_contiguous());
  }
  void* ptr() const { return t == nullptr ? nullptr : t->data_ptr(); }
};

bool dtype_code(at::ScalarType t, moda_dtype& d) {
  if (t == at::kBFloat16) d = MODA_BF16;
  else if (t == at::kFloat) d = MODA_F32;
  else return false;
  return true;
}

// None -> `otherwise`; an int that fits 32 bits; false for anything else.
bool int_arg(PyObject* o, int64_t otherwise, int32_t& v) {
  int64_t x = otherwise;
  if (o != Py_None) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    x = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) return false;
  }
  v = static_cast<int32_t>(x);
  return x == v;
}
bool bool_arg(PyObject* o, int32_t& v) {
  v = o == Py_True;
  return o == Py_True || o == Py_False;
}
bool scale_arg(PyObject* o, float& v) {
  if (o != Py_None && !PyFloat_CheckExact(o)) return false;
  v = o == Py_None ? 0.f : static_cast<float>(PyFloat_AS_DOUBLE(o));
  return true;
}

// Fits the shape struct (sizes of a tensor dimension are 64-bit).
bool fits(const at::Tensor& t) {
  for (int64_t n : t.sizes())
    if (n > INT32_MAX) return false;
  return true;
}

void* stream_of(c10::Device dev) { return c10::hip::getCurrentHIPStream(dev.index()).stream(); }

PyObject* tensor_or_none(const at::Tensor& t) {
  if (t.defined()) return THPVariable_Wrap(t);
  Py_RETURN_NONE;
}
template <size_t N>
PyObject* tuple_of(const at::Tensor (&ts)[N]) {
  PyObject* r = PyTuple_New(N);
  if (!r) return nullptr;
  for (size_t i = 0; i < N; ++i) {
    PyObject* o = tensor_or_none(ts[i]);
    if (!o) {
      Py_DECREF(r);
      return nullptr;
    }
    PyTuple_SET_ITEM(r, i, o);
  }
  return r;
}

// Runs a call of the library without the interpreter's lock.
template <class F>
moda_status unlocked(F&& f) {
  PyThreadState* s = PyEval_SaveThread();
  const moda_status st = f();
  PyEval_RestoreThread(s);
  return st;
}

#define MODA_TAKES(n)       \
  HANDLE_TH_ERRORS          \
  if (nargs != (n) || !g_fwd) Py_RETURN_NONE

// Q, K, V and the depth tensors of a forward or backward call; fills `s`.
bool layer_args(const Arg& q, const Arg& k, const Arg& v, const Arg& kd, const Arg& vd, PyObject* count, PyObject* causal,
                PyObject* scale, moda_shape& s) {
  if (!q.ok || !k.ok || !v.ok || !kd.ok || !vd.ok || !q || !k || !v) return false;
  if (q->dim() != 4 || k->dim() != 4 || !fits(*q.t) || !fits(*k.t) || (kd && (kd->dim() != 5 || !fits(*kd.t)))) return false;
  const int64_t B = q->size(0), Hq = q->size(1), Hk = k->size(1), T = q->size(2), d = q->size(3);
  const int64_t La = kd ? kd->size(3) : 0;
  const auto dt = q->scalar_type();
  const auto dev = q->device();
  s.B = B; s.Hq = Hq; s.Hk = Hk; s.T = T; s.d = d; s.depth_alloc = La;
  return dtype_code(dt, s.dtype) && int_arg(count, La, s.depth_count) && bool_arg(causal, s.causal) &&
         scale_arg(scale, s.scale) && q.is(dt, dev, {B, Hq, T, d}) && k.is(dt, dev, {B, Hk, T, d}) &&
         v.is(dt, dev, {B, Hk, T, d}) && kd.is(dt, dev, {B, Hk, T, La, d}) && vd.is(dt, dev, {B, Hk, T, La, d});
}

// (Q, Kseq, Vseq, Kdepth, Vdepth, depth_count, causal, scale, out, lse)
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  MODA_TAKES(10);
  const Arg q(a[0]), k(a[1]), v(a[2]), kd(a[3]), vd(a[4]), out(a[8]), lse(a[9]);
  moda_shape s;
  if (!layer_args(q, k, v, kd, vd, a[5], a[6], a[7], s) || !out.ok || !lse.ok) Py_RETURN_NONE;
  const auto dev = q->device();
  if (!out.is(q->scalar_type(), dev, q->sizes()) || !lse.is(at::kFloat, dev, {s.B, s.Hq, s.T})) Py_RETURN_NONE;
  const at::Tensor r[2] = {out ? *out.t : at::empty_like(*q.t),
                           lse ? *lse.t : at::empty({s.B, s.Hq, s.T}, q->options().dtype(at::kFloat))};
  const c10::DeviceGuard guard(dev);
  void* const p[] = {q.ptr(), k.ptr(), v.ptr(), kd.ptr(), vd.ptr(), r[0].data_ptr(), r[1].data_ptr()};
  void* const st = stream_of(dev);
  const moda_status rc = unlocked([&] { return g_fwd(p[0], p[1], p[2], p[3], p[4], p[5], (float*)p[6], &s, st); });
  return rc == MODA_OK ? tuple_of(r) : PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

// (Q, Kseq, Vseq, Kdepth, Vdepth, O, LSE, dO, depth_count, causal, scale, workspace)
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  MODA_TAKES(12);
  const Arg q(a[0]), k(a[1]), v(a[2]), kd(a[3]), vd(a[4]), o(a[5]), lse(a[6]), g(a[7]), ws(a[11]);
  moda_shape s;
  if (!layer_args(q, k, v, kd, vd, a[8], a[9], a[10], s) || !o.ok || !lse.ok || !g.ok || !ws.ok || !o || !lse || !g)
    Py_RETURN_NONE;
  const auto dev = q->device();
  const auto dt = q->scalar_type();
  if (!o.is(dt, dev, q->sizes()) || !g.is(dt, dev, q->sizes()) || !lse.is(at::kFloat, dev, {s.B, s.Hq, s.T})) Py_RETURN_NONE;
  const at::Tensor r[5] = {at::empty_like(*q.t), at::empty_like(*k.t), at::empty_like(*v.t),
                           kd ? at::empty_like(*kd.t) : at::Tensor(), vd ? at::empty_like(*vd.t) : at::Tensor()};
  at::Tensor w;
  if (ws) w = *ws.t;
  else if (const size_t need = g_bwd_bytes(&s)) w = at::empty({(int64_t)need}, q->options().dtype(at::kByte));
  const c10::DeviceGuard guard(dev);
  auto ptr = [](const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; };
  void* const p[] = {q.ptr(), k.ptr(), v.ptr(), kd.ptr(), vd.ptr(), o.ptr(), lse.ptr(), g.ptr(),
                     ptr(r[0]), ptr(r[1]), ptr(r[2]), ptr(r[3]), ptr(r[4]), ptr(w)};
  const size_t ws_bytes = w.defined() ? (size_t)w.numel() * w.element_size() : 0;
  void* const st = stream_of(dev);
  const moda_status rc = unlocked([&] {
    return g_bwd(p[0], p[1], p[2], p[3], p[4], p[5], (const float*)p[6], p[7], p[8], p[9], p[10], p[11], p[12], p[13],
                 ws_bytes, &s, st);
  });
  return rc == MODA_OK ? tuple_of(r) : PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

// (Q, Kseq, Vseq, Kdepth, Vdepth, T, depth_count, scale, out, lse, workspace)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  MODA_TAKES(11);
  const Arg q(a[0]), k(a[1]), v(a[2]), kd(a[3]), vd(a[4]), out(a[8]), lse(a[9]), ws(a[10]);
  if (!q.ok || !k.ok || !v.ok || !kd.ok || !vd.ok || !out.ok || !lse.ok || !ws.ok || !q || !k || !v) Py_RETURN_NONE;
  if (q->dim() != 3 || k->dim() != 4 || !fits(*q.t) || !fits(*k.t) || (kd && (kd->dim() != 4 || !fits(*kd.t)))) Py_RETURN_NONE;
  const int64_t B = q->size(0), Hq = q->size(1), d = q->size(2), Hk = k->size(1), rows = k->size(2);
  const int64_t La = kd ? kd->size(2) : 0;
  const auto dt = q->scalar_type();
  const auto dev = q->device();
  moda_shape s;
  s.B = B; s.Hq = Hq; s.Hk = Hk; s.d = d; s.depth_alloc = La; s.causal = 1;
  if (!dtype_code(dt, s.dtype) || !int_arg(a[5], rows, s.T) || !int_arg(a[6], La, s.depth_count) || !scale_arg(a[7], s.scale))
    Py_RETURN_NONE;
  if (!q.is(dt, dev, {B, Hq, d}) || !k.is(dt, dev, {B, Hk, rows, d}) || !v.is(dt, dev, {B, Hk, rows, d}) ||
      !kd.is(dt, dev, {B, Hk, La, d}) || !vd.is(dt, dev, {B, Hk, La, d}) || !out.is(dt, dev, {B, Hq, d}) ||
      !lse.is(at::kFloat, dev, {B, Hq}))
    Py_RETURN_NONE;
  const at::Tensor r[2] = {out ? *out.t : at::empty_like(*q.t), lse ? *lse.t : at::empty({B, Hq}, q->options().dtype(at::kFloat))};
  at::Tensor w = ws ? *ws.t : at::Tensor();
  if (!ws) {
    const size_t need = g_decode_bytes(&s);
    w = at::empty({(int64_t)(need > 16 ? need : 16)}, q->options().dtype(at::kByte));
  }
  const c10::DeviceGuard guard(dev);
  void* const p[] = {q.ptr(), k.ptr(), v.ptr(), kd.ptr(), vd.ptr(), r[0].data_ptr(), r[1].data_ptr(), w.data_ptr()};
  const size_t ws_bytes = (size_t)w.numel() * w.element_size();
  void* const st = stream_of(dev);
  const moda_status rc = unlocked([&] {
    return g_decode(p[0], p[1], p[2], p[3], p[4], p[5], (float*)p[6], (int32_t)rows, p[7], ws_bytes, &s, st);
  });
  return rc == MODA_OK ? tuple_of(r) : PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

// (K, V, Kdepth, Vdepth, slot); returns True
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  MODA_TAKES(5);
  const Arg k(a[0]), v(a[1]), kd(a[2]), vd(a[3]);
  int32_t slot;
  if (!k.ok || !v.ok || !kd.ok || !vd.ok || !k || !v || !kd || !vd || a[4] == Py_None || !int_arg(a[4], 0, slot)) Py_RETURN_NONE;
  if (k->dim() != 4 || kd->dim() != 5 || !fits(*k.t) || !fits(*kd.t)) Py_RETURN_NONE;
  const int64_t B = k->size(0), Hk = k->size(1), T = k->size(2), d = k->size(3), La = kd->size(3);
  const auto dt = k->scalar_type();
  const auto dev = k->device();
  moda_shape s;
  s.B = B; s.Hq = Hk; s.Hk = Hk; s.T = T; s.d = d; s.depth_alloc = La; s.depth_count = 0; s.causal = 1; s.scale = 0.f;
  if (!dtype_code(dt, s.dtype) || !k.is(dt, dev, {B, Hk, T, d}) || !v.is(dt, dev, {B, Hk, T, d}) ||
      !kd.is(dt, dev, {B, Hk, T, La, d}) || !vd.is(dt, dev, {B, Hk, T, La, d}))
    Py_RETURN_NONE;
  const c10::DeviceGuard guard(dev);
  void* const p[] = {k.ptr(), v.ptr(), kd.ptr(), vd.ptr()};
  void* const st = stream_of(dev);
  const moda_status rc = unlocked([&] { return g_append(p[0], p[1], p[2], p[3], slot, &s, st); });
  if (rc == MODA_OK) Py_RETURN_TRUE;
  return PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

// (addresses of the six entry points, in the order of the variables above)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  if (nargs != 6) {
    PyErr_SetString(PyExc_TypeError, "init takes six addresses");
    return nullptr;
  }
  void* p[6];
  for (int i = 0; i < 6; ++i)
    if (!(p[i] = PyLong_AsVoidPtr(a[i]))) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
      return nullptr;
    }
  g_bwd = (decltype(g_bwd))p[1];
  g_bwd_bytes = (decltype(g_bwd_bytes))p[2];
  g_decode = (decltype(g_decode))p[3];
  g_decode_bytes = (decltype(g_decode_bytes))p[4];
  g_append = (decltype(g_append))p[5];
  g_fwd = (decltype(g_fwd))p[0];
  Py_RETURN_NONE;
}

#define MODA_METHOD(f) {#f, (PyCFunction)(void (*)())f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MODA_METHOD(init), MODA_METHOD(fwd), MODA_METHOD(bwd), MODA_METHOD(decode), MODA_METHOD(append),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "moda_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_moda_torch(void) { return PyModule_Create(&module); }
