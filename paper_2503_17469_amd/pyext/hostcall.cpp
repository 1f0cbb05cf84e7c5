// Argument marshalling of the calls a training loop makes every step (controller, step, updates) through the CPython API.
//
// With a net of a few kernels the host work per step is what counts: through ctypes the controller's two calls and the
// step cost 9 us of it on one core, of which the library's own work is a fraction.  The functions here take the same
// arguments as binding.py's, which remain the interface; the library's entry points come in as addresses (init), so
// nothing is linked.  The GIL is released during the calls, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>
#include <memory>
#include <new>

#include "../../include/omnistep.h"

namespace {

typedef int (*SetThroughputsFn)(void*, const uint64_t*);
typedef int (*RunFn)(void*, int32_t*, int32_t*);
typedef int (*StepFn)(void*, void*, void*, const void*, const void*, const int32_t*, const int32_t*, int32_t, float, void*,
                      void*, void*, uint32_t);
typedef int (*SgdFn)(void*, void*, const void*, size_t, size_t, const int32_t*, int32_t, float, void*);
typedef int (*MomentumFn)(void*, void*, void*, const void*, size_t, size_t, const int32_t*, int32_t, float, float, float,
                          void*);
typedef int (*AspFn)(void*, void*, const void*, const void*, size_t, float, int32_t, int32_t, int32_t);

SetThroughputsFn g_set = nullptr;
RunFn g_run = nullptr;
StepFn g_step = nullptr;
SgdFn g_sgd = nullptr;
MomentumFn g_momentum = nullptr;
AspFn g_asp = nullptr;
PyObject *g_value = nullptr, *g_data_ptr = nullptr;   // interned attribute names

// A ctypes c_void_p handle, or an address.
bool handle(PyObject* o, void** out) {
  if (o == Py_None) { *out = nullptr; return true; }
  if (PyLong_Check(o)) { *out = PyLong_AsVoidPtr(o); return !PyErr_Occurred(); }
  PyObject* v = PyObject_GetAttr(o, g_value);
  if (!v) return false;
  const bool ok = v == Py_None || PyLong_Check(v);
  *out = v == Py_None ? nullptr : ok ? PyLong_AsVoidPtr(v) : nullptr;
  Py_DECREF(v);
  if (!ok) PyErr_SetString(PyExc_TypeError, "a handle's value is no address");
  return ok && !PyErr_Occurred();
}

// The address of a tensor's data; None is a null pointer.
bool pointer(PyObject* o, void** out) {
  if (o == Py_None) { *out = nullptr; return true; }
  PyObject* v = PyObject_CallMethodNoArgs(o, g_data_ptr);
  if (!v) return false;
  *out = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

// The low 64 bits of an integer, or of whatever int() makes of the value.
bool integer(PyObject* o, uint64_t* out) {
  if (PyLong_Check(o)) {
    *out = PyLong_AsUnsignedLongLongMask(o);
  } else {
    PyObject* v = PyNumber_Long(o);
    if (!v) return false;
    *out = PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
  }
  return !PyErr_Occurred();
}

// A sequence of integers as an array with zeros behind it, up to OMNI_MAX_WORKERS + 1 entries at least: a caller's list that is
// shorter than the number of workers the library knows of reads as zeros (which it refuses).  Short ones (every number of
// workers) stay on the stack.
template <typename T>
class Array {
 public:
  bool take(PyObject* seq, Py_ssize_t at_least = 0) {
    PyObject* fast = PySequence_Fast(seq, "a sequence of integers is wanted");
    if (!fast) return false;
    n_ = PySequence_Fast_GET_SIZE(fast);
    bool ok = room(n_ > at_least ? n_ : at_least);
    for (Py_ssize_t i = 0; i < n_ && ok; ++i) {
      uint64_t v = 0;
      ok = integer(PySequence_Fast_GET_ITEM(fast, i), &v);
      p_[i] = (T)v;
    }
    Py_DECREF(fast);
    return ok;
  }
  bool room(Py_ssize_t n) {
    if (n > kFixed) {
      more_.reset(new (std::nothrow) T[n]);
      p_ = more_.get();
      if (!p_) { PyErr_NoMemory(); return false; }
    }
    std::memset(p_, 0, (n > kFixed ? n : kFixed) * sizeof(T));
    return true;
  }
  T* data() { return p_; }
  Py_ssize_t size() const { return n_; }

 private:
  static constexpr Py_ssize_t kFixed = OMNI_MAX_WORKERS + 1;
  T fixed_[kFixed];
  std::unique_ptr<T[]> more_;
  T* p_ = fixed_;
  Py_ssize_t n_ = 0;
};

PyObject* list_of(const int32_t* v, Py_ssize_t n) {
  PyObject* l = PyList_New(n);
  for (Py_ssize_t i = 0; l && i < n; ++i) {
    PyObject* o = PyLong_FromLong(v[i]);
    if (!o) { Py_DECREF(l); return nullptr; }
    PyList_SET_ITEM(l, i, o);
  }
  return l;
}

bool arity(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments given, %zd wanted", n, want);
  return false;
}
bool real(PyObject* o, float* out) {
  const double d = PyFloat_AsDouble(o);
  *out = (float)d;
  return !(d == -1.0 && PyErr_Occurred());
}
bool size_of(PyObject* o, size_t* out) {
  uint64_t v = 0;
  if (!integer(o, &v)) return false;
  *out = (size_t)v;
  return true;
}

PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arity(n, 6)) return nullptr;
  void* p[6];
  for (int i = 0; i < 6; ++i)
    if (!handle(a[i], &p[i])) return nullptr;
  g_set = reinterpret_cast<SetThroughputsFn>(p[0]);
  g_run = reinterpret_cast<RunFn>(p[1]);
  g_step = reinterpret_cast<StepFn>(p[2]);
  g_sgd = reinterpret_cast<SgdFn>(p[3]);
  g_momentum = reinterpret_cast<MomentumFn>(p[4]);
  g_asp = reinterpret_cast<AspFn>(p[5]);
  Py_RETURN_NONE;
}

// (ctl, T) -> rc
PyObject* ctl_set_throughputs(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* ctl;
  Array<uint64_t> T;
  if (!arity(n, 2) || !handle(a[0], &ctl) || !T.take(a[1])) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_set(ctl, T.data());
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (ctl, K) -> rc, or (b, off) where rc is 0
PyObject* ctl_run(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* ctl;
  uint64_t K = 0;
  if (!arity(n, 2) || !handle(a[0], &ctl) || !integer(a[1], &K)) return nullptr;
  if (K > (1u << 20)) {
    PyErr_SetString(PyExc_ValueError, "K is not a number of workers");
    return nullptr;
  }
  Array<int32_t> b, off;
  if (!b.room((Py_ssize_t)K) || !off.room((Py_ssize_t)K + 1)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_run(ctl, b.data(), off.data());
  Py_END_ALLOW_THREADS
  if (rc != 0) return PyLong_FromLong(rc);
  PyObject *lb = list_of(b.data(), (Py_ssize_t)K), *lo = list_of(off.data(), (Py_ssize_t)K + 1);
  if (!lb || !lo) { Py_XDECREF(lb); Py_XDECREF(lo); return nullptr; }
  return Py_BuildValue("(NN)", lb, lo);
}

// (net, stream, params, x, labels, off, b, lr, workspace, loss_per_worker, loss, flags) -> rc
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *net, *stream, *params, *x, *labels, *ws, *lpw, *loss;
  Array<int32_t> off, b;
  float lr;
  uint64_t flags = 0;
  if (!arity(n, 12) || !handle(a[0], &net) || !handle(a[1], &stream) || !pointer(a[2], &params) || !pointer(a[3], &x) ||
      !pointer(a[4], &labels) || !b.take(a[6]) || !off.take(a[5], b.size() + 1) || !real(a[7], &lr) || !pointer(a[8], &ws) ||
      !pointer(a[9], &lpw) || !pointer(a[10], &loss) || !integer(a[11], &flags))
    return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_step(net, stream, params, x, labels, off.data(), b.data(), (int32_t)b.size(), lr, ws, lpw, loss, (uint32_t)flags);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (stream, params, grads, stride, P, b, lr, shadow) -> rc
PyObject* weighted_sgd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *stream, *params, *grads, *shadow;
  size_t stride, P;
  Array<int32_t> b;
  float lr;
  if (!arity(n, 8) || !handle(a[0], &stream) || !pointer(a[1], &params) || !pointer(a[2], &grads) || !size_of(a[3], &stride) ||
      !size_of(a[4], &P) || !b.take(a[5]) || !real(a[6], &lr) || !pointer(a[7], &shadow))
    return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_sgd(stream, params, grads, stride, P, b.data(), (int32_t)b.size(), lr, shadow);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (stream, params, velocity, grads, stride, P, b, lr, momentum, weight_decay, shadow) -> rc
PyObject* weighted_sgd_momentum(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *stream, *params, *velocity, *grads, *shadow;
  size_t stride, P;
  Array<int32_t> b;
  float lr, momentum, decay;
  if (!arity(n, 11) || !handle(a[0], &stream) || !pointer(a[1], &params) || !pointer(a[2], &velocity) ||
      !pointer(a[3], &grads) || !size_of(a[4], &stride) || !size_of(a[5], &P) || !b.take(a[6]) || !real(a[7], &lr) ||
      !real(a[8], &momentum) || !real(a[9], &decay) || !pointer(a[10], &shadow))
    return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_momentum(stream, params, velocity, grads, stride, P, b.data(), (int32_t)b.size(), lr, momentum, decay, shadow);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (stream, dst, base, grad, P, lr, b_k, B, lr_scaling) -> rc; grad: a tensor, or an address
PyObject* asp_update(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *stream, *dst, *base, *grad;
  size_t P;
  float lr;
  uint64_t b = 0, B = 0, scaling = 0;
  if (!arity(n, 9) || !handle(a[0], &stream) || !pointer(a[1], &dst) || !pointer(a[2], &base) ||
      !(PyLong_Check(a[3]) ? handle(a[3], &grad) : pointer(a[3], &grad)) || !size_of(a[4], &P) || !real(a[5], &lr) ||
      !integer(a[6], &b) || !integer(a[7], &B) || !integer(a[8], &scaling))
    return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_asp(stream, dst, base, grad, P, lr, (int32_t)b, (int32_t)B, (int32_t)scaling);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

#define OMNI_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {OMNI_METHOD(init), OMNI_METHOD(ctl_set_throughputs), OMNI_METHOD(ctl_run), OMNI_METHOD(step),
                         OMNI_METHOD(weighted_sgd), OMNI_METHOD(weighted_sgd_momentum), OMNI_METHOD(asp_update),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hostcall", "Argument marshalling for binding.py.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__hostcall() {
  g_value = PyUnicode_InternFromString("value");
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  if (!g_value || !g_data_ptr) return nullptr;
  return PyModule_Create(&module);
}
