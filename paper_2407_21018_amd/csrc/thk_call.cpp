// The calls a serving program issues once per layer and token, from Python without ctypes: tensors checked
// and unpacked natively, one crossing per call.
//
// What bounds such a call on short contexts is the host: through ctypes and Python-level tensor methods a
// decode call took 5.7 us to issue and 32 layers of append and decode 366, of which a launch is 2.5; here they take 3.7 and
// 261, less than the kernels (310), which the calls used to wait for: 346 -> 321 us a token.  A call is taken here only in its
// plain form (exact torch tensors, contiguous and large enough, the current stream or a handle); anything
// else is left to the Python code, which has the checks that raise.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "thk.h"

namespace {

constexpr long kNotTaken = -1;   // the Python code takes the call

decltype(&thk_decode_attn) f_decode = nullptr;
decltype(&thk_decode_attn_kv) f_decode_kv = nullptr;
decltype(&thk_tail_append) f_append = nullptr;
decltype(&thk_prune) f_prune = nullptr;
PyTypeObject *g_shape = nullptr;   // thk_shape of the Python code
PyObject *g_get_stream = nullptr, *g_get_device = nullptr;   // torch's raw getters, once the runtime is up

// The arguments of one call; ok turns false at the first one that is not in the plain form.
struct Args {
  bool ok = true;
  const thk_shape *shape = nullptr;
  Py_buffer view{};

  explicit Args(PyObject *s) {
    // (bytes of the same length are no shape, as for ctypes)
    if (g_shape == nullptr || !PyObject_TypeCheck(s, g_shape)) {
      ok = false;
      return;
    }
    if (PyObject_GetBuffer(s, &view, PyBUF_SIMPLE) != 0) {
      PyErr_Clear();
      ok = false;
      return;
    }
    ok = view.len == (Py_ssize_t)sizeof(thk_shape);
    shape = (const thk_shape *)view.buf;
  }
  ~Args() {
    if (view.obj != nullptr) PyBuffer_Release(&view);
  }
  static bool plain(PyObject *x) { return THPVariable_CheckExact(x); }
  // address of a tensor of at least n elements
  void *tensor(PyObject *x, int64_t n) {
    if (!ok || !plain(x)) return ok = false, nullptr;
    const at::Tensor &t = THPVariable_Unpack(x);
    if (t.layout() != at::kStrided || t.numel() < n || !t.is_contiguous()) return ok = false, nullptr;
    return t.data_ptr();
  }
  // ... or of None
  void *tensor_if(PyObject *x, int64_t n) {
    if (x == Py_None) return nullptr;
    return tensor(x, n);
  }
  void *workspace(PyObject *x, size_t &bytes) {
    bytes = 0;
    if (x == Py_None) return nullptr;
    if (!ok || !plain(x)) return ok = false, nullptr;
    const at::Tensor &t = THPVariable_Unpack(x);
    if (t.layout() != at::kStrided) return ok = false, nullptr;
    bytes = (size_t)t.numel() * t.element_size();
    return t.data_ptr();
  }
  int32_t integer(PyObject *x) {
    if (!ok || !PyLong_CheckExact(x)) return ok = false, 0;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(x, &overflow);
    if (overflow != 0 || v < INT32_MIN || v > INT32_MAX) return ok = false, 0;
    return (int32_t)v;
  }
  void *stream(PyObject *x) {
    if (!ok) return nullptr;
    PyObject *h = nullptr;
    if (x == Py_None) {
      if (g_get_stream == nullptr) return ok = false, nullptr;
      PyObject *dev = PyObject_CallNoArgs(g_get_device);
      h = dev != nullptr ? PyObject_CallOneArg(g_get_stream, dev) : nullptr;
      Py_XDECREF(dev);
    } else if (PyLong_CheckExact(x)) {
      h = Py_NewRef(x);
    }
    if (h == nullptr) return PyErr_Clear(), ok = false, nullptr;
    void *p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (PyErr_Occurred()) return PyErr_Clear(), ok = false, nullptr;
    return p;
  }
  // The product of a tensor's sizes.  A shape whose product does not fit 64 bits (a capacity that was never set)
  // would wrap to a size that every tensor has; it is left to the Python code, which counts without a bound.
  template <class... I>
  int64_t count(I... sizes) {
    int64_t n = 1;
    for (const int64_t f : {(int64_t)sizes...}) ok = !__builtin_mul_overflow(n, f, &n) && ok;
    return n;
  }
  int64_t less(int64_t a, int64_t b) {
    int64_t n = 0;
    ok = !__builtin_sub_overflow(a, b, &n) && ok;
    return n;
  }
  int64_t layers_units() { return count(shape->L, shape->B, shape->N_kv); }
  int64_t heads() { return count(shape->L, shape->B, shape->N_q); }
  int64_t ld() const { return shape->ld_keep ? shape->ld_keep : shape->T; }
  int64_t rows(int64_t used) { return count(layers_units(), shape->S_cap ? shape->S_cap : used); }
};

// A call without the interpreter lock (a launch may have to wait for room in the queue), which is taken again also
// when f throws.
struct Unlocked {
  PyThreadState *state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class F>
PyObject *issue(F f) {
  thk_status st;
  {
    Unlocked unlocked;
    st = f();
  }
  return PyLong_FromLong((long)st);
}
PyObject *not_taken() { return PyLong_FromLong(kNotTaken); }

// An exception (of a tensor without storage) is the Python code's to raise.
template <class F>
PyObject *guarded(F f) {
  try {
    return f();
  } catch (...) {
    return not_taken();
  }
}

// (shape, q, k_pruned, idx, v, k_tail, v_tail, s_tail, s_tail_cap, out, ws, stream)
PyObject *decode_attn(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 12 || f_decode == nullptr) return not_taken();
  return guarded([&]() -> PyObject * {
    Args x(a[0]);
    if (!x.ok) return not_taken();
    const thk_shape *s = x.shape;
    const int64_t U = x.layers_units(), hn = x.count(x.heads(), s->D), rows = x.rows(s->S);
    const int32_t s_tail = x.integer(a[7]), cap = x.integer(a[8]);
    void *q = x.tensor(a[1], hn), *kp = x.tensor(a[2], x.count(rows, x.ld())), *idx = x.tensor(a[3], x.count(U, s->T)), *v = x.tensor(a[4], x.count(rows, s->D));
    const int64_t tail = s_tail > 0 ? x.count(U, cap, s->D) : 0;
    void *kt = x.tensor_if(a[5], tail), *vt = x.tensor_if(a[6], tail), *out = x.tensor(a[9], hn);
    size_t bytes = 0;
    void *ws = x.workspace(a[10], bytes), *st = x.stream(a[11]);
    if (!x.ok) return not_taken();
    return issue([&] { return f_decode(s, q, kp, (const int16_t *)idx, v, kt, vt, s_tail, cap, out, ws, bytes, st); });
  });
}

// (shape, q, k_pruned, idx, v_pruned, idx_v, T_v, ld_v, k_tail, v_tail, s_tail, s_tail_cap, out, ws, stream)
PyObject *decode_attn_kv(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 15 || f_decode_kv == nullptr) return not_taken();
  return guarded([&]() -> PyObject * {
    Args x(a[0]);
    if (!x.ok) return not_taken();
    const thk_shape *s = x.shape;
    const int64_t U = x.layers_units(), hn = x.count(x.heads(), s->D), rows = x.rows(s->S);
    const int32_t T_v = x.integer(a[6]), ld_v = x.integer(a[7]), s_tail = x.integer(a[10]), cap = x.integer(a[11]);
    if (T_v < 0 || ld_v < 0) return not_taken();
    void *q = x.tensor(a[1], hn), *kp = x.tensor(a[2], x.count(rows, x.ld())), *idx = x.tensor(a[3], x.count(U, s->T));
    void *v = x.tensor(a[4], x.count(rows, ld_v)), *idxv = x.tensor(a[5], x.count(U, T_v));
    const int64_t tail = s_tail > 0 ? x.count(U, cap, s->D) : 0;
    void *kt = x.tensor_if(a[8], tail), *vt = x.tensor_if(a[9], tail), *out = x.tensor(a[12], hn);
    size_t bytes = 0;
    void *ws = x.workspace(a[13], bytes), *st = x.stream(a[14]);
    if (!x.ok) return not_taken();
    return issue([&] {
      return f_decode_kv(s, q, kp, (const int16_t *)idx, v, (const int16_t *)idxv, T_v, ld_v, kt, vt, s_tail, cap, out, ws, bytes, st);
    });
  });
}

// (shape, k_new, v_new, k_tail, v_tail, s_tail, s_tail_cap, stream)
PyObject *tail_append(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 8 || f_append == nullptr) return not_taken();
  return guarded([&]() -> PyObject * {
    Args x(a[0]);
    if (!x.ok) return not_taken();
    const thk_shape *s = x.shape;
    const int32_t s_tail = x.integer(a[5]), cap = x.integer(a[6]);
    const int64_t un = x.count(x.layers_units(), s->D), tail = x.count(un, cap);
    void *kn = x.tensor(a[1], un), *vn = x.tensor(a[2], un), *kt = x.tensor(a[3], tail), *vt = x.tensor(a[4], tail);
    void *st = x.stream(a[7]);
    if (!x.ok) return not_taken();
    return issue([&] { return f_append(s, kn, vn, kt, vt, s_tail, cap, st); });
  });
}

// (shape, q_obs, k, score, idx, k_pruned, ws, stream)
PyObject *prune(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 8 || f_prune == nullptr) return not_taken();
  return guarded([&]() -> PyObject * {
    Args x(a[0]);
    if (!x.ok) return not_taken();
    const thk_shape *s = x.shape;
    const int64_t U = x.layers_units();
    void *q = x.tensor(a[1], x.count(x.heads(), s->S_obs, s->D)), *k = x.tensor(a[2], x.count(U, s->S, s->D));
    void *sc = x.tensor_if(a[3], x.count(U, s->D)), *idx = x.tensor(a[4], x.count(U, s->T));
    void *kp = x.tensor(a[5], x.count(x.rows(x.less(s->S, s->S_recent)), x.ld()));
    size_t bytes = 0;
    void *ws = x.workspace(a[6], bytes), *st = x.stream(a[7]);
    if (!x.ok) return not_taken();
    return issue([&] { return f_prune(s, q, k, (float *)sc, (int16_t *)idx, kp, ws, bytes, st); });
  });
}

// bind(decode_attn, decode_attn_kv, tail_append, prune, thk_shape): the library's entry points, as addresses, and
// the type of a shape
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 5 || !PyType_Check(a[4])) return PyErr_SetString(PyExc_TypeError, "bind: four addresses and a type"), nullptr;
  void *p[4];
  for (int i = 0; i < 4; ++i) p[i] = PyLong_AsVoidPtr(a[i]);
  if (PyErr_Occurred()) return nullptr;
  f_decode = (decltype(f_decode))p[0];
  f_decode_kv = (decltype(f_decode_kv))p[1];
  f_append = (decltype(f_append))p[2];
  f_prune = (decltype(f_prune))p[3];
  PyTypeObject *old = g_shape;
  g_shape = (PyTypeObject *)Py_NewRef(a[4]);
  Py_XDECREF((PyObject *)old);
  Py_RETURN_NONE;
}

// stream_getters(get_stream, get_device), or (None, None) to forget them
PyObject *stream_getters(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 2) return PyErr_SetString(PyExc_TypeError, "stream_getters: two callables or None"), nullptr;
  const bool set = a[0] != Py_None && a[1] != Py_None;
  PyObject *old_s = g_get_stream, *old_d = g_get_device;
  g_get_stream = set ? Py_NewRef(a[0]) : nullptr;
  g_get_device = set ? Py_NewRef(a[1]) : nullptr;
  Py_XDECREF(old_s);
  Py_XDECREF(old_d);
  Py_RETURN_NONE;
}

#define THK_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {THK_METHOD(decode_attn), THK_METHOD(decode_attn_kv), THK_METHOD(tail_append), THK_METHOD(prune),
                         THK_METHOD(bind), THK_METHOD(stream_getters), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_thk_call", "Native issue of the per-token calls of libthk.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__thk_call(void) { return PyModule_Create(&module); }
