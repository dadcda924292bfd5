// Argument marshalling of the runtime entry points for the Python binding
// (ot.py): tensors checked and turned into device pointers natively.
//
// The same checks in Python take 0.3-0.5 us a tensor and ctypes another 0.6 us
// a call: of the 7.3 us of an ot_qlinear call, where a launch takes 3.0, 0.7
// are left here.  Each function here takes the C entry point's address (of the library
// that ot.py has loaded) and the binding's arguments, and returns the
// ot_status, or None where any argument is not exactly what it expects
// (another type, dtype, device, layout or shape): ot.py then runs its own
// checks, which name the fault or convert the argument.
#include <torch/csrc/autograd/python_variable.h>

#include <Python.h>
#include <stdint.h>

#include "../../include/ot.h"

namespace {

// ot.py's function for the current stream's handle.
PyObject *g_current_stream = nullptr;

// One call's arguments; ok turns false at the first that does not fit.
struct Args {
  PyObject *const *a;
  bool ok = true;

  // Plain tensors (and parameters) only, by their type: an object can claim to
  // be a tensor (its __class__) without a tensor's memory, and a subclass may
  // answer for itself, which only the Python checks ask it to.
  const at::Tensor *tensor(int i, at::ScalarType type) {
    if (!ok || !THPVariable_CheckExact(a[i])) return fail();
    const at::Tensor &t = THPVariable_Unpack(a[i]);
    if (t.scalar_type() != type || !t.is_cuda() || !t.is_contiguous()) return fail();
    return &t;
  }
  // A matrix that defines its two sizes.
  template <class T>
  const T *matrix(int i, at::ScalarType type, int64_t &rows, int64_t &cols) {
    const at::Tensor *t = tensor(i, type);
    if (t == nullptr || t->dim() != 2) return static_cast<const T *>(miss());
    rows = t->size(0);
    cols = t->size(1);
    return static_cast<const T *>(t->data_ptr());
  }
  // A matrix or vector of known sizes; none: None is nullptr.
  template <class T>
  T *sized(int i, at::ScalarType type, int64_t rows, int64_t cols, bool none = false) {
    if (ok && none && a[i] == Py_None) return nullptr;
    const at::Tensor *t = tensor(i, type);
    if (t == nullptr || t->dim() != 2 || t->size(0) != rows || t->size(1) != cols)
      return static_cast<T *>(miss());
    return static_cast<T *>(t->data_ptr());
  }
  template <class T>
  T *vec(int i, at::ScalarType type, int64_t n) {
    const at::Tensor *t = tensor(i, type);
    if (t == nullptr || t->dim() != 1 || t->size(0) != n) return static_cast<T *>(miss());
    return static_cast<T *>(t->data_ptr());
  }
  // Optional scratch of at least `need()` bytes.
  template <class F>
  void *scratch(int i, F need) {
    if (ok && a[i] == Py_None) return nullptr;
    const at::Tensor *t = tensor(i, at::kByte);
    if (t == nullptr || t->numel() < (int64_t)need()) return miss();
    return t->data_ptr();
  }
  int64_t integer(int i) {
    if (!ok || !PyLong_CheckExact(a[i])) {
      ok = false;
      return 0;
    }
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(a[i], &overflow);
    if (overflow != 0) ok = false;
    return v;
  }
  int bits(int i) {
    const int64_t v = integer(i);
    if (v < INT32_MIN || v > INT32_MAX) ok = false;
    return (int)v;
  }
  // The library call, without the interpreter lock (a launch can wait for room
  // in its queue).
  template <class F>
  int call(F f) {
    if (!ok) return 0;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = (int)f();
    Py_END_ALLOW_THREADS
    return rc;
  }
  // A stream handle, or None for the current stream (looked up only once
  // everything else fits: the call needs a GPU).
  void *stream(int i) {
    if (!ok || a[i] != Py_None) return address<void *>(i);
    PyObject *r = g_current_stream ? PyObject_CallObject(g_current_stream, nullptr) : nullptr;
    if (r == nullptr) {
      PyErr_Clear();
      return miss();
    }
    void *p = PyLong_CheckExact(r) ? PyLong_AsVoidPtr(r) : miss();
    Py_DECREF(r);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      return miss();
    }
    return p;
  }
  // An address as an unsigned integer.
  template <class F>
  F address(int i) {
    if (!ok || !PyLong_CheckExact(a[i])) {
      ok = false;
      return F{};
    }
    void *p = PyLong_AsVoidPtr(a[i]);
    if (p == nullptr && PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return reinterpret_cast<F>(p);
  }

 private:
  const at::Tensor *fail() {
    ok = false;
    return nullptr;
  }
  void *miss() {
    ok = false;
    return nullptr;
  }
};

constexpr at::ScalarType kCode = at::kChar, kF32 = at::kFloat, kF16 = at::kHalf, kI32 = at::kInt;

// Runs body(args) -> ot_status; None where an argument did not fit.
template <class Body>
PyObject *run(PyObject *const *a, Py_ssize_t n, Py_ssize_t want, Body body) {
  if (n != want) Py_RETURN_NONE;
  Args args{a};
  int rc = 0;
  try {
    rc = body(args);
  } catch (...) {  // a tensor without storage (under tracing, say) or one that raised
    args.ok = false;
    PyErr_Clear();  // ot.py asks the tensor again and lets its error through
  }
  if (!args.ok) Py_RETURN_NONE;
  return PyLong_FromLong(rc);
}

// (fn, x, a_bits, z, inv_s, Xq, stream)
PyObject *quantize_act(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 7, [](Args &g) -> int {
    int64_t M, K;
    auto fn = g.address<decltype(&ot_quantize_act)>(0);
    auto *x = g.matrix<uint16_t>(1, kF16, M, K);
    const int bits = g.bits(2);
    auto *z = g.vec<float>(3, kF32, K), *is = g.vec<float>(4, kF32, K);
    auto *q = g.sized<int8_t>(5, kCode, M, K);
    auto *st = g.stream(6);
    return g.call([&] { return fn(x, M, K, bits, z, is, q, st); });
  });
}

// (fn, x, a_bits, Xq, sX, stream)
PyObject *quantize_act_per_token(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 6, [](Args &g) -> int {
    int64_t M, K;
    auto fn = g.address<decltype(&ot_quantize_act_per_token)>(0);
    auto *x = g.matrix<uint16_t>(1, kF16, M, K);
    const int bits = g.bits(2);
    auto *q = g.sized<int8_t>(3, kCode, M, K);
    auto *s = g.vec<float>(4, kF32, M);
    auto *st = g.stream(5);
    return g.call([&] { return fn(x, M, K, bits, q, s, st); });
  });
}

// (fn, h, gamma, beta, eps, a_bits, z, inv_s, Xq, stream)
PyObject *ln_quantize_act(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 10, [](Args &g) -> int {
    int64_t M, K;
    auto fn = g.address<decltype(&ot_ln_quantize_act)>(0);
    auto *h = g.matrix<uint16_t>(1, kF16, M, K);
    auto *ga = g.vec<uint16_t>(2, kF16, K), *be = g.vec<uint16_t>(3, kF16, K);
    if (g.ok && !PyFloat_CheckExact(g.a[4])) g.ok = false;
    const float eps = g.ok ? (float)PyFloat_AS_DOUBLE(g.a[4]) : 0.f;
    const int bits = g.bits(5);
    auto *z = g.vec<float>(6, kF32, K), *is = g.vec<float>(7, kF32, K);
    auto *q = g.sized<int8_t>(8, kCode, M, K);
    auto *st = g.stream(9);
    return g.call([&] { return fn(h, M, K, ga, be, eps, bits, z, is, q, st); });
  });
}

using WsFn = size_t (*)(int64_t, int64_t, int64_t);

// (fn, ws_size, Xq, Wq, sW, bprime, a_bits, w_bits, Y, acc_out, workspace, stream)
PyObject *qlinear(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 12, [](Args &g) -> int {
    int64_t M, K, N, K2;
    auto fn = g.address<decltype(&ot_qlinear)>(0);
    auto ws_size = g.address<WsFn>(1);
    auto *x = g.matrix<int8_t>(2, kCode, M, K);
    auto *w = g.matrix<int8_t>(3, kCode, N, K2);
    if (g.ok && K2 != K) g.ok = false;
    auto *s = g.vec<float>(4, kF32, N), *b = g.vec<float>(5, kF32, N);
    const int ab = g.bits(6), wb = g.bits(7);
    auto *y = g.sized<uint16_t>(8, kF16, M, N);
    auto *acc = g.sized<int32_t>(9, kI32, M, N, true);
    auto *ws = g.scratch(10, [&] { return ws_size(M, N, K); });
    auto *st = g.stream(11);
    return g.call([&] { return fn(x, w, s, b, M, N, K, ab, wb, y, acc, ws, st); });
  });
}

// (fn, Xq, Wq, sW, bprime, a_bits, w_bits, Y, acc_out, stream)
PyObject *qlinear_noalloc(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 10, [](Args &g) -> int {
    int64_t M, K, N, K2;
    auto fn = g.address<decltype(&ot_qlinear_noalloc)>(0);
    auto *x = g.matrix<int8_t>(1, kCode, M, K);
    auto *w = g.matrix<int8_t>(2, kCode, N, K2);
    if (g.ok && K2 != K) g.ok = false;
    auto *s = g.vec<float>(3, kF32, N), *b = g.vec<float>(4, kF32, N);
    const int ab = g.bits(5), wb = g.bits(6);
    auto *y = g.sized<uint16_t>(7, kF16, M, N);
    auto *acc = g.sized<int32_t>(8, kI32, M, N, true);
    auto *st = g.stream(9);
    return g.call([&] { return fn(x, w, s, b, M, N, K, ab, wb, y, acc, st); });
  });
}

// (fn, ws_size, packed_size, Xq, Wp, N, sW, bprime, a_bits, w_bits, Y, acc_out,
//  workspace, stream)
PyObject *qlinear_packed(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 14, [](Args &g) -> int {
    int64_t M, K;
    auto fn = g.address<decltype(&ot_qlinear_packed)>(0);
    auto ws_size = g.address<WsFn>(1);
    auto packed = g.address<decltype(&ot_packed_weights_size)>(2);
    auto *x = g.matrix<int8_t>(3, kCode, M, K);
    const int64_t N = g.integer(5);
    auto *w = g.ok ? g.vec<int8_t>(4, kCode, (int64_t)packed(N, K)) : nullptr;
    auto *s = g.vec<float>(6, kF32, N), *b = g.vec<float>(7, kF32, N);
    const int ab = g.bits(8), wb = g.bits(9);
    auto *y = g.sized<uint16_t>(10, kF16, M, N);
    auto *acc = g.sized<int32_t>(11, kI32, M, N, true);
    auto *ws = g.scratch(12, [&] { return ws_size(M, N, K); });
    auto *st = g.stream(13);
    return g.call([&] { return fn(x, w, s, b, M, N, K, ab, wb, y, acc, ws, st); });
  });
}

// (fn, ws_size, Xq, Wq, sX, sW, bprime, a_bits, w_bits, Y, acc_out, workspace, stream)
PyObject *qlinear_per_token(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 13, [](Args &g) -> int {
    int64_t M, K, N, K2;
    auto fn = g.address<decltype(&ot_qlinear_per_token)>(0);
    auto ws_size = g.address<WsFn>(1);
    auto *x = g.matrix<int8_t>(2, kCode, M, K);
    auto *w = g.matrix<int8_t>(3, kCode, N, K2);
    if (g.ok && K2 != K) g.ok = false;
    auto *sx = g.vec<float>(4, kF32, M);
    auto *s = g.vec<float>(5, kF32, N), *b = g.vec<float>(6, kF32, N);
    const int ab = g.bits(7), wb = g.bits(8);
    auto *y = g.sized<uint16_t>(9, kF16, M, N);
    auto *acc = g.sized<int32_t>(10, kI32, M, N, true);
    auto *ws = g.scratch(11, [&] { return ws_size(M, N, K); });
    auto *st = g.stream(12);
    return g.call([&] { return fn(x, w, sx, s, b, M, N, K, ab, wb, y, acc, ws, st); });
  });
}

// (fn, ws_size, Xq, Wq, sW, zW, bprime, a_bits, w_bits, Y, acc_out, workspace, stream)
PyObject *qlinear_asym(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return run(a, n, 13, [](Args &g) -> int {
    int64_t M, K, N, K2;
    auto fn = g.address<decltype(&ot_qlinear_asym)>(0);
    auto ws_size = g.address<WsFn>(1);
    auto *x = g.matrix<int8_t>(2, kCode, M, K);
    auto *w = g.matrix<int8_t>(3, kCode, N, K2);
    if (g.ok && K2 != K) g.ok = false;
    auto *s = g.vec<float>(4, kF32, N);
    auto *zw = g.vec<int32_t>(5, kI32, N);
    auto *b = g.vec<float>(6, kF32, N);
    const int ab = g.bits(7), wb = g.bits(8);
    auto *y = g.sized<uint16_t>(9, kF16, M, N);
    auto *acc = g.sized<int32_t>(10, kI32, M, N, true);
    auto *ws = g.scratch(11, [&] { return ws_size(M, N, K); });
    auto *st = g.stream(12);
    return g.call([&] { return fn(x, w, s, zw, b, M, N, K, ab, wb, y, acc, ws, st); });
  });
}

// (fn): the function that returns the current stream's handle
PyObject *set_current_stream(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 1 || !PyCallable_Check(a[0])) {
    PyErr_SetString(PyExc_TypeError, "set_current_stream takes one function");
    return nullptr;
  }
  Py_INCREF(a[0]);
  Py_XDECREF(g_current_stream);
  g_current_stream = a[0];
  Py_RETURN_NONE;
}

#define OT_DEF(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    OT_DEF(set_current_stream), OT_DEF(quantize_act), OT_DEF(quantize_act_per_token), OT_DEF(ln_quantize_act),
    OT_DEF(qlinear), OT_DEF(qlinear_noalloc), OT_DEF(qlinear_packed),
    OT_DEF(qlinear_per_token), OT_DEF(qlinear_asym), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_otbind", nullptr, -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

// header_sha256: the include/ot.h whose signatures the calls use; ot.py compares
// it with the library's.  sources_sha256: what this file was built from.
PyMODINIT_FUNC PyInit__otbind(void) {
  PyObject *m = PyModule_Create(&kModule);
  if (m != nullptr && (PyModule_AddStringConstant(m, "header_sha256", OT_HEADER_SHA256) != 0 ||
                       PyModule_AddStringConstant(m, "sources_sha256", OT_BIND_SHA256) != 0)) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
