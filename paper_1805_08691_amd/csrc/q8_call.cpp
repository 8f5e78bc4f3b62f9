// The layer calls of the Python binding without its interpreter time: arguments checked and taken
// from the tensors here, one native call.  A layer of a small batch is 3 us of GPU time; through
// ctypes its call took 5.6 us of host time, of which the launch itself is 2.3.
//
// Only marshalling, as in binding.py: device tensors, contiguous, of the stated type (None: a null
// pointer); tensors of exactly torch.Tensor's type are read directly, others through the binding's
// own _ptr.  The functions called are the ones that the binding loaded (their addresses are handed
// over by bind()), on the current device's current stream; the interpreter lock is released during
// the call, as ctypes does.  Each function returns the library's return code.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include "../../include/q8conv.h"

namespace {

PyObject *g_ptr, *g_device, *g_stream, *g_desc_type, *g_int8, *g_int32, *g_float32, *g_uint8;
void* g_fn[8];
enum { kInt8, kU8, kPerChannel, kReal, kF32, kMaxabs, kQuantize, kDequantize };

// One call's arguments, read in order; `ok` turns false with a Python exception set.
struct Args {
  PyObject* const* a;
  bool ok = true;
  Py_buffer desc_buffer{};

  ~Args() {
    if (desc_buffer.obj) PyBuffer_Release(&desc_buffer);
  }
  const q8_conv_desc* desc(int i) {
    if (!ok) return nullptr;
    if (!PyObject_TypeCheck(a[i], (PyTypeObject*)g_desc_type)) {
      PyErr_SetString(PyExc_TypeError, "expected a ConvDesc");
      ok = false;
    } else if (PyObject_GetBuffer(a[i], &desc_buffer, PyBUF_SIMPLE) != 0) {
      ok = false;
    } else if (desc_buffer.len < (Py_ssize_t)sizeof(q8_conv_desc)) {
      PyErr_SetString(PyExc_TypeError, "ConvDesc is too small");
      ok = false;
    }
    return ok ? static_cast<const q8_conv_desc*>(desc_buffer.buf) : nullptr;
  }
  // Address of the tensor; elements: their number.
  // (type Undefined: any type)
  template <typename T>
  T* tensor(int i, at::ScalarType type, PyObject* dtype, long* elements = nullptr) {
    if (elements) *elements = 0;
    if (!ok || a[i] == Py_None) return nullptr;
    if (Py_TYPE(a[i]) == (PyTypeObject*)THPVariableClass) {
      const at::Tensor& t = THPVariable_Unpack(a[i]);
      try {
        if (t.is_cuda() && t.has_storage() && t.is_contiguous() &&
            (type == at::ScalarType::Undefined || t.scalar_type() == type)) {
          T* const p = static_cast<T*>(t.mutable_data_ptr());
          if (elements) *elements = t.numel();
          return p;
        }
      } catch (...) {        // (none may leave through the interpreter's frames)
      }
    }
    // The binding's own checks, and their exceptions: also for tensors of that type without storage,
    // as a function under vmap, grad or functionalize sees them.
    PyObject* address = PyObject_CallFunctionObjArgs(g_ptr, a[i], dtype, nullptr);
    void* p = address ? PyLong_AsVoidPtr(address) : nullptr;
    Py_XDECREF(address);
    if (elements && !PyErr_Occurred()) {
      PyObject* n = PyObject_CallMethod(a[i], "numel", nullptr);
      if (n) *elements = PyLong_AsLong(n);
      Py_XDECREF(n);
    }
    if (PyErr_Occurred()) ok = false;
    return ok ? static_cast<T*>(p) : nullptr;
  }
  // A tensor whose elements count: None has no number of them, and is none of length 0.
  template <typename T>
  T* counted(int i, at::ScalarType type, PyObject* dtype, long* elements) {
    if (ok && a[i] == Py_None) {
      Py_XDECREF(PyObject_GetAttrString(a[i], "numel"));       // the exception that this raises
      ok = false;
    }
    return tensor<T>(i, type, dtype, elements);
  }
  int8_t* i8(int i) { return tensor<int8_t>(i, at::kChar, g_int8); }
  int32_t* i32(int i) { return tensor<int32_t>(i, at::kInt, g_int32); }
  float* f32(int i) { return tensor<float>(i, at::kFloat, g_float32); }
  // The number inside an object of that ctypes type; null, with the exception as it is, for any other.
  static PyObject* boxed(PyObject* v, const char* type) {
    PyObject *kind, *error, *trace;
    PyErr_Fetch(&kind, &error, &trace);
    PyObject* ctypes = PyImport_ImportModule("ctypes");
    PyObject* t = ctypes ? PyObject_GetAttrString(ctypes, type) : nullptr;
    PyObject* n = t && PyObject_IsInstance(v, t) == 1 ? PyObject_GetAttrString(v, "value") : nullptr;
    Py_XDECREF(ctypes);
    Py_XDECREF(t);
    PyErr_Clear();
    if (!n) {
      PyErr_Restore(kind, error, trace);
      return nullptr;
    }
    Py_XDECREF(kind);
    Py_XDECREF(error);
    Py_XDECREF(trace);
    return n;
  }
  // As ctypes takes a c_float: whatever has __float__ or __index__, and its own objects.
  float factor(int i) {
    if (!ok) return 0.0f;
    double v = PyFloat_AsDouble(a[i]);
    if (v == -1.0 && PyErr_Occurred()) {
      PyObject* n = boxed(a[i], "c_float");
      if (n) v = PyFloat_AsDouble(n);
      Py_XDECREF(n);
    }
    if (PyErr_Occurred()) ok = false;
    return (float)v;
  }
  int integer(int i) {                       // ... and a c_int: whatever has __index__
    if (!ok) return 0;
    PyObject* n = PyNumber_Index(a[i]);
    if (!n) n = boxed(a[i], "c_int");
    const int v = n ? (int)PyLong_AsUnsignedLongMask(n) : 0;
    Py_XDECREF(n);
    if (PyErr_Occurred()) ok = false;
    return v;
  }
  int flag(int i) {
    if (!ok) return 0;
    PyObject* n = PyNumber_Long(a[i]);      // as int() takes it
    const int v = n ? (int)PyLong_AsUnsignedLongMask(n) : 0;
    Py_XDECREF(n);
    if (PyErr_Occurred()) ok = false;
    return v;
  }
  void* stream() {
    if (!ok) return nullptr;
    PyObject* d = PyObject_CallNoArgs(g_device);
    PyObject* s = d ? PyObject_CallOneArg(g_stream, d) : nullptr;
    void* p = s ? PyLong_AsVoidPtr(s) : nullptr;
    Py_XDECREF(d);
    Py_XDECREF(s);
    if (PyErr_Occurred()) ok = false;
    return p;
  }
};

bool count(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
  return false;
}

template <typename F>
PyObject* finish(Args& g, F call) {
  if (!g.ok) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// (desc, x, w, bias, q_x, q_w, q_out, residual, q_res, out, acc_dump, workspace)
PyObject* conv_int8(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 12)) return nullptr;
  Args g{args};
  const q8_conv_desc* d = g.desc(0);
  const int8_t *x = g.i8(1), *w = g.i8(2);
  const int32_t* b = g.i32(3);
  const float q_x = g.factor(4), q_w = g.factor(5), q_out = g.factor(6);
  const int8_t* res = g.i8(7);
  const float q_res = g.factor(8);
  int8_t* y = g.i8(9);
  int32_t* dump = g.i32(10);
  long bytes = 0;
  void* ws = g.tensor<uint8_t>(11, at::kByte, g_uint8, &bytes);
  void* s = g.stream();
  return finish(g, [&] {
    return ((decltype(&q8_conv_int8))g_fn[kInt8])(d, x, w, b, q_x, q_w, q_out, res, q_res, y, dump, ws,
                                                  (size_t)bytes, s);
  });
}

// (desc, in_u8, out_u8, res_u8, x, w, bias, taps, q_x, q_w, q_out, residual, q_res, out, acc_dump)
PyObject* conv_u8(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 15)) return nullptr;
  Args g{args};
  const q8_conv_desc* d = g.desc(0);
  const int in = g.flag(1), out = g.flag(2), ru = g.flag(3);
  const int8_t *x = g.i8(4), *w = g.i8(5);
  const int32_t *b = g.i32(6), *taps = g.i32(7);
  const float q_x = g.factor(8), q_w = g.factor(9), q_out = g.factor(10);
  const int8_t* res = g.i8(11);
  const float q_res = g.factor(12);
  int8_t* y = g.i8(13);
  int32_t* dump = g.i32(14);
  void* s = g.stream();
  return finish(g, [&] {
    return ((decltype(&q8_conv_u8))g_fn[kU8])(d, in, out, ru, x, w, b, taps, q_x, q_w, q_out, res, q_res, y,
                                              dump, s);
  });
}

// (desc, x, w, bias, m, q_out, residual, q_res, out, acc_dump)
PyObject* conv_per_channel(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 10)) return nullptr;
  Args g{args};
  const q8_conv_desc* d = g.desc(0);
  const int8_t *x = g.i8(1), *w = g.i8(2);
  const int32_t* b = g.i32(3);
  const float* m = g.f32(4);
  const float q_out = g.factor(5);
  const int8_t* res = g.i8(6);
  const float q_res = g.factor(7);
  int8_t* y = g.i8(8);
  int32_t* dump = g.i32(9);
  void* s = g.stream();
  return finish(g, [&] {
    return ((decltype(&q8_conv_int8_per_channel))g_fn[kPerChannel])(d, x, w, b, m, q_out, res, q_res, y, dump, s);
  });
}

// (desc, x, w, bias, q_x, q_w, residual, q_res, out)
PyObject* conv_real(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 9)) return nullptr;
  Args g{args};
  const q8_conv_desc* d = g.desc(0);
  const int8_t* x = g.i8(1);
  const void* w = g.tensor<void>(2, at::ScalarType::Undefined, Py_None);
  const int32_t* b = g.i32(3);
  const float q_x = g.factor(4), q_w = g.factor(5);
  const int8_t* res = g.i8(6);
  const float q_res = g.factor(7);
  float* y = g.f32(8);
  void* s = g.stream();
  return finish(g, [&] {
    return ((decltype(&q8_conv_int8_real_output))g_fn[kReal])(d, x, w, b, q_x, q_w, res, q_res, y, s);
  });
}

// (desc, x, w, bias, residual, out, maxabs_sum, maxabs_out, copies)
PyObject* conv_f32(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 9)) return nullptr;
  Args g{args};
  const q8_conv_desc* d = g.desc(0);
  const float *x = g.f32(1), *w = g.f32(2), *b = g.f32(3), *res = g.f32(4);
  float *y = g.f32(5), *m_sum = g.f32(6), *m_out = g.f32(7);
  const int copies = g.ok ? (int)PyLong_AsLong(args[8]) : 0;
  if (PyErr_Occurred()) g.ok = false;
  void* s = g.stream();
  return finish(g, [&] {
    return ((decltype(&q8_conv_f32_observed_spread))g_fn[kF32])(d, x, w, b, res, y, m_sum, m_out, copies, s);
  });
}

// (x, maximum)
PyObject* maxabs(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 2)) return nullptr;
  Args g{args};
  long len = 0;
  const float* x = g.counted<float>(0, at::kFloat, g_float32, &len);
  float* m = g.f32(1);
  void* s = g.stream();
  return finish(g, [&] { return ((decltype(&q8_calibrate_maxabs))g_fn[kMaxabs])(x, (size_t)len, m, s); });
}

// (r, q, p, z)
PyObject* quantize(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 4)) return nullptr;
  Args g{args};
  long len = 0;
  const float* r = g.counted<float>(0, at::kFloat, g_float32, &len);
  const float q = g.factor(1);
  const int p = g.integer(2);
  int8_t* z = g.i8(3);
  void* s = g.stream();
  return finish(g, [&] { return ((decltype(&q8_quantize))g_fn[kQuantize])(r, (size_t)len, q, p, z, s); });
}

// (z, q, r)
PyObject* dequantize(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 3)) return nullptr;
  Args g{args};
  long len = 0;
  const int8_t* z = g.counted<int8_t>(0, at::kChar, g_int8, &len);
  const float q = g.factor(1);
  float* r = g.f32(2);
  void* s = g.stream();
  return finish(g, [&] { return ((decltype(&q8_dequantize))g_fn[kDequantize])(z, (size_t)len, q, r, s); });
}

// bind(_ptr, get_device, get_stream, ConvDesc, int8, int32, float32, uint8, eight addresses)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 16)) return nullptr;
  PyObject** keep[] = {&g_ptr, &g_device, &g_stream, &g_desc_type, &g_int8, &g_int32, &g_float32, &g_uint8};
  for (int i = 0; i < 8; ++i) {
    Py_INCREF(args[i]);
    *keep[i] = args[i];
  }
  for (int i = 0; i < 8; ++i) {
    g_fn[i] = PyLong_AsVoidPtr(args[8 + i]);
    if (PyErr_Occurred()) return nullptr;
  }
  Py_RETURN_NONE;
}

#define Q8_METHOD(F) {#F, (PyCFunction)(void (*)(void))F, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {Q8_METHOD(conv_int8), Q8_METHOD(conv_u8), Q8_METHOD(conv_per_channel),
                         Q8_METHOD(conv_real), Q8_METHOD(conv_f32), Q8_METHOD(maxabs), Q8_METHOD(quantize),
                         Q8_METHOD(dequantize), Q8_METHOD(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_q8call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__q8call(void) { return PyModule_Create(&module); }
