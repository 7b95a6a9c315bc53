// The Python module _pycall: the calls a serving or training loop makes for every layer, marshalled natively.
//
// The small calls of this library are as long as their host side, and through ctypes 1.08 us of that were marshalling:
// an argument conversion each, three attribute reads per tensor, two calls for the stream.  Here a tensor is unpacked to
// its C++ object and the stream asked of torch directly, 0.22 us in all (both around a function that does nothing; the GPU hides part:
// 4096 x 4096 x 1 4.50 -> 4.10 us a call, an 8-bit 1000 x 512 x 64 4.39 -> 3.93).
// Nothing but arguments passes through: the functions of librmsmp.so are handed over by address (bind), so
// this module neither links to it nor knows it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include <cstdint>
#include <exception>

#include "rmsmp.h"

namespace {

decltype(&rmsmp_gemm) call_gemm;
decltype(&rmsmp_conv2d) call_conv2d;
decltype(&rmsmp_fake_quant_rows) call_fake_quant_rows;
decltype(&rmsmp_ste_backward) call_ste_backward;

// (a Python exception is set)
struct Raised {};

struct Owned {
  PyObject* o;
  explicit Owned(PyObject* obj) : o(obj) {
    if (!o) throw Raised{};
  }
  Owned(const Owned&) = delete;
  ~Owned() { Py_DECREF(o); }
};

bool truth(PyObject* o) {
  const int t = PyObject_IsTrue(o);
  if (t < 0) throw Raised{};
  return t != 0;
}

// Device pointer of a contiguous GPU tensor, null for None.  Tensors as such are read directly; a subclass, or
// whatever else has these attributes, is asked for them, and so is everything while a function mode watches.
void* device_pointer(PyObject* o) {
  if (o == Py_None) return nullptr;
  bool ok;
  if (THPVariable_CheckExact(o) && !at::impl::torch_function_mode_enabled()) {
    const at::Tensor& t = THPVariable_Unpack(o);
    ok = t.is_cuda() && t.is_contiguous();
    if (ok) return t.data_ptr();
  } else {
    const Owned cuda(PyObject_GetAttrString(o, "is_cuda"));
    ok = truth(cuda.o);
    if (ok) {
      const Owned contiguous(PyObject_CallMethod(o, "is_contiguous", nullptr));
      ok = truth(contiguous.o);
    }
    if (ok) {
      const Owned p(PyObject_CallMethod(o, "data_ptr", nullptr));
      void* v = PyLong_AsVoidPtr(p.o);
      if (PyErr_Occurred()) throw Raised{};
      return v;
    }
  }
  PyErr_SetString(PyExc_ValueError, "expected a contiguous GPU tensor");
  throw Raised{};
}

// The memory of a ctypes object of `size` bytes.
struct Memory {
  Py_buffer view;
  Memory(PyObject* o, size_t size) {
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Raised{};
    if ((size_t)view.len == size) return;
    PyBuffer_Release(&view);
    PyErr_SetString(PyExc_TypeError, "not the structure this call takes");
    throw Raised{};
  }
  Memory(const Memory&) = delete;
  ~Memory() { PyBuffer_Release(&view); }
  template <class T>
  const T* as() const {
    return (const T*)view.buf;
  }
};

// A packed layer's handle, a ctypes void pointer or None.
const rmsmp_packed* packed_handle(PyObject* o) {
  if (o == Py_None) return nullptr;
  const Memory m(o, sizeof(void*));
  return *m.as<const rmsmp_packed*>();
}

// None: torch's current stream; else a torch stream, or the number of one.
void* stream_of(PyObject* o) {
  if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream().stream();
  PyObject* s = PyObject_GetAttrString(o, "cuda_stream");
  if (!s) {
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) throw Raised{};
    PyErr_Clear();
    s = PyNumber_Long(o);
  }
  const Owned n(s);
  void* v = PyLong_AsVoidPtr(n.o);
  if (PyErr_Occurred()) throw Raised{};
  return v;
}

int64_t integer(PyObject* o) {
  const int64_t v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Raised{};
  return v;
}

// The two sizes of a matrix.
void matrix_sizes(PyObject* o, int64_t* rows, int64_t* columns) {
  const Owned shape(PyObject_GetAttrString(o, "shape"));
  const Owned fast(PySequence_Fast(shape.o, "shape"));
  if (PySequence_Fast_GET_SIZE(fast.o) != 2) {
    PyErr_SetString(PyExc_ValueError, "expected a matrix");
    throw Raised{};
  }
  *rows = integer(PySequence_Fast_GET_ITEM(fast.o, 0));
  *columns = integer(PySequence_Fast_GET_ITEM(fast.o, 1));
}

// Runs f with the number of arguments checked and every C++ exception turned into a Python one (which takes the
// interpreter's lock: see Unlocked); f returns the status.
template <class F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F&& f) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
    return nullptr;
  }
  try {
    return PyLong_FromLong((long)f());
  } catch (const Raised&) {
  } catch (const python_error&) {  // (torch's, with the Python exception set)
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  } catch (...) {
    PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
  }
  return nullptr;
}

// While one lives, the thread runs without the interpreter's lock; it is taken back however the scope is left.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  Unlocked() = default;
  Unlocked(const Unlocked&) = delete;
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// The library's call itself, without the interpreter's lock.
template <class F>
rmsmp_status unlocked(F&& f) {
  const Unlocked scope;
  return f();
}

// gemm(handle, X, N, ep, Y, stream)
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&] {
    const rmsmp_packed* w = packed_handle(a[0]);
    void* x = device_pointer(a[1]);
    const int64_t columns = integer(a[2]);
    const Memory ep(a[3], sizeof(rmsmp_epilogue));
    void* y = device_pointer(a[4]);
    void* s = stream_of(a[5]);
    return unlocked([&] { return call_gemm(w, x, columns, ep.as<rmsmp_epilogue>(), y, s); });
  });
}

// conv2d(handle, X, desc, ep, Y, workspace, workspace_bytes, stream)
PyObject* conv2d(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 8, [&] {
    const rmsmp_packed* w = packed_handle(a[0]);
    void* x = device_pointer(a[1]);
    const Memory d(a[2], sizeof(rmsmp_conv_desc));
    const Memory ep(a[3], sizeof(rmsmp_epilogue));
    void* y = device_pointer(a[4]);
    void* ws = device_pointer(a[5]);
    const int64_t bytes = integer(a[6]);
    void* s = stream_of(a[7]);
    return unlocked([&] { return call_conv2d(w, x, d.as<rmsmp_conv_desc>(), ep.as<rmsmp_epilogue>(), y, ws, (size_t)bytes, s); });
  });
}

// fake_quant_rows(W, scheme, What, alpha, alpha_out, stream)
PyObject* fake_quant_rows(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&] {
    int64_t rows, columns;
    matrix_sizes(a[0], &rows, &columns);
    void* w = device_pointer(a[0]);
    void* scheme = device_pointer(a[1]);
    void* alpha = device_pointer(a[3]);
    void* what = device_pointer(a[2]);
    void* alpha_out = device_pointer(a[4]);
    void* s = stream_of(a[5]);
    return unlocked([&] { return call_fake_quant_rows((const float*)w, rows, columns, (const uint8_t*)scheme, (const float*)alpha, (float*)what, (float*)alpha_out, s); });
  });
}

// ste_backward(dWhat, dW, W, alpha, stream)
PyObject* ste_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 5, [&] {
    int64_t rows, columns;
    matrix_sizes(a[0], &rows, &columns);
    void* w = device_pointer(a[2]);
    void* alpha = device_pointer(a[3]);
    void* grad = device_pointer(a[0]);
    void* out = device_pointer(a[1]);
    void* s = stream_of(a[4]);
    return unlocked([&] { return call_ste_backward((const float*)w, (const float*)alpha, (const float*)grad, rows, columns, (float*)out, s); });
  });
}

// bind(gemm, conv2d, fake_quant_rows, ste_backward): their addresses
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 4, [&] {
    void* p[4];
    for (int i = 0; i < 4; ++i) {
      p[i] = PyLong_AsVoidPtr(a[i]);
      if (PyErr_Occurred()) throw Raised{};
    }
    call_gemm = (decltype(call_gemm))p[0];
    call_conv2d = (decltype(call_conv2d))p[1];
    call_fake_quant_rows = (decltype(call_fake_quant_rows))p[2];
    call_ste_backward = (decltype(call_ste_backward))p[3];
    return 0;
  });
}

#define PYCALL(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PYCALL(bind), PYCALL(gemm), PYCALL(conv2d), PYCALL(fake_quant_rows), PYCALL(ste_backward), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) { return PyModule_Create(&module); }
