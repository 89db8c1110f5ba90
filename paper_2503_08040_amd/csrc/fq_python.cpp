// The calls of a layer's every step (quantize, multiply) without ctypes in between.
//
// A small layer is bound by the host: of the 10.8 us that fq_quantize + fq_gemm took to issue, the runtime's two
// launches are 5.4; the rest was Python reading a tensor's properties one by one, ctypes converting nine
// arguments and torch.empty parsing its own.  Here a call reads them from the tensor itself: 7.8 us.  Only the plain case is
// taken (torch.Tensor itself, the expected types, the current stream): for anything else these functions return
// None and the Python code in front of them, which is the definition of what is accepted and of every error, runs.
// What torch throws here leaves as torch's own Python functions translate it (torch.OutOfMemoryError from the
// output's allocation, a Python exception from a dispatch mode).
#include <Python.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <algorithm>

#include "../../include/fq.h"

namespace {

typedef fq_status (*QuantizeFn)(const void*, int32_t, int32_t, int64_t, int32_t, fq_criterion, float, fq_qtensor*, void*);
typedef fq_status (*QuantizeSrFn)(const void*, int32_t, int32_t, int64_t, int32_t, uint64_t, fq_qtensor*, void*);
typedef fq_status (*GemmFn)(fq_op, const fq_qtensor*, const fq_qtensor*, void*, fq_out_dtype, int64_t, void*);

QuantizeFn g_quantize;
QuantizeSrFn g_quantize_sr;
GemmFn g_gemm;
PyObject *g_device, *g_stream;       // torch's current device, and the raw handle of a device's current stream

// setup(address of fq_quantize, of fq_quantize_sr, of fq_gemm, current device, raw stream): the loaded library's
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 5) return PyErr_Format(PyExc_TypeError, "setup takes 5 arguments");
  void* p[3];
  for (int i = 0; i < 3; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  g_quantize = reinterpret_cast<QuantizeFn>(p[0]);
  g_quantize_sr = reinterpret_cast<QuantizeSrFn>(p[1]);
  g_gemm = reinterpret_cast<GemmFn>(p[2]);
  Py_INCREF(a[3]);
  Py_INCREF(a[4]);
  Py_XSETREF(g_device, a[3]);
  Py_XSETREF(g_stream, a[4]);
  Py_RETURN_NONE;
}

bool current_stream(void** out) {
  PyObject* dev = PyObject_CallNoArgs(g_device);
  if (!dev) return false;
  PyObject* s = PyObject_CallOneArg(g_stream, dev);
  Py_DECREF(dev);
  if (!s) return false;
  *out = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return !PyErr_Occurred();
}

struct Matrix {
  void* ptr;
  int32_t rows, cols;
  int64_t ld;
};

// A bf16 matrix on the GPU with unit column stride.
bool matrix(PyObject* o, Matrix* m) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.layout() != at::kStrided || t.dim() != 2 || t.scalar_type() != at::kBFloat16) return false;
  const int64_t rows = t.size(0), cols = t.size(1);
  if (rows > INT32_MAX || cols > INT32_MAX || (t.stride(1) != 1 && cols > 1)) return false;
  *m = {t.data_ptr(), (int32_t)rows, (int32_t)cols, rows > 1 ? t.stride(0) : std::max<int64_t>(cols, 1)};
  return true;
}

bool int_arg(PyObject* o, long* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongAndOverflow(o, &over);
  return !over && *v >= INT32_MIN && *v <= INT32_MAX;
}

// call() while other Python threads run.
template <class F>
auto without_gil(const F& call) {
  pybind11::gil_scoped_release others;
  return call();
}

template <class F>
PyObject* launch(const F& call) {
  return PyLong_FromLong(without_gil(call));
}

// quantize(x, crit, theta, address of the fq_qtensor, block) -> status or None
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Matrix m;
  long crit, block;
  if (n != 5 || !PyFloat_CheckExact(a[2]) || !int_arg(a[1], &crit) || !int_arg(a[4], &block) || !matrix(a[0], &m))
    Py_RETURN_NONE;
  const float theta = (float)PyFloat_AS_DOUBLE(a[2]);
  fq_qtensor* const q = static_cast<fq_qtensor*>(PyLong_AsVoidPtr(a[3]));
  void* st;
  if (PyErr_Occurred() || !current_stream(&st)) return nullptr;
  return launch([&] { return g_quantize(m.ptr, m.rows, m.cols, m.ld, (int32_t)block, (fq_criterion)crit, theta, q, st); });
  END_HANDLE_TH_ERRORS
}

// quantize_sr(x, seed, address of the fq_qtensor) -> status or None
PyObject* quantize_sr(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Matrix m;
  if (n != 3 || !PyLong_CheckExact(a[1]) || !matrix(a[0], &m)) Py_RETURN_NONE;
  const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[1]);
  fq_qtensor* const q = static_cast<fq_qtensor*>(PyLong_AsVoidPtr(a[2]));
  void* st;
  if (PyErr_Occurred() || !current_stream(&st)) return nullptr;
  return launch([&] { return g_quantize_sr(m.ptr, m.rows, m.cols, m.ld, FQ_BLOCK, seed, q, st); });
  END_HANDLE_TH_ERRORS
}

// gemm(op, address of A's fq_qtensor, of B's, a tensor on the output's device, out or None, dtype or None)
// -> (status, out) or None
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  long op;
  if (n != 6 || !int_arg(a[0], &op) || !THPVariable_CheckExact(a[3])) Py_RETURN_NONE;
  const fq_qtensor* const A = static_cast<fq_qtensor*>(PyLong_AsVoidPtr(a[1]));
  const fq_qtensor* const B = static_cast<fq_qtensor*>(PyLong_AsVoidPtr(a[2]));
  if (PyErr_Occurred()) return nullptr;
  int64_t rows, cols;
  switch (op) {
    case FQ_OP_NT: rows = A->rows; cols = B->rows; break;
    case FQ_OP_NN: rows = A->rows; cols = B->cols; break;
    case FQ_OP_TN: rows = A->cols; cols = B->cols; break;
    default: Py_RETURN_NONE;
  }
  at::ScalarType type = at::kFloat;
  int64_t ld = std::max<int64_t>(cols, 1);
  at::Tensor out;
  if (a[4] == Py_None) {
    if (a[5] != Py_None) {
      if (!THPDtype_Check(a[5])) Py_RETURN_NONE;
      type = reinterpret_cast<THPDtype*>(a[5])->scalar_type;
    }
    if (type != at::kFloat && type != at::kBFloat16) Py_RETURN_NONE;
    // a mode that sees torch's functions sees torch.empty of the Python code
    if (at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    const at::TensorOptions options = THPVariable_Unpack(a[3]).options().dtype(type);
    out = without_gil([&] { return at::empty({rows, cols}, options); });     // may wait for the device or the driver
  } else {
    if (!THPVariable_CheckExact(a[4])) Py_RETURN_NONE;
    out = THPVariable_Unpack(a[4]);
    type = out.scalar_type();
    if (!out.is_cuda() || (type != at::kFloat && type != at::kBFloat16) || out.layout() != at::kStrided || out.dim() != 2 ||
        out.size(0) != rows || out.size(1) != cols || (out.stride(1) != 1 && cols > 1))
      Py_RETURN_NONE;
    if (rows > 1) ld = out.stride(0);
  }
  void* st;
  if (!current_stream(&st)) return nullptr;
  void* const c = out.data_ptr();
  PyObject* status = launch([&] { return g_gemm((fq_op)op, A, B, c, type == at::kFloat ? FQ_OUT_F32 : FQ_OUT_BF16, ld, st); });
  if (!status) return nullptr;
  PyObject* t = a[4] == Py_None ? THPVariable_Wrap(out) : Py_NewRef(a[4]);
  if (!t) {
    Py_DECREF(status);
    return nullptr;
  }
  PyObject* r = PyTuple_Pack(2, status, t);
  Py_DECREF(status);
  Py_DECREF(t);
  return r;
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"setup", reinterpret_cast<PyCFunction>(setup), METH_FASTCALL, nullptr},
    {"quantize", reinterpret_cast<PyCFunction>(quantize), METH_FASTCALL, nullptr},
    {"quantize_sr", reinterpret_cast<PyCFunction>(quantize_sr), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(gemm), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fqnative", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fqnative() {
  PyObject* m = PyModule_Create(&module);
  if (m) {
    PyModule_AddStringConstant(m, "torch_version", FQ_TORCH_VERSION);
    PyModule_AddStringConstant(m, "header_tag", FQ_HEADER_TAG);      // of fq.h: the structs read and the entry points called
  }
  return m;
}
