// Argument marshalling of the launch entry points for torch tensors, as a CPython extension: reads the addresses of the
// tensors of a call, looks up the current stream and calls the C ABI of libsfmp.so.
//
// A decode launch takes 4 to 12 us on the GPU.  Marshalled in Python (ctypes, four tensor methods per argument) an
// sfmp_gemm call took 12.1 us of host time and a launch of three projections 16.2, so that a program waited for the host;
// marshalled here 3.8 and 3.9, most of it the launch itself (back to back, 512 -> 512: 11.6 -> 4.2 us a call, a decoder
// layer of an 8B model in four calls 46 -> 29 us).
//
// Only plain calls are taken: torch.Tensor or Parameter objects themselves (no subclass, which may have methods of its
// own), None, an SfmpLayout.  For anything else a function returns None, nothing having been launched, and the general
// path in binding.py decides, with its own errors.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sfmp.h"

namespace {

struct Api {
  decltype(&sfmp_gemm) gemm = nullptr;
  decltype(&sfmp_gemm_static) gemm_static = nullptr;
  decltype(&sfmp_gemv_batched) gemv_batched = nullptr;
  decltype(&sfmp_gemm_batched) gemm_batched = nullptr;
};

// set by bind()
Api api;
PyObject* layout_type = nullptr;
PyObject* get_device = nullptr;      // torch._C._cuda_getDevice
PyObject* get_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream
PyObject* names[9];                  // attributes of a DevicePacked, then "cuda_stream"
const char* const kNames[9] = {"layout", "s2", "s3", "s4", "index", "scales", "zeros", "bitmap", "cuda_stream"};

// What became of reading an argument: taken, not a plain one (the general path decides), or a Python error is set
enum Read { kTaken, kOther, kError };

// Address of a tensor (null for None and for an empty one).  device: the tensor has to be a contiguous one on the GPU.
Read tensor_address(PyObject* o, bool device, const void** out) {
  *out = nullptr;
  if (o == Py_None) return kTaken;
  if (!THPVariable_CheckExact(o)) return kOther;
  try {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.numel() == 0) return kTaken;
    if (device && (!t.is_cuda() || !t.is_contiguous())) return kOther;
    *out = t.data_ptr();
    return kTaken;
  } catch (const std::exception&) {  // a tensor without memory of its own: the general path raises its error
    return kOther;
  }
}

Read tensor_rows(PyObject* o, int64_t* rows, int64_t* numel, int64_t* bytes) {
  if (!THPVariable_CheckExact(o)) return kOther;
  try {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (rows) {
      if (t.dim() < 1 || t.size(0) > INT32_MAX) return kOther;
      *rows = t.size(0);
    }
    if (numel) *numel = t.numel();
    if (bytes) *bytes = t.numel() * (int64_t)t.element_size();
    return kTaken;
  } catch (const std::exception&) {
    return kOther;
  }
}

// Address of the C struct of an SfmpLayout (the caller holds a reference through the call)
Read layout_address(PyObject* o, const sfmp_layout_t** out) {
  if ((PyObject*)Py_TYPE(o) != layout_type) return kOther;
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return kError;
  *out = b.len == (Py_ssize_t)sizeof(sfmp_layout_t) ? (const sfmp_layout_t*)b.buf : nullptr;
  PyBuffer_Release(&b);
  return *out ? kTaken : kOther;
}

Read stream_handle(PyObject* stream, void** out) {
  PyObject* h;
  if (stream == Py_None) {
    PyObject* dev = PyObject_CallNoArgs(get_device);
    h = dev ? PyObject_CallOneArg(get_raw_stream, dev) : nullptr;
    Py_XDECREF(dev);
    if (!h) {  // no usable GPU: the general path initialises torch's side, or raises its error
      PyErr_Clear();
      return kOther;
    }
  } else {
    h = PyObject_GetAttr(stream, names[8]);
  }
  if (!h) return kError;
  *out = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  return PyErr_Occurred() ? kError : kTaken;
}

#define SFMP_READ(expr)                        \
  do {                                         \
    const Read r_ = (expr);                    \
    if (r_ == kError) return nullptr;          \
    if (r_ == kOther) Py_RETURN_NONE;          \
  } while (0)

// gemm(X, col_perm, layout, s2, s3, s4, index, scales, zeros, bitmap, row_perm, Y, workspace or missing, stream)
template <bool STATIC>
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr Py_ssize_t kArgs = STATIC ? 13 : 14;
  if (n != kArgs) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  int64_t M = 0, nbytes = 0;
  const sfmp_layout_t* layout = nullptr;
  const void* p[13] = {};
  if constexpr (!STATIC) SFMP_READ(tensor_rows(a[12], nullptr, nullptr, &nbytes));
  SFMP_READ(tensor_rows(a[0], &M, nullptr, nullptr));
  SFMP_READ(layout_address(a[2], &layout));
  for (int i = 0; i < kArgs - 1; ++i)
    if (i != 2) SFMP_READ(tensor_address(a[i], true, &p[i]));
  void* stream = nullptr;
  SFMP_READ(stream_handle(a[kArgs - 1], &stream));
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  if constexpr (STATIC)
    rc = api.gemm_static(p[0], (int32_t)M, (const int32_t*)p[1], layout, p[3], p[4], p[5], (const int32_t*)p[6], p[7],
                         p[8], (const int8_t*)p[9], (const int32_t*)p[10], (void*)p[11], stream);
  else
    rc = api.gemm(p[0], (int32_t)M, (const int32_t*)p[1], layout, p[3], p[4], p[5], (const int32_t*)p[6], p[7], p[8],
                  (const int8_t*)p[9], (const int32_t*)p[10], (void*)p[11], (void*)p[12], nbytes, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(rc);
}

constexpr Py_ssize_t kMaxBatch = 8;  // more are refused by the library: left to the general path

// References to everything whose address has been read, dropped when the call returns (with the GIL held).  The tensors
// and layouts of a batch hang on a list and on attributes that other Python code - an attribute lookup of this call, a
// stream object's property, another thread while the library runs without the GIL - may change or clear meanwhile.
struct Held {
  PyObject* ref[1 + 8 * kMaxBatch];
  int count = 0;
  void take(PyObject* owned) { ref[count++] = owned; }
  Held() = default;
  Held(const Held&) = delete;
  Held& operator=(const Held&) = delete;
  ~Held() {
    while (count > 0) Py_DECREF(ref[--count]);
  }
};

// problems: list or tuple of (X, col_perm, DevicePacked, row_perm, Y)
Read read_problems(PyObject* problems, sfmp_gemv_problem_t* out, int32_t* count, Held* held) {
  if (!PyList_CheckExact(problems) && !PyTuple_CheckExact(problems)) return kOther;
  PyObject* all = PySequence_Tuple(problems);  // (its items, and theirs, stay as they are through the call)
  if (!all) return kError;
  held->take(all);
  const Py_ssize_t n = PyTuple_GET_SIZE(all);
  if (n > kMaxBatch) return kOther;
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* q = PyTuple_GET_ITEM(all, i);
    if (!PyTuple_CheckExact(q) || PyTuple_GET_SIZE(q) != 5) return kOther;
    PyObject* dp = PyTuple_GET_ITEM(q, 2);
    const void* v[12] = {};
    if (Read r = tensor_address(PyTuple_GET_ITEM(q, 0), false, &v[0])) return r;
    if (Read r = tensor_address(PyTuple_GET_ITEM(q, 1), false, &v[1])) return r;
    for (int k = 0; k < 8; ++k) {
      PyObject* o = PyObject_GetAttr(dp, names[k]);
      if (!o) return kError;
      held->take(o);
      const Read r = k == 0 ? layout_address(o, (const sfmp_layout_t**)&v[2]) : tensor_address(o, false, &v[2 + k]);
      if (r != kTaken) return r;
    }
    if (Read r = tensor_address(PyTuple_GET_ITEM(q, 3), false, &v[10])) return r;
    if (Read r = tensor_address(PyTuple_GET_ITEM(q, 4), false, &v[11])) return r;
    out[i] = sfmp_gemv_problem_t{v[0], (const int32_t*)v[1], (const sfmp_layout_t*)v[2], v[3], v[4], v[5],
                                 (const int32_t*)v[6], v[7], v[8], (const int8_t*)v[9], (const int32_t*)v[10],
                                 (void*)v[11]};
  }
  *count = (int32_t)n;
  return kTaken;
}

// gemv_batched(problems, stream)
PyObject* gemv_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 2) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  Held held;
  sfmp_gemv_problem_t q[kMaxBatch];
  int32_t count = 0;
  void* stream = nullptr;
  SFMP_READ(read_problems(a[0], q, &count, &held));
  SFMP_READ(stream_handle(a[1], &stream));
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = api.gemv_batched(q, count, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(rc);
}

// gemm_batched(problems, M, workspace, stream)
PyObject* gemm_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 4) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  Held held;
  sfmp_gemv_problem_t q[kMaxBatch];
  int32_t count = 0;
  void* stream = nullptr;
  const void* ws = nullptr;
  int64_t numel = 0;
  if (!PyLong_CheckExact(a[1])) Py_RETURN_NONE;
  int overflow = 0;
  const long M = PyLong_AsLongAndOverflow(a[1], &overflow);
  if (overflow || M < INT32_MIN || M > INT32_MAX) Py_RETURN_NONE;
  SFMP_READ(read_problems(a[0], q, &count, &held));
  if (a[2] == Py_None) Py_RETURN_NONE;
  SFMP_READ(tensor_rows(a[2], nullptr, &numel, nullptr));
  if (numel == 0) Py_RETURN_NONE;
  SFMP_READ(tensor_address(a[2], false, &ws));
  SFMP_READ(stream_handle(a[3], &stream));
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = api.gemm_batched(q, count, (int32_t)M, (void*)ws, numel, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(rc);
}

// bind(SfmpLayout, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, addresses of the four C functions)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 7) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  void* f[4];
  for (int i = 0; i < 4; ++i) {
    f[i] = PyLong_AsVoidPtr(a[3 + i]);
    if (!f[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null function");
      return nullptr;
    }
  }
  PyObject** const slot[3] = {&layout_type, &get_device, &get_raw_stream};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(a[i]);
    Py_XSETREF(*slot[i], a[i]);
  }
  api.gemm = (decltype(api.gemm))f[0];
  api.gemm_static = (decltype(api.gemm_static))f[1];
  api.gemv_batched = (decltype(api.gemv_batched))f[2];
  api.gemm_batched = (decltype(api.gemm_batched))f[3];
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"gemm", (PyCFunction)(void (*)(void))gemm<false>, METH_FASTCALL, nullptr},
    {"gemm_static", (PyCFunction)(void (*)(void))gemm<true>, METH_FASTCALL, nullptr},
    {"gemv_batched", (PyCFunction)(void (*)(void))gemv_batched, METH_FASTCALL, nullptr},
    {"gemm_batched", (PyCFunction)(void (*)(void))gemm_batched, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sfmp_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sfmp_torch(void) {
  for (int i = 0; i < 9; ++i)
    if (!(names[i] = PyUnicode_InternFromString(kNames[i]))) return nullptr;
  PyObject* m = PyModule_Create(&module);
  // (checked by binding.py before anything else of the module is used)
  if (m && PyModule_AddStringConstant(m, "built_for", SFMP_BUILT_FOR) != 0) Py_CLEAR(m);
  return m;
}
