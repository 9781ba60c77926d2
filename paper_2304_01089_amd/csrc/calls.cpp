// CPython module `_calls`: the argument marshalling of the entry points that a serving loop calls, in native code.
//
// A short call is paced by the host, and Python-level marshalling was half of its time there (one linear layer,
// rptq_ln_quant + rptq_cluster_gemm: 15.0 us a pass with ctypes, of which 6.5 in the two launches, 9.78 with this).  Every function takes the binding's arguments by position and covers the ordinary case only:
// contiguous device tensors of the right type, one-dimensional float32 / int32 tables that support the buffer protocol,
// ints in range, the current stream.  For anything else it returns None without having called the library, and
// binding.py's own code converts, or raises, as it always has.  It keeps nothing between calls but the library's entry
// points and torch's dtype objects and stream query.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "rptq.h"

namespace {

decltype(&rptq_ln_quant) f_ln_quant;
decltype(&rptq_cluster_gemm) f_cluster_gemm;
decltype(&rptq_cluster_gemm_quant) f_cluster_gemm_quant;
decltype(&rptq_cluster_rowsums) f_cluster_rowsums;
decltype(&rptq_cluster_gemm_cw) f_cluster_gemm_cw;
decltype(&rptq_kv_quant) f_kv_quant;
decltype(&rptq_kv_dequant) f_kv_dequant;

PyObject *n_is_cuda, *n_is_contiguous, *n_dtype, *n_data_ptr, *n_nbytes;     // attribute names
PyObject *t_bf16, *t_f32, *t_i32, *get_device, *get_stream;         // torch's objects

// Each getter returns false, with no Python error set, where the ordinary case does not apply.
bool no_error() {
  PyErr_Clear();
  return false;
}

bool get_i64(PyObject* o, int64_t* out) {
  if (!PyLong_Check(o)) return false;
  int overflow = 0;
  *out = PyLong_AsLongLongAndOverflow(o, &overflow);
  return overflow == 0;
}

bool get_i32(PyObject* o, int32_t* out) {
  int64_t v;
  if (!get_i64(o, &v) || v < INT32_MIN || v > INT32_MAX) return false;
  *out = static_cast<int32_t>(v);
  return true;
}

bool get_f32(PyObject* o, float* out) {
  if (!PyFloat_Check(o)) return false;
  *out = static_cast<float>(PyFloat_AS_DOUBLE(o));
  return true;
}

bool get_flag(PyObject* o, int32_t* out) {
  if (o != Py_True && o != Py_False) return false;
  *out = o == Py_True;
  return true;
}

bool is_true(PyObject* owned) {
  if (owned == nullptr) return no_error();
  const bool t = owned == Py_True;
  Py_DECREF(owned);
  return t;
}

PyObject* dtype_of(PyObject* t) {                        // (borrowed in effect: dtype objects live as long as torch)
  PyObject* d = PyObject_GetAttr(t, n_dtype);
  if (d == nullptr) {
    PyErr_Clear();
    return nullptr;
  }
  Py_DECREF(d);
  return d;
}

// Address of a contiguous device tensor of that dtype (any if NULL); None is NULL where it is allowed.
template <typename T>
bool get_tensor(PyObject* t, PyObject* dtype, bool allow_none, T** out) {
  if (t == Py_None) {
    *out = nullptr;
    return allow_none;
  }
  if (!is_true(PyObject_GetAttr(t, n_is_cuda)) || !is_true(PyObject_CallMethodNoArgs(t, n_is_contiguous))) return false;
  if (dtype != nullptr && dtype_of(t) != dtype) return false;
  PyObject* p = PyObject_CallMethodNoArgs(t, n_data_ptr);
  if (p == nullptr) return no_error();
  void* v = PyLong_Check(p) ? PyLong_AsVoidPtr(p) : nullptr;
  const bool ok = PyLong_Check(p) && !PyErr_Occurred();
  Py_DECREF(p);
  *out = static_cast<T*>(v);
  return ok || no_error();
}

bool get_bytes(PyObject* t, int64_t* out) {
  PyObject* b = PyObject_GetAttr(t, n_nbytes);
  if (b == nullptr) return no_error();
  const bool ok = get_i64(b, out) && *out >= 0;
  Py_DECREF(b);
  return ok;
}

// A one-dimensional table of 4-byte elements ('f' or 'i'), borrowed for the call.
struct Table {
  Py_buffer b;
  bool held = false;
  ~Table() {
    if (held) PyBuffer_Release(&b);
  }
  bool get(PyObject* o, char format) {
    if (!PyObject_CheckBuffer(o)) return false;
    if (PyObject_GetBuffer(o, &b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) return no_error();
    held = true;
    return b.ndim == 1 && b.itemsize == 4 && b.format != nullptr && b.format[0] == format && b.format[1] == 0 &&
           (reinterpret_cast<uintptr_t>(b.buf) & 3u) == 0;
  }
  const int32_t* ints() const { return static_cast<const int32_t*>(b.buf); }
  const float* floats() const { return static_cast<const float*>(b.buf); }
  int32_t size() const { return static_cast<int32_t>(b.shape[0]); }
};

bool get_current_stream(PyObject* stream, void** out) {
  if (stream != Py_None) return false;
  PyObject* device = PyObject_CallNoArgs(get_device);
  if (device == nullptr) return no_error();
  PyObject* s = PyObject_CallOneArg(get_stream, device);
  Py_DECREF(device);
  if (s == nullptr) return no_error();
  const bool ok = PyLong_Check(s);
  *out = ok ? PyLong_AsVoidPtr(s) : nullptr;
  Py_DECREF(s);
  return (ok && !PyErr_Occurred()) || no_error();
}

// Y's dtype as the library names it.
bool get_y_dtype(PyObject* y, int32_t* out) {
  PyObject* d = dtype_of(y);
  *out = d == t_f32 ? RPTQ_DTYPE_F32 : RPTQ_DTYPE_BF16;
  return d == t_f32 || d == t_bf16;
}

template <typename F>
PyObject* run(F&& call) {                                // (other Python threads go on meanwhile, as under ctypes)
  int32_t status;
  Py_BEGIN_ALLOW_THREADS
  status = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// (x, M, d, gamma_pad, beta_pad, eps, relu, perm_pad, cluster_off, s, inv_s, z, bits, codes, xsum, rowterm, stream)
PyObject* ln_quant(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *x, *codes, *stream;
  float *gamma, *beta, *rowterm, eps;
  int32_t *perm, *xsum, d, relu, bits;
  int64_t M;
  Table off, s, inv, z;
  if (n != 17 || f_ln_quant == nullptr || !get_tensor(a[0], t_bf16, false, &x) || !get_i64(a[1], &M) || !get_i32(a[2], &d) ||
      !get_tensor(a[3], t_f32, true, &gamma) || !get_tensor(a[4], t_f32, true, &beta) || !get_f32(a[5], &eps) ||
      !get_flag(a[6], &relu) || !get_tensor(a[7], t_i32, false, &perm) || !off.get(a[8], 'i') || !s.get(a[9], 'f') ||
      !inv.get(a[10], 'f') || !z.get(a[11], 'i') || !get_i32(a[12], &bits) || !get_tensor(a[13], nullptr, false, &codes) ||
      !get_tensor(a[14], t_i32, true, &xsum) || !get_tensor(a[15], t_f32, true, &rowterm) || !get_current_stream(a[16], &stream))
    Py_RETURN_NONE;
  return run([&] {
    return f_ln_quant(x, M, d, gamma, beta, eps, relu, perm, off.ints(), off.size() - 1, s.floats(), inv.floats(), z.ints(),
                      bits, codes, xsum, rowterm, stream);
  });
}

// (codes, M, bits, Wq, N, cluster_off, sX, sW, zW, colterm, rowterm, y, stream)
PyObject* cluster_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *codes, *wq, *y, *stream;
  float *sw, *colterm, *rowterm;
  int32_t *zw, bits, N, y_dtype;
  int64_t M;
  Table off, sx;
  if (n != 13 || f_cluster_gemm == nullptr || !get_tensor(a[0], nullptr, false, &codes) || !get_i64(a[1], &M) ||
      !get_i32(a[2], &bits) || !get_tensor(a[3], nullptr, false, &wq) || !get_i32(a[4], &N) || !off.get(a[5], 'i') ||
      !sx.get(a[6], 'f') || !get_tensor(a[7], t_f32, false, &sw) || !get_tensor(a[8], t_i32, false, &zw) ||
      !get_tensor(a[9], t_f32, false, &colterm) || !get_tensor(a[10], t_f32, false, &rowterm) ||
      !get_y_dtype(a[11], &y_dtype) || !get_tensor(a[11], nullptr, false, &y) || !get_current_stream(a[12], &stream))
    Py_RETURN_NONE;
  return run([&] {
    return f_cluster_gemm(codes, M, bits, wq, N, off.ints(), off.size() - 1, sx.floats(), sw, zw, colterm, rowterm, y,
                          y_dtype, stream);
  });
}

// (codes, M, bits, Wq, N, cluster_off, sX, sW, zW, colterm, rowterm, relu, next_cluster_off, next_s, next_inv_s, next_z,
//  next_bits, next_codes, next_rowterm, workspace, stream)
PyObject* cluster_gemm_quant(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *codes, *wq, *next_codes, *workspace, *stream;
  float *sw, *colterm, *rowterm, *next_rowterm;
  int32_t *zw, bits, N, relu, next_bits;
  int64_t M, bytes;
  Table off, sx, noff, ns, ni, nz;
  if (n != 21 || f_cluster_gemm_quant == nullptr || !get_tensor(a[0], nullptr, false, &codes) || !get_i64(a[1], &M) ||
      !get_i32(a[2], &bits) || !get_tensor(a[3], nullptr, false, &wq) || !get_i32(a[4], &N) || !off.get(a[5], 'i') ||
      !sx.get(a[6], 'f') || !get_tensor(a[7], t_f32, false, &sw) || !get_tensor(a[8], t_i32, false, &zw) ||
      !get_tensor(a[9], t_f32, false, &colterm) || !get_tensor(a[10], t_f32, false, &rowterm) || !get_flag(a[11], &relu) ||
      !noff.get(a[12], 'i') || !ns.get(a[13], 'f') || !ni.get(a[14], 'f') || !nz.get(a[15], 'i') ||
      !get_i32(a[16], &next_bits) || !get_tensor(a[17], nullptr, false, &next_codes) ||
      !get_tensor(a[18], t_f32, false, &next_rowterm) || !get_tensor(a[19], nullptr, false, &workspace) ||
      !get_bytes(a[19], &bytes) || !get_current_stream(a[20], &stream))
    Py_RETURN_NONE;
  return run([&] {
    return f_cluster_gemm_quant(codes, M, bits, wq, N, off.ints(), off.size() - 1, sx.floats(), sw, zw, colterm, rowterm, relu,
                                noff.ints(), noff.size() - 1, ns.floats(), ni.floats(), nz.ints(), next_bits, next_codes,
                                next_rowterm, workspace, static_cast<size_t>(bytes), stream);
  });
}

// (codes, M, bits, cluster_off, sX, zX, rowsums, stream)
PyObject* cluster_rowsums(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *codes, *stream;
  float* rowsums;
  int32_t bits;
  int64_t M;
  Table off, sx, zx;
  if (n != 8 || f_cluster_rowsums == nullptr || !get_tensor(a[0], nullptr, false, &codes) || !get_i64(a[1], &M) ||
      !get_i32(a[2], &bits) || !off.get(a[3], 'i') || !sx.get(a[4], 'f') || !zx.get(a[5], 'i') ||
      !get_tensor(a[6], t_f32, false, &rowsums) || !get_current_stream(a[7], &stream))
    Py_RETURN_NONE;
  return run([&] { return f_cluster_rowsums(codes, M, bits, off.ints(), off.size() - 1, sx.floats(), zx.ints(), rowsums, stream); });
}

// (codes, M, bits, Wq, N, cluster_off, scale_tab, cross_tab, colterm, rowsums, y, stream)
PyObject* cluster_gemm_cw(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *codes, *wq, *y, *stream;
  float *scale, *cross, *colterm, *rowsums;
  int32_t bits, N, y_dtype;
  int64_t M;
  Table off;
  if (n != 12 || f_cluster_gemm_cw == nullptr || !get_tensor(a[0], nullptr, false, &codes) || !get_i64(a[1], &M) ||
      !get_i32(a[2], &bits) || !get_tensor(a[3], nullptr, false, &wq) || !get_i32(a[4], &N) || !off.get(a[5], 'i') ||
      !get_tensor(a[6], t_f32, false, &scale) || !get_tensor(a[7], t_f32, false, &cross) ||
      !get_tensor(a[8], t_f32, false, &colterm) || !get_tensor(a[9], t_f32, false, &rowsums) ||
      !get_y_dtype(a[10], &y_dtype) || !get_tensor(a[10], nullptr, false, &y) || !get_current_stream(a[11], &stream))
    Py_RETURN_NONE;
  return run([&] {
    return f_cluster_gemm_cw(codes, M, bits, wq, N, off.ints(), off.size() - 1, scale, cross, colterm, rowsums, y, y_dtype, stream);
  });
}

// (x, T, d, table, bits, codes, stream) and (codes, T, d, table, bits, out, stream)
PyObject* kv_call(PyObject* const* a, Py_ssize_t n, bool quant) {
  void *from, *table, *to, *stream;
  int32_t d, bits;
  int64_t T;
  if (n != 7 || (quant ? f_kv_quant == nullptr : f_kv_dequant == nullptr) ||
      !get_tensor(a[0], quant ? t_bf16 : nullptr, false, &from) || !get_i64(a[1], &T) || !get_i32(a[2], &d) ||
      !get_tensor(a[3], nullptr, false, &table) || !get_i32(a[4], &bits) ||
      !get_tensor(a[5], quant ? nullptr : t_bf16, false, &to) || !get_current_stream(a[6], &stream))
    Py_RETURN_NONE;
  return run([&] { return quant ? f_kv_quant(from, T, d, table, bits, to, stream) : f_kv_dequant(from, T, d, table, bits, to, stream); });
}
PyObject* kv_quant(PyObject*, PyObject* const* a, Py_ssize_t n) { return kv_call(a, n, true); }
PyObject* kv_dequant(PyObject*, PyObject* const* a, Py_ssize_t n) { return kv_call(a, n, false); }

template <typename F>
bool set_entry(PyObject* addresses, const char* name, F* f) {
  PyObject* o = PyDict_GetItemString(addresses, name);   // (borrowed)
  if (o == nullptr) {
    PyErr_Format(PyExc_KeyError, "%s", name);
    return false;
  }
  void* p = PyLong_AsVoidPtr(o);
  *f = reinterpret_cast<F>(p);
  return !PyErr_Occurred();
}

// setup({entry point: address}, {name: torch object}): called whenever a library is loaded.
PyObject* setup(PyObject*, PyObject* args) {
  PyObject *addresses, *objects;
  if (!PyArg_ParseTuple(args, "O!O!", &PyDict_Type, &addresses, &PyDict_Type, &objects)) return nullptr;
  const struct { const char* name; PyObject** at; } wanted[] = {
      {"bfloat16", &t_bf16}, {"float32", &t_f32}, {"int32", &t_i32}, {"get_device", &get_device}, {"get_stream", &get_stream}};
  for (const auto& w : wanted) {
    PyObject* o = PyDict_GetItemString(objects, w.name);
    if (o == nullptr) return PyErr_Format(PyExc_KeyError, "%s", w.name);
    Py_INCREF(o);
    Py_XSETREF(*w.at, o);
  }
  if (!set_entry(addresses, "rptq_ln_quant", &f_ln_quant) || !set_entry(addresses, "rptq_cluster_gemm", &f_cluster_gemm) ||
      !set_entry(addresses, "rptq_cluster_gemm_quant", &f_cluster_gemm_quant) ||
      !set_entry(addresses, "rptq_cluster_rowsums", &f_cluster_rowsums) ||
      !set_entry(addresses, "rptq_cluster_gemm_cw", &f_cluster_gemm_cw) || !set_entry(addresses, "rptq_kv_quant", &f_kv_quant) ||
      !set_entry(addresses, "rptq_kv_dequant", &f_kv_dequant))
    return nullptr;
  Py_RETURN_NONE;
}

#define RPTQ_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {RPTQ_METHOD(ln_quant), RPTQ_METHOD(cluster_gemm), RPTQ_METHOD(cluster_gemm_quant),
                         RPTQ_METHOD(cluster_rowsums), RPTQ_METHOD(cluster_gemm_cw), RPTQ_METHOD(kv_quant),
                         RPTQ_METHOD(kv_dequant), {"setup", setup, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  n_is_cuda = PyUnicode_InternFromString("is_cuda");
  n_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  n_dtype = PyUnicode_InternFromString("dtype");
  n_data_ptr = PyUnicode_InternFromString("data_ptr");
  n_nbytes = PyUnicode_InternFromString("nbytes");
  if (!n_is_cuda || !n_is_contiguous || !n_dtype || !n_data_ptr || !n_nbytes) return nullptr;
  return PyModule_Create(&module);
}
