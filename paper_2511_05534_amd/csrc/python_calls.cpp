// The calls of libflowmm.so (include/flowmm.h) as a CPython extension module: arguments are taken apart
// here instead of by ctypes.  A call that enqueues one small kernel costs about as much on the host as on
// the GPU (a cache append: 10.7 us a call through ctypes and numpy, of which the launch itself is 3), so
// the path from a Python program to the launch counts.  Pointers arrive as Python ints (None is NULL), the
// parameters as the address of a flowmm_params; every function returns the flowmm_status.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <climits>

#include "../../include/flowmm.h"

namespace {

// integer of a Python int, or of anything that converts to one; false with an exception set
bool as_int64(PyObject *o, long long *v) {
  if (PyLong_CheckExact(o)) {
    *v = PyLong_AsLongLong(o);
  } else {
    PyObject *i = PyNumber_Long(o);
    if (!i) return false;
    *v = PyLong_AsLongLong(i);
    Py_DECREF(i);
  }
  return !(*v == -1 && PyErr_Occurred());
}

template <typename T>
bool as_pointer(PyObject *o, T **p) {
  if (o == Py_None) { *p = nullptr; return true; }
  PyObject *i = PyNumber_Index(o);  // integers only: an address is never a float or a text
  if (!i) return false;
  *p = reinterpret_cast<T *>(PyLong_AsUnsignedLongLongMask(i));
  Py_DECREF(i);
  return !PyErr_Occurred();
}

bool as_size(PyObject *o, size_t *v) {
  PyObject *i = PyNumber_Index(o);
  if (!i) return false;
  *v = (size_t)PyLong_AsUnsignedLongLongMask(i);
  Py_DECREF(i);
  return !PyErr_Occurred();
}

bool as_int32(PyObject *o, int32_t *v) {
  long long x;
  if (!as_int64(o, &x)) return false;
  if (x < INT32_MIN || x > INT32_MAX) { PyErr_SetString(PyExc_OverflowError, "integer does not fit 32 bits"); return false; }
  *v = (int32_t)x;
  return true;
}

// Integers as an int32 array (few of them without an allocation): a list or tuple of ints directly, everything else as
// numpy.asarray(.., int32) reads it.  Fewer than the call reads are refused here: the library gets no count.
class Ints {
 public:
  ~Ints() { if (data_ != small_) PyMem_Free(data_); }
  bool take(PyObject *o, Py_ssize_t least, const char *name) {
    int got = PyList_CheckExact(o) || PyTuple_CheckExact(o) ? copy(o) : 0;
    if (got == 0) {
      PyObject *flat = through_numpy(o);
      if (!flat) return false;
      got = copy(flat);
      Py_DECREF(flat);
    }
    if (got < 0) return false;
    if (n_ >= least) return true;
    PyErr_Format(PyExc_ValueError, "%s has %zd entries, %zd expected", name, n_, least);
    return false;
  }
  const int32_t *data() const { return data_; }

 private:
  static constexpr Py_ssize_t kSmall = 128;
  // 1: done, 0: not all of them are plain ints, -1: an exception is set
  int copy(PyObject *seq) {
    PyObject **it = PySequence_Fast_ITEMS(seq);
    n_ = PySequence_Fast_GET_SIZE(seq);
    for (Py_ssize_t i = 0; i < n_; ++i)
      if (!PyLong_CheckExact(it[i])) return 0;
    if (n_ > kSmall && !(data_ = static_cast<int32_t *>(PyMem_Malloc((size_t)n_ * sizeof(int32_t))))) {
      data_ = small_;
      PyErr_NoMemory();
      return -1;
    }
    for (Py_ssize_t i = 0; i < n_; ++i)
      if (!as_int32(it[i], &data_[i])) return -1;
    return 1;
  }
  static PyObject *through_numpy(PyObject *o) {
    PyObject *np = PyImport_ImportModule("numpy");
    PyObject *array = np ? PyObject_CallMethod(np, "asarray", "Os", o, "int32") : nullptr;
    PyObject *flat = array ? PyObject_CallMethod(array, "ravel", nullptr) : nullptr;
    PyObject *list = flat ? PyObject_CallMethod(flat, "tolist", nullptr) : nullptr;
    Py_XDECREF(flat);
    Py_XDECREF(array);
    Py_XDECREF(np);
    return list;
  }
  int32_t small_[kSmall];
  int32_t *data_ = small_;
  Py_ssize_t n_ = 0;
};

// sequences of the call that the parameters describe (0 where the library will refuse them)
Py_ssize_t sequences(const flowmm_params *p) { return p && p->batch > 0 ? p->batch : 0; }

bool as_plan(PyObject *o, flowmm_plan_buffers *b) {
  PyObject *seq = PySequence_Fast(o, "the six plan pointers are expected");
  if (!seq) return false;
  bool ok = PySequence_Fast_GET_SIZE(seq) == 6;
  if (!ok) PyErr_SetString(PyExc_ValueError, "the six plan pointers are expected");
  PyObject **it = PySequence_Fast_ITEMS(seq);
  ok = ok && as_pointer(it[0], &b->importance) && as_pointer(it[1], &b->rho) && as_pointer(it[2], &b->mode) &&
       as_pointer(it[3], &b->kept_idx) && as_pointer(it[4], &b->assign) && as_pointer(it[5], &b->n_dropped);
  Py_DECREF(seq);
  return ok;
}

bool count(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, n);
  return false;
}

// the call itself, without the interpreter lock (the library keeps no Python state)
template <typename F>
PyObject *call(F f) {
  flowmm_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

using Args = PyObject *const *;

// (params, K, Q_window, plan, workspace, workspace_bytes, stream)
PyObject *plan(PyObject *, Args a, Py_ssize_t n) {
  const flowmm_params *p; const void *K, *Q; flowmm_plan_buffers b; void *ws, *stream; size_t bytes;
  if (!count(n, 7) || !as_pointer(a[0], &p) || !as_pointer(a[1], &K) || !as_pointer(a[2], &Q) || !as_plan(a[3], &b) ||
      !as_pointer(a[4], &ws) || !as_size(a[5], &bytes) || !as_pointer(a[6], &stream)) return nullptr;
  return call([&] { return flowmm_plan(p, K, Q, &b, ws, bytes, stream); });
}

// (params, plan, K, V, K_out, V_out, workspace, workspace_bytes, stream)
PyObject *merge(PyObject *, Args a, Py_ssize_t n) {
  const flowmm_params *p; const void *K, *V; flowmm_plan_buffers b; void *Ko, *Vo, *ws, *stream; size_t bytes;
  if (!count(n, 9) || !as_pointer(a[0], &p) || !as_plan(a[1], &b) || !as_pointer(a[2], &K) || !as_pointer(a[3], &V) ||
      !as_pointer(a[4], &Ko) || !as_pointer(a[5], &Vo) || !as_pointer(a[6], &ws) || !as_size(a[7], &bytes) ||
      !as_pointer(a[8], &stream)) return nullptr;
  return call([&] { return flowmm_merge(p, &b, K, V, Ko, Vo, ws, bytes, stream); });
}

// (params, K, V, Q_window, plan, K_out, V_out, workspace, workspace_bytes, stream)
PyObject *plan_merge(PyObject *, Args a, Py_ssize_t n) {
  const flowmm_params *p; const void *K, *V, *Q; flowmm_plan_buffers b; void *Ko, *Vo, *ws, *stream; size_t bytes;
  if (!count(n, 10) || !as_pointer(a[0], &p) || !as_pointer(a[1], &K) || !as_pointer(a[2], &V) || !as_pointer(a[3], &Q) ||
      !as_plan(a[4], &b) || !as_pointer(a[5], &Ko) || !as_pointer(a[6], &Vo) || !as_pointer(a[7], &ws) || !as_size(a[8], &bytes) ||
      !as_pointer(a[9], &stream)) return nullptr;
  return call([&] { return flowmm_plan_merge(p, K, V, Q, &b, Ko, Vo, ws, bytes, stream); });
}

// (params, K, V, Q_window, plan, K_out, V_out, stream)
PyObject *plan_merge_static(PyObject *, Args a, Py_ssize_t n) {
  const flowmm_params *p; const void *K, *V, *Q; flowmm_plan_buffers b; void *Ko, *Vo, *stream;
  if (!count(n, 8) || !as_pointer(a[0], &p) || !as_pointer(a[1], &K) || !as_pointer(a[2], &V) || !as_pointer(a[3], &Q) ||
      !as_plan(a[4], &b) || !as_pointer(a[5], &Ko) || !as_pointer(a[6], &Vo) || !as_pointer(a[7], &stream)) return nullptr;
  return call([&] { return flowmm_plan_merge_static(p, K, V, Q, &b, Ko, Vo, stream); });
}

// (params, q, K_c, V_c, out, workspace, workspace_bytes, stream)
PyObject *decode_attention(PyObject *, Args a, Py_ssize_t n) {
  const flowmm_params *p; const void *q, *K, *V; void *out, *ws, *stream; size_t bytes;
  if (!count(n, 8) || !as_pointer(a[0], &p) || !as_pointer(a[1], &q) || !as_pointer(a[2], &K) || !as_pointer(a[3], &V) ||
      !as_pointer(a[4], &out) || !as_pointer(a[5], &ws) || !as_size(a[6], &bytes) || !as_pointer(a[7], &stream)) return nullptr;
  return call([&] { return flowmm_decode_attention(p, q, K, V, out, ws, bytes, stream); });
}

// (params, cu_capacity, lengths, K_c, V_c, k_new, v_new, stream)
PyObject *cache_append(PyObject *, Args a, Py_ssize_t n) {
  const flowmm_params *p; Ints cu, len; void *K, *V, *stream; const void *k, *v;
  if (!count(n, 8) || !as_pointer(a[0], &p) || !cu.take(a[1], sequences(p) + 1, "cu_capacity") || !len.take(a[2], sequences(p), "lengths") ||
      !as_pointer(a[3], &K) || !as_pointer(a[4], &V) || !as_pointer(a[5], &k) || !as_pointer(a[6], &v) || !as_pointer(a[7], &stream)) return nullptr;
  return call([&] { return flowmm_cache_append(p, cu.data(), len.data(), K, V, k, v, stream); });
}

// (params, cu_capacity, lengths, seq, K_c, V_c, Q_window, plan, workspace, workspace_bytes, stream)
PyObject *cache_remerge(PyObject *, Args a, Py_ssize_t n) {
  const flowmm_params *p; Ints cu, len; int32_t seq; void *K, *V, *ws, *stream; const void *Q; flowmm_plan_buffers b; size_t bytes;
  if (!count(n, 11) || !as_pointer(a[0], &p) || !cu.take(a[1], sequences(p) + 1, "cu_capacity") || !len.take(a[2], sequences(p), "lengths") ||
      !as_int32(a[3], &seq) || !as_pointer(a[4], &K) || !as_pointer(a[5], &V) || !as_pointer(a[6], &Q) || !as_plan(a[7], &b) || !as_pointer(a[8], &ws) || !as_size(a[9], &bytes) ||
      !as_pointer(a[10], &stream)) return nullptr;
  return call([&] { return flowmm_cache_remerge(p, cu.data(), len.data(), seq, K, V, Q, &b, ws, bytes, stream); });
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(plan), METHOD(merge), METHOD(plan_merge), METHOD(plan_merge_static), METHOD(decode_attention),
                         METHOD(cache_append), METHOD(cache_remerge), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_flowmm_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__flowmm_calls(void) { return PyModule_Create(&module); }
