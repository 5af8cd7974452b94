// Native marshalling of the Python binding: each function here takes the
// arguments of the mosaic.py function of the same name, checks the tensors
// as mosaic._need and mosaic._need_dig do, and calls the C ABI entry point on
// the current stream. It returns the entry point's status, or None for
// anything but a well-formed call (wrong types, sizes or strides, empty
// matrices, tensors without plain memory): the Python code then handles the
// call, and raises what is to be raised. A decode call is a handful of short
// kernels, and with every argument converted through ctypes and every check
// in Python a call of the ABI cost the host 10-12 us, more than most of those
// kernels run: one-token calls waited for the host. Here it costs 1 us beside
// the launches.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mosaic.h"
#include "dispatch.h"

namespace {

// Entry points of the loaded library, by address (set by bind()).
struct Abi {
  decltype(&mosaic_sample) sample;
  decltype(&mosaic_mask) mask;
  decltype(&mosaic_masked_matmul) masked_matmul;
  decltype(&mosaic_integrity_check) integrity_check;
  decltype(&mosaic_unmask) unmask;
  decltype(&mosaic_unmask_words) unmask_words;
  decltype(&mosaic_rotate_quantize_mask) rotate_quantize_mask;
  decltype(&mosaic_sparse_stream_gather_rows_terms) stream_terms;
  decltype(&mosaic_sparse_gather_cols_terms) cols_terms;
  decltype(&mosaic_sparse_gather_cols) gather_cols;
  decltype(&mosaic_hadamard_rotate) hadamard_rotate;
  decltype(&mosaic_quantize_rows) quantize_rows;
} abi;

PyObject *s_buf, *s_col0, *s_row_ptr, *s_col_idx, *s_values, *s_rows, *s_cols;   // interned attribute names
PyObject *get_device, *get_stream;                                               // torch._C functions
PyObject* rng_type;                                                              // the ctypes struct of mosaic_rng

struct Mat {
  void* p = nullptr;
  int64_t ld = 0;
  bool given() const { return p != nullptr; }
};

// A plain tensor on the device, or null.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
  return &t;
}

// A rows x cols matrix of dtype dt with contiguous rows, or None if optional.
bool matrix(PyObject* o, int64_t rows, int64_t cols, at::ScalarType dt, bool optional, Mat* m) {
  if (o == Py_None) return optional;
  const at::Tensor* t = plain(o);
  if (t == nullptr || t->dim() != 2 || t->scalar_type() != dt) return false;
  if (t->size(0) < rows || t->size(1) < cols || (cols > 1 && t->stride(1) != 1)) return false;
  m->p = t->data_ptr();
  m->ld = t->stride(0);
  return m->p != nullptr;
}

// A contiguous vector of n elements, or None if optional.
bool vec(PyObject* o, int64_t n, at::ScalarType dt, bool optional, Mat* m) {
  if (o == Py_None) return optional;
  const at::Tensor* t = plain(o);
  if (t == nullptr || t->dim() != 1 || t->scalar_type() != dt || t->size(0) < n || t->stride(0) != 1) return false;
  m->p = t->data_ptr();
  return m->p != nullptr;
}

// A Digits view that holds rows x cols, or None if optional.
bool digits(PyObject* o, int64_t rows, int64_t cols, bool optional, Mat* m) {
  if (o == Py_None) return optional;
  PyObject* b = PyObject_GetAttr(o, s_buf);
  PyObject* c = b != nullptr ? PyObject_GetAttr(o, s_col0) : nullptr;
  bool ok = false;
  if (c != nullptr && PyLong_CheckExact(c)) {
    const int64_t col0 = PyLong_AsLongLong(c);
    const at::Tensor* t = plain(b);
    if (t != nullptr && t->dim() == 2 && t->scalar_type() == at::kChar && t->stride(1) == 1 && t->size(0) >= rows &&
        col0 >= 0 && col0 % 64 == 0 && 4 * (col0 + 64 * ((cols + 63) / 64)) <= t->size(1)) {
      m->p = (char*)t->data_ptr() + 4 * col0;
      m->ld = t->size(1);
      ok = t->data_ptr() != nullptr;
    }
  }
  Py_XDECREF(b);     // its owner keeps the tensor
  Py_XDECREF(c);
  PyErr_Clear();
  return ok;
}

bool integer(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = PyLong_AsLongLong(o);
  if (*v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}
bool size(PyObject* o, int64_t* v) { return integer(o, v) && *v > 0; }

// The struct behind a ctypes MosaicRng (or None if optional), held while the
// object lives.
class Rng {
 public:
  bool get(PyObject* o, bool optional) {
    if (o == Py_None) return optional;
    if (!PyObject_TypeCheck(o, (PyTypeObject*)rng_type)) return false;
    if (PyObject_GetBuffer(o, &b_, PyBUF_SIMPLE) != 0) {
      PyErr_Clear();
      return false;
    }
    held_ = true;
    return b_.len == (Py_ssize_t)sizeof(mosaic_rng);
  }
  const mosaic_rng* p() const { return held_ ? (const mosaic_rng*)b_.buf : nullptr; }
  Rng() = default;
  Rng(const Rng&) = delete;
  Rng& operator=(const Rng&) = delete;
  ~Rng() {
    if (held_) PyBuffer_Release(&b_);
  }

 private:
  Py_buffer b_;
  bool held_ = false;
};

// The current stream of the current device.
bool current_stream(void** s) {
  PyObject* d = PyObject_CallNoArgs(get_device);
  PyObject* r = d != nullptr ? PyObject_CallOneArg(get_stream, d) : nullptr;
  Py_XDECREF(d);
  if (r == nullptr) {
    PyErr_Clear();
    return false;
  }
  *s = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  return true;
}

bool truth(PyObject* o, int32_t* v) {
  *v = PyObject_IsTrue(o);
  if (*v < 0) PyErr_Clear();
  return *v >= 0;
}

// The status of an ABI call, made without the interpreter lock: a launch may
// wait for room in its stream's queue, and other threads go on meanwhile (the
// caller's frame holds the arguments).
template <class Call>
PyObject* status(Call call) {
  int32_t st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

#define NEED(cond) \
  if (!(cond)) Py_RETURN_NONE
#define FUNCTION(name, count)                                                     \
  PyObject* name##_body(PyObject* const* a);                                      \
  PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) {                   \
    NEED(n == (count));                                                           \
    try {                                                                         \
      return name##_body(a);                                                      \
    } catch (...) { /* a tensor without memory of its own */                      \
      PyErr_Clear();                                                              \
      Py_RETURN_NONE;                                                             \
    }                                                                             \
  }                                                                               \
  PyObject* name##_body(PyObject* const* a)

// (r, rows, cols, out, out_dig)
FUNCTION(sample, 5) {
  Rng r;
  int64_t rows, cols;
  Mat out, dig;
  void* s;
  NEED(r.get(a[0], false) && size(a[1], &rows) && size(a[2], &cols));
  NEED(matrix(a[3], rows, cols, at::kInt, true, &out) && digits(a[4], rows, cols, true, &dig) && current_stream(&s));
  return status([&] {
    return abi.sample(r.p(), rows, cols, (uint32_t*)out.p, out.ld, (int8_t*)dig.p, dig.ld, s);
  });
}

// (x, u, noise, rows, cols, out, out_dig, x_transposed)
FUNCTION(mask, 8) {
  Rng noise;
  int64_t rows, cols;
  Mat u, out, dig;
  void *s, *xp = nullptr;
  int64_t rs = 0, cs = 0;
  int32_t dt = MOSAIC_U32;
  NEED(noise.get(a[2], true) && size(a[3], &rows) && size(a[4], &cols));
  if (a[0] != Py_None) {
    const at::Tensor* x = plain(a[0]);
    NEED(x != nullptr && x->dim() == 2);
    int32_t turned;
    NEED(truth(a[7], &turned));
    switch (x->scalar_type()) {
      case at::kChar: dt = MOSAIC_I8; break;
      case at::kShort: dt = MOSAIC_I16; break;
      case at::kInt: dt = MOSAIC_I32; break;
      default: Py_RETURN_NONE;
    }
    NEED(x->size(0) >= (turned ? cols : rows) && x->size(1) >= (turned ? rows : cols));
    rs = x->stride(turned ? 1 : 0);
    cs = x->stride(turned ? 0 : 1);
    xp = x->data_ptr();
    NEED(xp != nullptr);
  }
  NEED(matrix(a[1], rows, cols, at::kInt, true, &u) && matrix(a[5], rows, cols, at::kInt, true, &out) &&
       digits(a[6], rows, cols, true, &dig) && current_stream(&s));
  return status([&] {
    return abi.mask(xp, dt, rs, cs, (const uint32_t*)u.p, u.ld, noise.p(), rows, cols, (uint32_t*)out.p, out.ld,
                    (int8_t*)dig.p, dig.ld, s);
  });
}

// (a, b, M, N, K, c)
FUNCTION(masked_matmul, 6) {
  int64_t M, N, K;
  Mat x, y, c;
  void* s;
  NEED(size(a[2], &M) && size(a[3], &N) && size(a[4], &K));
  NEED(digits(a[0], M, K, false, &x) && digits(a[1], N, K, false, &y) && matrix(a[5], M, N, at::kInt, false, &c) &&
       current_stream(&s));
  return status([&] {
    return abi.masked_matmul((const int8_t*)x.p, x.ld, (const int8_t*)y.p, y.ld, M, N, K, (uint32_t*)c.p, c.ld, s);
  });
}

// (ct, a, v, yq, t, M, K, NR, d, count)
FUNCTION(integrity_check, 10) {
  int64_t t, M, K, NR;
  Mat ct, x, v, yq, d, count;
  void* s;
  NEED(size(a[4], &t) && size(a[5], &M) && size(a[6], &K) && size(a[7], &NR));
  NEED(digits(a[0], t, K, false, &ct) && digits(a[1], M, K, false, &x) && digits(a[2], t, NR, false, &v) &&
       matrix(a[3], M, NR, at::kInt, false, &yq) && matrix(a[8], t, M, at::kInt, false, &d) &&
       vec(a[9], 1, at::kLong, false, &count) && current_stream(&s));
  return status([&] {
    return abi.integrity_check((const int8_t*)ct.p, ct.ld, (const int8_t*)x.p, x.ld, (const int8_t*)v.p, v.ld,
                               (const uint32_t*)yq.p, yq.ld, t, M, K, NR, (uint32_t*)d.p, d.ld, (int64_t*)count.p, s);
  });
}

// Outputs of the unmask calls: y, s_rows, s_cols, y_f32, bias.
struct Outputs {
  Mat y, sr, sc, f, bias;
  bool get(PyObject* const* a, int64_t M, int64_t N) {
    return matrix(a[0], M, N, at::kInt, true, &y) && matrix(a[3], M, N, at::kFloat, true, &f) &&
           vec(a[1], M, at::kFloat, !f.given(), &sr) && vec(a[2], N, at::kFloat, !f.given(), &sc) &&
           vec(a[4], N, at::kFloat, true, &bias);
  }
};

// (ym, kc, q, l, M, N, R, y, s_rows, s_cols, y_f32, bias); q as digits
FUNCTION(unmask, 12) {
  int64_t M, N, R;
  Mat ym, kc, q, l;
  Outputs o;
  void* s;
  NEED(size(a[4], &M) && size(a[5], &N) && size(a[6], &R));
  NEED(matrix(a[0], M, N, at::kInt, false, &ym) && matrix(a[1], M, N, at::kInt, true, &kc) &&
       digits(a[2], M, R, false, &q) && digits(a[3], N, R, false, &l) && o.get(a + 7, M, N) && current_stream(&s));
  return status([&] {
    return abi.unmask((const uint32_t*)ym.p, ym.ld, (const uint32_t*)kc.p, kc.ld, (const int8_t*)q.p, q.ld,
                      (const int8_t*)l.p, l.ld, M, N, R, (int32_t*)o.y.p, o.y.ld, (const float*)o.sr.p,
                      (const float*)o.sc.p, (const float*)o.bias.p, (float*)o.f.p, o.f.ld, s);
  });
}

// the same with q as ring words
FUNCTION(unmask_words, 12) {
  int64_t M, N, R;
  Mat ym, kc, q, l;
  Outputs o;
  void* s;
  NEED(size(a[4], &M) && size(a[5], &N) && size(a[6], &R));
  NEED(matrix(a[0], M, N, at::kInt, false, &ym) && matrix(a[1], M, N, at::kInt, true, &kc) &&
       matrix(a[2], M, R, at::kInt, false, &q) && digits(a[3], N, R, false, &l) && o.get(a + 7, M, N) &&
       current_stream(&s));
  return status([&] {
    return abi.unmask_words((const uint32_t*)ym.p, ym.ld, (const uint32_t*)kc.p, kc.ld, (const uint32_t*)q.p, q.ld,
                            (const int8_t*)l.p, l.ld, M, N, R, (int32_t*)o.y.p, o.y.ld, (const float*)o.sr.p,
                            (const float*)o.sc.p, (const float*)o.bias.p, (float*)o.f.p, o.f.ld, s);
  });
}

// rows and columns of a float matrix that a pass reads whole
bool whole(PyObject* o, Mat* x, int64_t* rows, int64_t* n) {
  const at::Tensor* t = plain(o);
  if (t == nullptr || t->dim() != 2) return false;
  *rows = t->size(0);
  *n = t->size(1);
  return *rows > 0 && *n > 0 && matrix(o, *rows, *n, at::kFloat, false, x);
}

// (x, qmax, out_dig, block, signs, u, noise, scale)
FUNCTION(rotate_quantize_mask, 8) {
  int64_t rows, n, qmax, block;
  Mat x, dig, signs, u, scale;
  Rng noise;
  void* s;
  NEED(whole(a[0], &x, &rows, &n) && integer(a[1], &qmax) && qmax <= INT32_MAX && qmax >= INT32_MIN);
  block = n;
  NEED(a[3] == Py_None || integer(a[3], &block));
  NEED(digits(a[2], rows, n, false, &dig) && vec(a[4], n, at::kChar, true, &signs) &&
       matrix(a[5], rows, n, at::kInt, true, &u) && noise.get(a[6], true) && vec(a[7], rows, at::kFloat, true, &scale) &&
       current_stream(&s));
  return status([&] {
    return abi.rotate_quantize_mask((const float*)x.p, x.ld, rows, n, block, (const int8_t*)signs.p, (int32_t)qmax,
                                    (const uint32_t*)u.p, u.ld, noise.p(), (int8_t*)dig.p, dig.ld, (float*)scale.p, s);
  });
}

// (x, y, block, signs, inverse)
FUNCTION(hadamard_rotate, 5) {
  int64_t rows, n, block;
  int32_t inverse;
  Mat x, y, signs;
  void* s;
  NEED(whole(a[0], &x, &rows, &n));
  block = n;
  NEED(a[2] == Py_None || integer(a[2], &block));
  NEED(matrix(a[1], rows, n, at::kFloat, false, &y) && vec(a[3], n, at::kChar, true, &signs) &&
       truth(a[4], &inverse) && current_stream(&s));
  return status([&] {
    return abi.hadamard_rotate((const float*)x.p, x.ld, (float*)y.p, y.ld, rows, n, block, (const int8_t*)signs.p,
                               inverse, s);
  });
}

// (x, qmax, q, q_dig, scale)
FUNCTION(quantize_rows, 5) {
  int64_t rows, n, qmax;
  Mat x, q, dig, scale;
  void* s;
  NEED(whole(a[0], &x, &rows, &n) && integer(a[1], &qmax) && qmax <= INT32_MAX && qmax >= INT32_MIN);
  NEED(matrix(a[2], rows, n, at::kInt, true, &q) && digits(a[3], rows, n, true, &dig) &&
       vec(a[4], rows, at::kFloat, true, &scale) && current_stream(&s));
  return status([&] {
    return abi.quantize_rows((const float*)x.p, x.ld, rows, n, (int32_t)qmax, (int32_t*)q.p, q.ld, (int8_t*)dig.p,
                             dig.ld, (float*)scale.p, s);
  });
}

constexpr int kMaxTerms = 4;

// (terms, rows, ncols, c, subtract); a term is a tuple (r, rcols, d)
FUNCTION(stream_terms, 5) {
  int64_t rows, ncols;
  int32_t subtract;
  Mat c;
  void* s;
  NEED(PyList_CheckExact(a[0]) && size(a[1], &rows) && size(a[2], &ncols) &&
       matrix(a[3], rows, ncols, at::kInt, false, &c));
  const Py_ssize_t n = PyList_GET_SIZE(a[0]);
  NEED(n >= 1 && n <= kMaxTerms);
  mosaic_stream_term terms[kMaxTerms];
  for (Py_ssize_t l = 0; l < n; ++l) {
    PyObject* t = PyList_GET_ITEM(a[0], l);
    Rng r;
    Mat d;
    int64_t rcols;
    NEED(PyTuple_CheckExact(t) && PyTuple_GET_SIZE(t) == 3 && r.get(PyTuple_GET_ITEM(t, 0), false) &&
         size(PyTuple_GET_ITEM(t, 1), &rcols) && matrix(PyTuple_GET_ITEM(t, 2), rcols, ncols, at::kInt, false, &d));
    terms[l] = mosaic_stream_term{*r.p(), rcols, (const uint32_t*)d.p, d.ld};
  }
  NEED(truth(a[4], &subtract) && current_stream(&s));
  return status([&] {
    return abi.stream_terms(terms, (int32_t)n, rows, ncols, (uint32_t*)c.p, c.ld, subtract, s);
  });
}

bool attr_ptr(PyObject* o, PyObject* name, at::ScalarType dt, const void** p, int64_t* n = nullptr) {
  PyObject* v = PyObject_GetAttr(o, name);
  const at::Tensor* t = v != nullptr ? plain(v) : nullptr;
  const bool ok = t != nullptr && t->dim() == 1 && t->scalar_type() == dt && t->stride(0) == 1;
  if (ok) *p = t->data_ptr();
  if (ok && n != nullptr) *n = t->size(0);
  Py_XDECREF(v);
  PyErr_Clear();
  return ok && *p != nullptr;
}

bool attr_size(PyObject* o, PyObject* name, int64_t* n) {
  PyObject* v = PyObject_GetAttr(o, name);
  const bool ok = v != nullptr && size(v, n);
  Py_XDECREF(v);
  PyErr_Clear();
  return ok;
}

// (terms, M, c, subtract, y_f32, s_rows, s_cols, bias); a term is a tuple
// (SparseRows, d)
FUNCTION(cols_terms, 8) {
  int64_t M, N = 0, all_cols = 0, all_entries = 0;
  int32_t subtract;
  void* s;
  NEED(PyList_CheckExact(a[0]) && size(a[1], &M));
  const Py_ssize_t n = PyList_GET_SIZE(a[0]);
  NEED(n >= 1 && n <= kMaxTerms);
  mosaic_sparse_term terms[kMaxTerms];
  for (Py_ssize_t l = 0; l < n; ++l) {
    PyObject* t = PyList_GET_ITEM(a[0], l);
    NEED(PyTuple_CheckExact(t) && PyTuple_GET_SIZE(t) == 2);
    PyObject* p = PyTuple_GET_ITEM(t, 0);
    int64_t rows, cols, capacity = 0;
    const void *rp, *ci, *va;
    Mat d;
    NEED(attr_size(p, s_rows, &rows) && attr_size(p, s_cols, &cols) && (l == 0 || rows == N));
    N = rows;
    NEED(attr_ptr(p, s_row_ptr, at::kLong, &rp) && attr_ptr(p, s_col_idx, at::kInt, &ci) &&
         attr_ptr(p, s_values, at::kInt, &va, &capacity) && matrix(PyTuple_GET_ITEM(t, 1), M, cols, at::kInt, false, &d));
    terms[l] = mosaic_sparse_term{(const int64_t*)rp, (const int32_t*)ci, (const uint32_t*)va, cols,
                                  (const uint32_t*)d.p, d.ld};
    all_cols += cols;
    all_entries += capacity / rows;     // the arrays hold at least the entries
  }
  Mat c, f, sr, sc, bias;
  NEED(matrix(a[2], M, N, at::kInt, false, &c) && matrix(a[4], M, N, at::kFloat, true, &f) &&
       vec(a[5], M, at::kFloat, !f.given(), &sr) && vec(a[6], N, at::kFloat, !f.given(), &sc) &&
       vec(a[7], N, at::kFloat, true, &bias) && truth(a[3], &subtract) && current_stream(&s));
  // outputs that the last call would refuse are refused before the first has added anything
  const bool outputs_ok = f.given() ? f.ld >= N : !bias.given();
  if (outputs_ok && mosaic::gather_cols_sparse((int)n, M, N, all_cols, all_entries))
    return status([&] {
      for (Py_ssize_t l = 0; l < n; ++l) {
        const mosaic_sparse_term& t = terms[l];
        const bool last = l + 1 == n;     // which also writes the dequantised output
        const mosaic_status st = abi.gather_cols(
            M, N, t.row_ptr, t.col_idx, t.values, t.d, t.ldd, (uint32_t*)c.p, c.ld, subtract,
            last ? (const float*)sr.p : nullptr, last ? (const float*)sc.p : nullptr,
            last ? (const float*)bias.p : nullptr, last ? (float*)f.p : nullptr, last ? f.ld : 0, s);
        if (st != MOSAIC_OK) return st;
      }
      return MOSAIC_OK;
    });
  return status([&] {
    return abi.cols_terms(terms, (int32_t)n, M, N, (uint32_t*)c.p, c.ld, subtract, (const float*)sr.p,
                          (const float*)sc.p, (const float*)bias.p, (float*)f.p, f.ld, s);
  });
}

// bind(addresses, get_device, get_stream, rng_type): addresses of the library's
// entry points in the order of Abi; torch._C's current device and raw stream;
// the type that generators are of.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr Py_ssize_t count = sizeof(Abi) / sizeof(void*);
  if (n != 4 || !PyTuple_CheckExact(a[0]) || PyTuple_GET_SIZE(a[0]) != count || !PyType_Check(a[3])) {
    PyErr_Format(PyExc_TypeError, "bind takes a tuple of %zd addresses, two functions and a type", count);
    return nullptr;
  }
  void* p[count];
  for (Py_ssize_t i = 0; i < count; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[0], i));
    if (p[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  memcpy(&abi, p, sizeof(p));
  PyObject** const kept[] = {&get_device, &get_stream, &rng_type};
  for (int i = 0; i < 3; ++i) {
    PyObject* const old = *kept[i];
    Py_INCREF(a[1 + i]);
    *kept[i] = a[1 + i];
    Py_XDECREF(old);
  }
  Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind), METHOD(sample), METHOD(mask), METHOD(masked_matmul), METHOD(integrity_check),
                         METHOD(unmask), METHOD(unmask_words), METHOD(rotate_quantize_mask), METHOD(hadamard_rotate),
                         METHOD(quantize_rows), METHOD(stream_terms), METHOD(cols_terms), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  s_buf = PyUnicode_InternFromString("buf");
  s_col0 = PyUnicode_InternFromString("col0");
  s_row_ptr = PyUnicode_InternFromString("row_ptr");
  s_col_idx = PyUnicode_InternFromString("col_idx");
  s_values = PyUnicode_InternFromString("values");
  s_rows = PyUnicode_InternFromString("rows");
  s_cols = PyUnicode_InternFromString("cols");
  if (!s_buf || !s_col0 || !s_row_ptr || !s_col_idx || !s_values || !s_rows || !s_cols) return nullptr;
  return PyModule_Create(&module);
}
