// Native half of the Python binding (binding.py): checks a call's tensors
// against what the library will address and makes the call, without the
// Python-level checks and the foreign-function marshalling (together about
// 9 us a decode call, against 1 us here).
//
// Each function takes the arguments of the binding.py function of its name,
// all positional, and returns the library's status, or None where it cannot
// vouch for an argument (another type than expected, a failed check, a number
// outside the C type): binding.py then runs its own checks, which raise what
// is to be raised or make the call themselves.  Nothing is kept between calls
// but the library's entry points and torch's stream query.
#include <Python.h>

#include <climits>
#include <cstdint>

#include <torch/csrc/autograd/python_variable.h>

#include "sckv.h"

namespace {

PyObject* g_raw_stream = nullptr;  // device index -> the current stream's handle

#define ENTRY(name) decltype(&::name) p_##name = nullptr;
#define ENTRIES(X)                                                                               \
  X(compacted_decode_attn) X(compacted_decode_attn_noalloc) X(local_decode_attn) X(kv_commit)    \
  X(kv_extend) X(kv_start) X(kv_compact) X(rope_apply) X(rope_apply_at) X(rope_block)            \
  X(span_masked_prefill_attn)                                                                    \
  X(span_masked_prefill_attn_planned) X(span_masked_prefill_attn_cached)                         \
  X(span_masked_prefill_attn_cached_planned) X(sckv_prefill_plan) X(sckv_prefill_cached_plan)
ENTRIES(ENTRY)
#undef ENTRY

// thrown where binding.py has to take over
struct Defer {};

// The arguments of one call, taken in order.
class Args {
 public:
  Args(PyObject* const* a, Py_ssize_t n, Py_ssize_t want) : a_(a) {
    if (n != want) throw Defer();
  }
  int32_t i32() {
    const int64_t v = i64();
    if (v < INT32_MIN || v > INT32_MAX) throw Defer();
    return (int32_t)v;
  }
  int64_t i64() {
    PyObject* o = a_[at_++];
    if (!PyLong_Check(o)) throw Defer();
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    if (over) throw Defer();
    return v;
  }
  double f64() {
    PyObject* o = a_[at_++];
    if (PyFloat_Check(o)) return PyFloat_AS_DOUBLE(o);
    if (!PyLong_Check(o)) throw Defer();
    const double v = PyLong_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Defer();
    return v;
  }
  float f32() { return (float)f64(); }
  // a tensor on a GPU; null for None
  const at::Tensor* tensor() {
    PyObject* o = a_[at_++];
    if (o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) throw Defer();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.has_storage()) throw Defer();
    return &t;
  }
  // the stream argument, or the current stream of t's device
  hipStream_t stream(const at::Tensor* t) {
    PyObject* o = a_[at_++];
    void* p = nullptr;
    if (o == Py_None) {
      PyObject* dev = PyLong_FromLong(t->get_device());
      PyObject* r = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
      Py_XDECREF(dev);
      if (!r) throw Defer();
      p = PyLong_AsVoidPtr(r);
      Py_DECREF(r);
    } else {
      if (!PyLong_Check(o)) throw Defer();
      p = PyLong_AsVoidPtr(o);
    }
    if (!p && PyErr_Occurred()) throw Defer();
    return (hipStream_t)p;
  }

 private:
  PyObject* const* a_;
  Py_ssize_t at_ = 0;
};

int64_t available(const at::Tensor& t) {
  return (int64_t)(t.storage().nbytes() / t.element_size()) - t.storage_offset();
}

void* address(const at::Tensor& t) { return t.mutable_data_ptr(); }

// a contiguous int32 array of at least `need` elements (null only if allowed)
int32_t* ints(const at::Tensor* t, int64_t need, bool nullable = false) {
  if (!t) {
    if (nullable) return nullptr;
    throw Defer();
  }
  if (t->scalar_type() != at::kInt || !t->is_contiguous() || need > t->numel()) throw Defer();
  return (int32_t*)address(*t);
}

// the status word: int32, one element in its storage (null allowed)
int32_t* word(const at::Tensor* t) {
  if (!t) return nullptr;
  if (t->scalar_type() != at::kInt || available(*t) < 1) throw Defer();
  return (int32_t*)address(*t);
}

sckv_dtype type_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return SCKV_F32;
  if (t.scalar_type() == at::kBFloat16) return SCKV_BF16;
  throw Defer();
}

// a contiguous array of `like`'s type with at least `need` elements
void* floats(const at::Tensor* t, int64_t need, sckv_dtype like) {
  if (!t || type_code(*t) != like || !t->is_contiguous() || need > t->numel()) throw Defer();
  return address(*t);
}

// (b, H, n, d) slices with (b, h) stride `stride` (see _rows of binding.py)
void* rows(const at::Tensor* t, int64_t b, int64_t H, int64_t n, int64_t d, int64_t stride,
           sckv_dtype like) {
  if (!t || type_code(*t) != like) throw Defer();
  if (b < 0 || H < 0 || n < 0 || d < 0 || stride < 0) throw Defer();
  if (t->dim() == 4 && t->size(0) == b && t->size(1) == H) {
    if ((n > 1 && t->stride(2) != d) || t->stride(3) != 1) throw Defer();
    if ((H > 1 && t->stride(1) != stride) || (b > 1 && t->stride(0) != H * stride)) throw Defer();
  } else if (!t->is_contiguous()) {
    throw Defer();
  }
  if (b * H > 0 && n > 0 && (b * H - 1) * (__int128)stride + n * (__int128)d > available(*t))
    throw Defer();
  return address(*t);
}

struct Work {
  void* p;
  size_t n;
};
Work workspace(const at::Tensor* t) {
  if (!t || !t->is_contiguous()) throw Defer();
  return {address(*t), (size_t)t->numel() * t->element_size()};
}

// b * H * L * d and the like; Defer where it leaves 62 bits
int64_t times(std::initializer_list<int64_t> f) {
  __int128 v = 1;
  for (int64_t x : f) {
    v *= x;
    if (v < 0 || v > ((__int128)1 << 62)) throw Defer();
  }
  return (int64_t)v;
}

template <typename F>
PyObject* status_of(F call) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

enum DecodeKind { WITH_WS, NOALLOC, LOCAL };

template <DecodeKind KIND>
PyObject* decode(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, KIND == NOALLOC ? 19 : 20);
  const at::Tensor *q = g.tensor(), *kn = g.tensor(), *vn = g.tensor(), *kc = g.tensor(),
                   *vc = g.tensor(), *kv_len = nullptr;
  int32_t W = 0;
  if (KIND == LOCAL) W = g.i32();
  else kv_len = g.tensor();
  const at::Tensor *cur = g.tensor(), *vu = g.tensor(), *pos = g.tensor();
  const int32_t L_meta = g.i32();
  const at::Tensor* o = g.tensor();
  const int32_t b = g.i32(), H = g.i32(), L_cap = g.i32(), d = g.i32();
  const float scale = g.f32();
  const double theta_in = g.f64();  // 0 by value, not by its rounding: pos is needed otherwise
  const float theta = (float)theta_in;
  const at::Tensor* ws = KIND == NOALLOC ? nullptr : g.tensor();
  const at::Tensor* st = g.tensor();
  if (!q) throw Defer();
  const hipStream_t stream = g.stream(q);
  const sckv_dtype dt = type_code(*q);
  const int64_t nh = times({b, H, d}), nc = times({b, H, L_cap, d}), nm = times({b, L_meta});
  void *pq = floats(q, nh, dt), *pkn = floats(kn, nh, dt), *pvn = floats(vn, nh, dt),
       *pkc = floats(kc, nc, dt), *pvc = floats(vc, nc, dt), *po = floats(o, nh, dt);
  const int32_t *pvu = ints(vu, nm), *ppos = ints(pos, nm, theta_in == 0.0), *pcur = ints(cur, b);
  int32_t* pst = word(st);
  if (KIND == LOCAL) {
    const Work w = workspace(ws);
    return status_of([&] {
      return p_local_decode_attn(pq, pkn, pvn, pkc, pvc, W, pcur, pvu, ppos, L_meta, po, b, H,
                                 L_cap, d, dt, scale, theta, w.p, w.n, pst, stream);
    });
  }
  const int32_t* plen = ints(kv_len, b);
  if (KIND == NOALLOC)
    return status_of([&] {
      return p_compacted_decode_attn_noalloc(pq, pkn, pvn, pkc, pvc, plen, pcur, pvu, ppos,
                                             L_meta, po, b, H, L_cap, d, dt, scale, theta, pst,
                                             stream);
    });
  const Work w = workspace(ws);
  return status_of([&] {
    return p_compacted_decode_attn(pq, pkn, pvn, pkc, pvc, plen, pcur, pvu, ppos, L_meta, po, b,
                                   H, L_cap, d, dt, scale, theta, w.p, w.n, pst, stream);
  });
}

PyObject* commit(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 11);
  const at::Tensor *len = g.tensor(), *tok = g.tensor(), *ids = g.tensor(), *cur = g.tensor(),
                   *vu = g.tensor(), *pos = g.tensor();
  const int32_t L_meta = g.i32(), b = g.i32(), L_cap = g.i32();
  const at::Tensor* st = g.tensor();
  const int64_t nc = times({b, L_cap}), nm = times({b, L_meta});
  int32_t *plen = ints(len, b), *ptok = ints(tok, nc), *pids = ints(ids, nc), *pcur = ints(cur, b),
          *pvu = ints(vu, nm), *ppos = ints(pos, nm), *pst = word(st);
  const hipStream_t stream = g.stream(len);
  return status_of([&] {
    return p_kv_commit(plen, ptok, pids, pcur, pvu, ppos, L_meta, b, L_cap, pst, stream);
  });
}

PyObject* extend(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 12);
  const at::Tensor *len = g.tensor(), *tok = g.tensor(), *ids = g.tensor(), *row0 = g.tensor(),
                   *pos = g.tensor();
  const int32_t L_meta = g.i32(), tok0 = g.i32(), rows_ = g.i32(), b = g.i32(), L_cap = g.i32();
  const at::Tensor* st = g.tensor();
  const int64_t nc = times({b, L_cap});
  int32_t *plen = ints(len, b), *ptok = ints(tok, nc), *pids = ints(ids, nc),
          *prow = ints(row0, b), *ppos = ints(pos, times({b, L_meta})), *pst = word(st);
  const hipStream_t stream = g.stream(len);
  return status_of([&] {
    return p_kv_extend(plen, ptok, pids, prow, ppos, L_meta, tok0, rows_, b, L_cap, pst, stream);
  });
}

PyObject* compact(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 15);
  const at::Tensor *kv = g.tensor(), *out = g.tensor();
  const int32_t M = g.i32(), b = g.i32(), H = g.i32(), L_cap = g.i32(), d = g.i32();
  const at::Tensor *len = g.tensor(), *tok = g.tensor(), *ids = g.tensor(), *next = g.tensor(),
                   *vu = g.tensor();
  const int32_t L_meta = g.i32();
  const at::Tensor* src = g.tensor();
  if (!kv) throw Defer();
  const sckv_dtype dt = type_code(*kv);
  const int64_t all = times({M, 2, b, H, L_cap, d}), nc = times({b, L_cap});
  void *pkv = floats(kv, all, dt), *pout = out ? floats(out, all, dt) : nullptr;
  int32_t *plen = ints(len, b), *ptok = ints(tok, nc), *pids = ints(ids, nc), *pnext = ints(next, b),
          *pvu = ints(vu, times({b, L_meta})), *psrc = ints(src, nc);
  const hipStream_t stream = g.stream(kv);
  return status_of([&] {
    return p_kv_compact(pkv, pout, M, b, H, L_cap, d, dt, plen, ptok, pids, pnext, pvu, L_meta,
                        psrc, stream);
  });
}

template <bool AT>
PyObject* rope(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, AT ? 16 : 13);
  const at::Tensor *x = g.tensor(), *y = g.tensor(), *row0 = AT ? g.tensor() : nullptr;
  const int32_t y_rows = AT ? g.i32() : 0;
  const int32_t b = g.i32(), H = g.i32(), rows_ = g.i32();
  const int64_t xs = g.i64(), ys = g.i64();
  const int32_t d = g.i32();
  const at::Tensor* pos = g.tensor();
  const int32_t L_meta = g.i32(), tok0 = g.i32();
  const double theta_in = g.f64();
  const float theta = (float)theta_in;
  const at::Tensor* st = AT ? g.tensor() : nullptr;
  if (!x) throw Defer();
  const sckv_dtype dt = type_code(*x);
  void *px = rows(x, b, H, rows_, d, xs, dt), *py = rows(y, b, H, AT ? y_rows : rows_, d, ys, dt);
  const int32_t* ppos = ints(pos, times({b, L_meta}), theta_in == 0.0);
  const int32_t* prow = AT ? ints(row0, b) : nullptr;
  int32_t* pst = word(st);
  const hipStream_t stream = g.stream(x);
  return status_of([&] {
    return AT ? p_rope_apply_at(px, py, prow, y_rows, b, H, rows_, xs, ys, d, dt, ppos, L_meta,
                                tok0, theta, pst, stream)
              : p_rope_apply(px, py, b, H, rows_, xs, ys, d, dt, ppos, L_meta, tok0, theta, stream);
  });
}

PyObject* block(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 23);
  const at::Tensor *q = g.tensor(), *k = g.tensor(), *v = g.tensor(), *qr = g.tensor(),
                   *kc = g.tensor(), *vc = g.tensor(), *row0 = g.tensor();
  const int32_t L_cap = g.i32(), b = g.i32(), H = g.i32(), rows_ = g.i32();
  const int64_t qs = g.i64(), ks = g.i64(), vs = g.i64(), qrs = g.i64(), cs = g.i64();
  const int32_t d = g.i32();
  const at::Tensor* pos = g.tensor();
  const int32_t L_meta = g.i32(), tok0 = g.i32();
  const double theta_in = g.f64();
  const float theta = (float)theta_in;
  const at::Tensor* st = g.tensor();
  if (!q) throw Defer();
  const sckv_dtype dt = type_code(*q);
  void *pq = rows(q, b, H, rows_, d, qs, dt), *pk = rows(k, b, H, rows_, d, ks, dt),
       *pv = rows(v, b, H, rows_, d, vs, dt), *pr = rows(qr, b, H, rows_, d, qrs, dt),
       *pkc = rows(kc, b, H, L_cap, d, cs, dt), *pvc = rows(vc, b, H, L_cap, d, cs, dt);
  const int32_t *ppos = ints(pos, times({b, L_meta}), theta_in == 0.0), *prow = ints(row0, b);
  int32_t* pst = word(st);
  const hipStream_t stream = g.stream(q);
  return status_of([&] {
    return p_rope_block(pq, pk, pv, pr, pkc, pvc, prow, L_cap, b, H, rows_, qs, ks, vs, qrs, cs, d,
                        dt, ppos, L_meta, tok0, theta, pst, stream);
  });
}

PyObject* start(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 10);
  const at::Tensor *len = g.tensor(), *tok = g.tensor(), *ids = g.tensor(), *cur = g.tensor(),
                   *pos = g.tensor();
  const int32_t L_meta = g.i32(), rows_ = g.i32(), b = g.i32(), L_cap = g.i32();
  const int64_t nc = times({b, L_cap});
  int32_t *plen = ints(len, b), *ptok = ints(tok, nc), *pids = ints(ids, nc), *pcur = ints(cur, b),
          *ppos = ints(pos, times({b, L_meta}));
  const hipStream_t stream = g.stream(len);
  return status_of([&] {
    return p_kv_start(plen, ptok, pids, pcur, ppos, L_meta, rows_, b, L_cap, stream);
  });
}

template <bool PLANNED>
PyObject* prefill(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 16);
  const at::Tensor *q = g.tensor(), *k = g.tensor(), *v = g.tensor(), *o = g.tensor();
  const int32_t b = g.i32(), H = g.i32(), L = g.i32(), d = g.i32();
  const int64_t qs = g.i64(), kvs = g.i64(), os = g.i64();
  const float scale = g.f32();
  const at::Tensor* vu = g.tensor();
  const int32_t L_meta = g.i32();
  const at::Tensor* ws = g.tensor();
  if (!q) throw Defer();
  const sckv_dtype dt = type_code(*q);
  void *pq = rows(q, b, H, L, d, qs, dt), *pk = rows(k, b, H, L, d, kvs, dt),
       *pv = rows(v, b, H, L, d, kvs, dt), *po = rows(o, b, H, L, d, os, dt);
  const int32_t* pvu = ints(vu, times({b, L_meta}));
  const Work w = workspace(ws);
  const hipStream_t stream = g.stream(q);
  return status_of([&] {
    return (PLANNED ? p_span_masked_prefill_attn_planned : p_span_masked_prefill_attn)(
        pq, pk, pv, po, b, H, L, d, qs, kvs, os, dt, scale, pvu, L_meta, w.p, w.n, stream);
  });
}

template <bool PLANNED>
PyObject* cached(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 21);
  const at::Tensor *q = g.tensor(), *k = g.tensor(), *v = g.tensor(), *o = g.tensor();
  const int32_t b = g.i32(), H = g.i32(), nq = g.i32(), d = g.i32();
  const int64_t qs = g.i64(), kvs = g.i64(), os = g.i64();
  const float scale = g.f32();
  const at::Tensor* vu = g.tensor();
  const int32_t L_meta = g.i32(), tok0 = g.i32();
  const at::Tensor *row0 = g.tensor(), *tok = g.tensor();
  const int32_t L_cap = g.i32();
  const at::Tensor *ws = g.tensor(), *st = g.tensor();
  if (!q) throw Defer();
  const sckv_dtype dt = type_code(*q);
  void *pq = rows(q, b, H, nq, d, qs, dt), *pk = rows(k, b, H, L_cap, d, kvs, dt),
       *pv = rows(v, b, H, L_cap, d, kvs, dt), *po = rows(o, b, H, nq, d, os, dt);
  const int32_t *pvu = ints(vu, times({b, L_meta})), *prow = ints(row0, b),
                *ptok = ints(tok, times({b, L_cap}));
  const Work w = workspace(ws);
  int32_t* pst = word(st);
  const hipStream_t stream = g.stream(q);
  return status_of([&] {
    return (PLANNED ? p_span_masked_prefill_attn_cached_planned : p_span_masked_prefill_attn_cached)(
        pq, pk, pv, po, b, H, nq, d, qs, kvs, os, dt, scale, pvu, L_meta, tok0, prow, ptok, L_cap,
        w.p, w.n, pst, stream);
  });
}

PyObject* plan(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 6);
  const at::Tensor* vu = g.tensor();
  const int32_t L_meta = g.i32(), b = g.i32(), L = g.i32();
  const at::Tensor* ws = g.tensor();
  const int32_t* pvu = ints(vu, times({b, L_meta}));
  const Work w = workspace(ws);
  const hipStream_t stream = g.stream(ws);
  return status_of([&] { return p_sckv_prefill_plan(pvu, L_meta, b, L, w.p, w.n, stream); });
}

PyObject* cached_plan(PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 10);
  const at::Tensor* vu = g.tensor();
  const int32_t L_meta = g.i32(), tok0 = g.i32();
  const at::Tensor *row0 = g.tensor(), *tok = g.tensor();
  const int32_t L_cap = g.i32(), b = g.i32(), nq = g.i32();
  const at::Tensor* ws = g.tensor();
  const int32_t *pvu = ints(vu, times({b, L_meta})), *prow = ints(row0, b),
                *ptok = ints(tok, times({b, L_cap}));
  const Work w = workspace(ws);
  const hipStream_t stream = g.stream(ws);
  return status_of([&] {
    return p_sckv_prefill_cached_plan(pvu, L_meta, tok0, prow, ptok, L_cap, b, nq, w.p, w.n,
                                      stream);
  });
}

// no C++ exception crosses into Python: whatever a check throws, binding.py
// takes over
template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    return F(a, n);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// init({entry name: address}, stream query)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 2 || !PyDict_Check(a[0])) {
    PyErr_SetString(PyExc_TypeError, "init(dict of entry points, stream query)");
    return nullptr;
  }
#define TAKE(name)                                                    \
  {                                                                   \
    PyObject* v = PyDict_GetItemString(a[0], #name);                  \
    void* p = v ? PyLong_AsVoidPtr(v) : nullptr;                      \
    if (!p) {                                                         \
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);  \
      return nullptr;                                                 \
    }                                                                 \
    p_##name = (decltype(p_##name))p;                                 \
  }
  ENTRIES(TAKE)
#undef TAKE
  Py_INCREF(a[1]);
  Py_XSETREF(g_raw_stream, a[1]);
  Py_RETURN_NONE;
}

#define METHOD(name, f) {name, (PyCFunction)(void (*)(void))guarded<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"init", (PyCFunction)(void (*)(void))init, METH_FASTCALL, nullptr},
    METHOD("compacted_decode_attn", decode<WITH_WS>),
    METHOD("compacted_decode_attn_noalloc", decode<NOALLOC>),
    METHOD("local_decode_attn", decode<LOCAL>),
    METHOD("kv_commit", commit),
    METHOD("kv_extend", extend),
    METHOD("kv_start", start),
    METHOD("kv_compact", compact),
    METHOD("rope_apply", rope<false>),
    METHOD("rope_apply_at", rope<true>),
    METHOD("rope_block", block),
    METHOD("span_masked_prefill_attn", prefill<false>),
    METHOD("span_masked_prefill_attn_planned", prefill<true>),
    METHOD("span_masked_prefill_attn_cached", cached<false>),
    METHOD("span_masked_prefill_attn_cached_planned", cached<true>),
    METHOD("sckv_prefill_plan", plan),
    METHOD("sckv_prefill_cached_plan", cached_plan),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind() { return PyModule_Create(&module); }
