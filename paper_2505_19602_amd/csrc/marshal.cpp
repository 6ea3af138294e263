// Argument marshalling of the Python binding in native code: tensor checks, pointers, strides and
// torch's current stream, then one call through the C ABI.  A step of a small map runs for about
// 10 us on the GPU; the same checks and ctypes structures in Python take 15-20 us per call
// (enqueueing a step of 16 queries: 19.2 us before, 8.1 us here, 7.3 us of it the two kernel launches).
//
// The functions answer None whenever an argument is not exactly what the common case expects
// (another type, a shape that does not match, a non-contiguous tensor): binding.py then takes
// its own checks, which raise the error that names the argument.  A non-OK status of the library
// comes back as its negative.  No arithmetic of the method happens here.
//
// Torch throws where a tensor has no memory of its own (one that vmap or functionalize has wrapped) or
// there is no device.  No C++ exception may leave an entry function: it answers None, and binding.py's
// own way to the same place raises torch's Python exception.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/TensorBase.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/scalekv.h"

namespace {

// Entry points of the library that binding.py has loaded, in the order of bind().
struct Entry {
  decltype(&scalekv_step) step;
  decltype(&scalekv_step_static) step_static;
  decltype(&scalekv_step_append_first) append_first;
  decltype(&scalekv_score) score;
  decltype(&scalekv_select) select;
  decltype(&scalekv_select_window) select_window;
  decltype(&scalekv_select_positional) select_positional;
  decltype(&scalekv_compact) compact;
  decltype(&scalekv_attend) attend;
  decltype(&scalekv_asi) asi;
} g_entry;
bool g_bound = false;

PyObject *g_n_seq, *g_n_head, *g_head_dim, *g_dtype, *g_sm_scale;  // interned attribute names

struct Shape {
  scalekv_shape c;
  at::ScalarType type;
};

bool to_int(PyObject* o, int32_t* out) {
  if (!PyLong_Check(o)) return false;
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || v < INT32_MIN || v > INT32_MAX) return false;
  *out = (int32_t)v;
  return true;
}

bool attr_int(PyObject* o, PyObject* name, int32_t* out) {
  PyObject* a = PyObject_GetAttr(o, name);
  if (!a) { PyErr_Clear(); return false; }
  const bool ok = to_int(a, out);
  Py_DECREF(a);
  return ok;
}

bool to_shape(PyObject* o, Shape* s) {
  if (!attr_int(o, g_n_seq, &s->c.n_seq) || !attr_int(o, g_n_head, &s->c.n_head) ||
      !attr_int(o, g_head_dim, &s->c.head_dim))
    return false;
  PyObject* t = PyObject_GetAttr(o, g_dtype);
  if (!t) { PyErr_Clear(); return false; }
  bool ok = THPDtype_Check(t);
  if (ok) s->type = reinterpret_cast<THPDtype*>(t)->scalar_type;
  Py_DECREF(t);
  if (!ok || (s->type != at::kFloat && s->type != at::kBFloat16)) return false;
  s->c.dtype = s->type == at::kFloat ? SCALEKV_F32 : SCALEKV_BF16;
  PyObject* f = PyObject_GetAttr(o, g_sm_scale);
  if (!f) { PyErr_Clear(); return false; }
  s->c.sm_scale = (float)PyFloat_AsDouble(f);
  Py_DECREF(f);
  if (PyErr_Occurred()) { PyErr_Clear(); return false; }
  return true;
}

// A contiguous device tensor [n_seq, n_head, ...]; NULL if it is anything else.
const at::TensorBase* device_tensor(PyObject* o, const Shape& s, int dims, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::TensorBase& t = THPVariable_Unpack(o);
  if (t.dim() != dims || t.scalar_type() != type || !t.is_cuda()) return nullptr;
  if (t.size(0) != s.c.n_seq || t.size(1) != s.c.n_head) return nullptr;
  return &t;
}

// dense [S, H, rows, d]; *rows < 0: take the tensor's own
bool dense(PyObject* o, const Shape& s, int32_t* rows, void** p) {
  const at::TensorBase* t = device_tensor(o, s, 4, s.type);
  if (!t || !t->is_contiguous() || t->size(3) != s.c.head_dim || t->size(2) > INT32_MAX) return false;
  if (*rows < 0) *rows = (int32_t)t->size(2);
  if (t->size(2) != *rows) return false;
  *p = t->data_ptr();
  return true;
}

bool cache(PyObject* o, const Shape& s, scalekv_kv* kv) {
  const at::TensorBase* t = device_tensor(o, s, 4, s.type);
  if (!t || t->size(3) != s.c.head_dim || t->stride(3) != 1 || t->stride(2) != s.c.head_dim ||
      t->size(2) > INT32_MAX)
    return false;
  *kv = scalekv_kv{t->data_ptr(), t->stride(0), t->stride(1), (int32_t)t->size(2)};
  return true;
}

// contiguous [S, H, n] of the given type
bool plane(PyObject* o, const Shape& s, at::ScalarType type, int64_t n, void** p) {
  const at::TensorBase* t = device_tensor(o, s, 3, type);
  if (!t || !t->is_contiguous() || t->size(2) != n) return false;
  *p = t->data_ptr();
  return true;
}

bool optional_plane(PyObject* o, const Shape& s, int64_t n, int32_t** p) {
  *p = nullptr;
  return o == Py_None || plane(o, s, at::kInt, n, reinterpret_cast<void**>(p));
}

bool workspace(PyObject* o, void** p, size_t* bytes) {
  *p = nullptr;
  *bytes = 0;
  if (o == Py_None) return true;
  if (!THPVariable_CheckExact(o)) return false;
  const at::TensorBase& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous()) return false;
  *p = t.data_ptr();
  *bytes = (size_t)t.numel() * t.element_size();
  return true;
}

struct Window {
  int32_t row[SCALEKV_MAX_WINDOW];
  int32_t n;
};

bool to_window(PyObject* o, Window* w) {
  if (!PyList_Check(o) && !PyTuple_Check(o)) return false;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
  if (n > INT32_MAX) return false;
  // (the library reads no row of a longer window: it refuses it or, where nothing is ranked, has no use for it)
  for (Py_ssize_t i = 0; i < n && i < SCALEKV_MAX_WINDOW; ++i)
    if (!to_int(PySequence_Fast_GET_ITEM(o, i), &w->row[i])) return false;
  w->n = (int32_t)n;
  return true;
}

// The library call runs without the interpreter lock: enqueueing waits when the stream's queue is full.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

int32_t kept(int32_t budget, int32_t len) { return budget < 0 ? 0 : budget < len ? budget : (len > 0 ? len : 0); }

PyObject* none() { Py_RETURN_NONE; }
template <typename Call>
scalekv_status unlocked(Call call) {
  Unlocked released;
  return call();
}
PyObject* answer(scalekv_status st, long value) { return PyLong_FromLong(st == SCALEKV_OK ? value : -(long)st); }

// ---- the arguments of one step, marshalled
struct StepArgs {
  Shape shape;
  void *q, *k_cur, *v_cur, *out, *ws;
  size_t ws_bytes;
  int32_t* idx;
  int32_t n_cur, cache_len, budget, pool_w;
  Window win;
  scalekv_kv k_src, v_src, k_dst, v_dst;
  bool has_k_dst, has_v_dst;
  int32_t keep;

  // step and step_static: (shape, q, k_cur, v_cur, win, k_src, v_src, cache_len, budget, k_dst, v_dst, out, idx[, ws])
  bool parse_step(PyObject* const* a, bool with_ws) {
    n_cur = -1;
    has_k_dst = has_v_dst = true;
    if (!to_shape(a[0], &shape) || !dense(a[1], shape, &n_cur, &q) || !dense(a[2], shape, &n_cur, &k_cur) ||
        !dense(a[3], shape, &n_cur, &v_cur) || !to_window(a[4], &win) || !cache(a[5], shape, &k_src) ||
        !cache(a[6], shape, &v_src) || !to_int(a[7], &cache_len) || !to_int(a[8], &budget) ||
        !cache(a[9], shape, &k_dst) || !cache(a[10], shape, &v_dst) || !dense(a[11], shape, &n_cur, &out))
      return false;
    keep = kept(budget, cache_len);
    if (!optional_plane(a[12], shape, keep, &idx)) return false;
    return !with_ws || workspace(a[13], &ws, &ws_bytes);
  }
  // step_append_first: (shape, q, k_cur, v_cur, win, pool_w, k_cache, v_cache, cache_len, budget, k_next, v_next,
  // out, idx, ws)
  bool parse_append_first(PyObject* const* a) {
    n_cur = -1;
    if (!to_shape(a[0], &shape) || !dense(a[1], shape, &n_cur, &q) || !dense(a[2], shape, &n_cur, &k_cur) ||
        !dense(a[3], shape, &n_cur, &v_cur) || !to_window(a[4], &win) || !to_int(a[5], &pool_w) ||
        !cache(a[6], shape, &k_src) || !cache(a[7], shape, &v_src) || !to_int(a[8], &cache_len) ||
        !to_int(a[9], &budget))
      return false;
    has_k_dst = a[10] != Py_None;
    has_v_dst = a[11] != Py_None;
    if ((has_k_dst && !cache(a[10], shape, &k_dst)) || (has_v_dst && !cache(a[11], shape, &v_dst))) return false;
    const int64_t rest = (int64_t)cache_len + n_cur - win.n;
    const int64_t some = budget < rest ? budget : rest;
    keep = (int32_t)(win.n + (some > 0 ? some : 0));
    return dense(a[12], shape, &n_cur, &out) && optional_plane(a[13], shape, keep, &idx) &&
           workspace(a[14], &ws, &ws_bytes);
  }
  // the new cache length, or the negative status
  long run_step(void* stream) const {
    int32_t len = -1;
    Unlocked unlocked;
    const scalekv_status st =
        g_entry.step(&shape.c, q, k_cur, v_cur, n_cur, win.row, win.n, &k_src, &v_src, cache_len, budget, &k_dst,
                     &v_dst, &len, out, idx, ws, ws_bytes, stream);
    return st == SCALEKV_OK ? len : -(long)st;
  }
  scalekv_status run_append_first(void* stream, int32_t* keep_out, int32_t* moved) const {
    Unlocked unlocked;
    return g_entry.append_first(&shape.c, q, k_cur, v_cur, n_cur, win.row, win.n, pool_w, &k_src, &v_src, cache_len,
                                budget, has_k_dst ? &k_dst : nullptr, has_v_dst ? &v_dst : nullptr, keep_out, moved, out,
                                idx, ws, ws_bytes, stream);
  }
};

#define SCALEKV_ARITY(want) \
  if (!g_bound || n != (want)) return none()

PyObject* py_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(14);
  StepArgs s;
  if (!s.parse_step(a, true)) return none();
  return PyLong_FromLong(s.run_step(current_stream()));
}

PyObject* py_step_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(13);
  StepArgs s;
  if (!s.parse_step(a, false)) return none();
  int32_t len = -1;
  void* const stream = current_stream();
  const scalekv_status st = unlocked([&] {
    return g_entry.step_static(&s.shape.c, s.q, s.k_cur, s.v_cur, s.n_cur, s.win.row, s.win.n, &s.k_src, &s.v_src,
                               s.cache_len, s.budget, &s.k_dst, &s.v_dst, &len, s.out, s.idx, stream);
  });
  return answer(st, len);
}

PyObject* py_append_first(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(15);
  StepArgs s;
  if (!s.parse_append_first(a)) return none();
  int32_t keep = -1, moved = -1;
  const scalekv_status st = s.run_append_first(current_stream(), &keep, &moved);
  if (st != SCALEKV_OK) return answer(st, 0);
  return PyLong_FromLong(2L * keep + (moved != 0));
}

// (shape, q_win, k, cache_len, log_scores, ws)
PyObject* py_score(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(6);
  Shape s;
  int32_t n_win = -1, len;
  void *q, *ls, *ws;
  size_t bytes;
  scalekv_kv k;
  if (!to_shape(a[0], &s) || !dense(a[1], s, &n_win, &q) || !cache(a[2], s, &k) || !to_int(a[3], &len) ||
      !plane(a[4], s, at::kFloat, len, &ls) || !workspace(a[5], &ws, &bytes))
    return none();
  void* const stream = current_stream();
  return answer(unlocked([&] { return g_entry.score(&s.c, q, n_win, &k, len, (float*)ls, ws, bytes, stream); }), 0);
}

// (shape, scores, cache_len, budget, idx)
PyObject* py_select(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(5);
  Shape s;
  int32_t len, budget, keep = -1;
  void *scores, *idx;
  if (!to_shape(a[0], &s) || !to_int(a[2], &len) || !plane(a[1], s, at::kFloat, len, &scores) ||
      !to_int(a[3], &budget) || !plane(a[4], s, at::kInt, kept(budget, len), &idx))
    return none();
  void* const stream = current_stream();
  const scalekv_status st = unlocked(
      [&] { return g_entry.select(&s.c, (const float*)scores, len, budget, (int32_t*)idx, &keep, stream); });
  return answer(st, keep);
}

// (shape, log_scores, cache_len, budget, forced, pool_w, idx)
PyObject* py_select_window(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(7);
  Shape s;
  int32_t len, budget, pool_w, keep = -1;
  Window forced;
  void *scores, *idx;
  if (!to_shape(a[0], &s) || !to_int(a[2], &len) || !plane(a[1], s, at::kFloat, len, &scores) ||
      !to_int(a[3], &budget) || !to_window(a[4], &forced) || !to_int(a[5], &pool_w) ||
      !plane(a[6], s, at::kInt, (int64_t)forced.n + kept(budget, len - forced.n), &idx))
    return none();
  void* const stream = current_stream();
  const scalekv_status st = unlocked([&] {
    return g_entry.select_window(&s.c, (const float*)scores, len, budget, forced.row, forced.n, pool_w, (int32_t*)idx,
                                 &keep, stream);
  });
  return answer(st, keep);
}

// (shape, cache_len, n_sink, n_recent, idx)
PyObject* py_select_positional(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(5);
  Shape s;
  int32_t len, sink, recent, keep = -1;
  void* idx;
  if (!to_shape(a[0], &s) || !to_int(a[1], &len) || !to_int(a[2], &sink) || !to_int(a[3], &recent)) return none();
  const int32_t first = kept(sink, len);
  if (!plane(a[4], s, at::kInt, (int64_t)first + kept(recent, len - first), &idx)) return none();
  void* const stream = current_stream();
  const scalekv_status st =
      unlocked([&] { return g_entry.select_positional(&s.c, len, sink, recent, (int32_t*)idx, &keep, stream); });
  return answer(st, keep);
}

// (shape, k_src, v_src, cache_len, idx, keep, k_cur, v_cur, k_dst, v_dst)
PyObject* py_compact(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(10);
  Shape s;
  int32_t len, keep, n_cur = 0;
  int32_t* idx;
  void *kc = nullptr, *vc = nullptr;
  scalekv_kv ks, vs, kd, vd;
  if (!to_shape(a[0], &s) || !cache(a[1], s, &ks) || !cache(a[2], s, &vs) || !to_int(a[3], &len) ||
      !to_int(a[5], &keep) || !optional_plane(a[4], s, keep, &idx) || !cache(a[8], s, &kd) || !cache(a[9], s, &vd))
    return none();
  if (a[6] != Py_None) {
    n_cur = -1;
    if (!dense(a[6], s, &n_cur, &kc) || !dense(a[7], s, &n_cur, &vc)) return none();
  } else if (a[7] != Py_None) {
    return none();
  }
  void* const stream = current_stream();
  return answer(
      unlocked([&] { return g_entry.compact(&s.c, &ks, &vs, len, idx, keep, kc, vc, n_cur, &kd, &vd, stream); }),
      (long)keep + n_cur);
}

// (shape, q, k, v, kv_len, out)
PyObject* py_attend(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(6);
  Shape s;
  int32_t n_q = -1, len;
  void *q, *out;
  scalekv_kv k, v;
  if (!to_shape(a[0], &s) || !dense(a[1], s, &n_q, &q) || !cache(a[2], s, &k) || !cache(a[3], s, &v) ||
      !to_int(a[4], &len) || !dense(a[5], s, &n_q, &out))
    return none();
  void* const stream = current_stream();
  return answer(unlocked([&] { return g_entry.attend(&s.c, q, n_q, &k, &v, len, out, stream); }), 0);
}

// (shape, q_samp, k, hist_len, cur_len, top_k, terms, asi_out, ws)
PyObject* py_asi(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SCALEKV_ARITY(9);
  Shape s;
  int32_t n_samp = -1, hist, cur, top_k;
  void *q, *ws, *mean = nullptr;
  size_t bytes;
  scalekv_kv k;
  if (!to_shape(a[0], &s) || !dense(a[1], s, &n_samp, &q) || !cache(a[2], s, &k) || !to_int(a[3], &hist) ||
      !to_int(a[4], &cur) || !to_int(a[5], &top_k) || !workspace(a[8], &ws, &bytes))
    return none();
  const at::TensorBase* terms = device_tensor(a[6], s, 4, at::kFloat);
  if (!terms || !terms->is_contiguous() || terms->size(2) != n_samp || terms->size(3) != 2) return none();
  if (a[7] != Py_None) {
    if (!THPVariable_CheckExact(a[7])) return none();
    const at::TensorBase& t = THPVariable_Unpack(a[7]);
    if (t.scalar_type() != at::kFloat || !t.is_cuda() || !t.is_contiguous() || t.numel() != 3) return none();
    mean = t.data_ptr();
  }
  void* const stream = current_stream();
  float* const terms_p = (float*)terms->data_ptr();
  return answer(unlocked([&] {
                  return g_entry.asi(&s.c, q, n_samp, &k, hist, cur, top_k, terms_p, (float*)mean, ws, bytes, stream);
                }),
                0);
}

// ---- a call whose arguments are marshalled once: prepared(stream or None) -> as the call itself
struct Prepared {
  PyObject_HEAD
  StepArgs args;
  bool append_first;
  vectorcallfunc vectorcall;
};

PyObject* prepared_call(PyObject* self, PyObject* const* a, size_t nf, PyObject*) try {
  const Prepared* p = reinterpret_cast<Prepared*>(self);
  void* stream;
  if (PyVectorcall_NARGS(nf) < 1 || a[0] == Py_None) {
    stream = current_stream();
  } else {
    stream = PyLong_AsVoidPtr(a[0]);
    if (!stream && PyErr_Occurred()) return nullptr;
  }
  if (!p->append_first) return PyLong_FromLong(p->args.run_step(stream));
  int32_t keep = -1, moved = -1;
  const scalekv_status st = p->args.run_append_first(stream, &keep, &moved);
  if (st != SCALEKV_OK) return answer(st, 0);
  return PyLong_FromLong(2L * keep + (moved != 0));
} catch (const std::exception& e) {
  PyErr_SetString(PyExc_RuntimeError, e.what());
  return nullptr;
}

PyTypeObject g_prepared_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* py_prepare(PyObject* const* a, Py_ssize_t n, bool append_first) {
  SCALEKV_ARITY(append_first ? 15 : 14);
  StepArgs s;
  if (!(append_first ? s.parse_append_first(a) : s.parse_step(a, true))) return none();
  Prepared* p = PyObject_New(Prepared, &g_prepared_type);
  if (!p) return nullptr;
  p->args = s;
  p->append_first = append_first;
  p->vectorcall = prepared_call;
  return reinterpret_cast<PyObject*>(p);
}
PyObject* py_prepare_step(PyObject*, PyObject* const* a, Py_ssize_t n) { return py_prepare(a, n, false); }
PyObject* py_prepare_append_first(PyObject*, PyObject* const* a, Py_ssize_t n) { return py_prepare(a, n, true); }

// bind(addresses): the library's entry points as integers, in the order of struct Entry
PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* addr[sizeof(Entry) / sizeof(void*)];
  if (n != (Py_ssize_t)(sizeof(addr) / sizeof(addr[0]))) {
    PyErr_SetString(PyExc_TypeError, "bind() takes one address for each entry point");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    addr[i] = PyLong_AsVoidPtr(a[i]);
    if (!addr[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind() got a NULL address");
      return nullptr;
    }
  }
  static_assert(sizeof(addr) == sizeof(Entry), "one pointer for each entry point");
  memcpy(&g_entry, addr, sizeof(addr));
  g_bound = true;
  return none();
}

typedef PyObject* (*FastCall)(PyObject*, PyObject* const*, Py_ssize_t);
template <FastCall CALL>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n) try {
  return CALL(self, a, n);
} catch (const std::exception&) {  // before anything was enqueued: the library does not throw
  return none();
}

#define SCALEKV_METHOD(name) {#name, (PyCFunction)(void (*)(void))guarded<py_##name>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    SCALEKV_METHOD(bind), SCALEKV_METHOD(step), SCALEKV_METHOD(step_static), SCALEKV_METHOD(append_first),
    SCALEKV_METHOD(score), SCALEKV_METHOD(select), SCALEKV_METHOD(select_window), SCALEKV_METHOD(select_positional),
    SCALEKV_METHOD(compact), SCALEKV_METHOD(attend), SCALEKV_METHOD(asi), SCALEKV_METHOD(prepare_step),
    SCALEKV_METHOD(prepare_append_first), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  g_n_seq = PyUnicode_InternFromString("n_seq");
  g_n_head = PyUnicode_InternFromString("n_head");
  g_head_dim = PyUnicode_InternFromString("head_dim");
  g_dtype = PyUnicode_InternFromString("dtype");
  g_sm_scale = PyUnicode_InternFromString("sm_scale");
  g_prepared_type.tp_name = "_marshal.Prepared";
  g_prepared_type.tp_basicsize = sizeof(Prepared);
  g_prepared_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
  g_prepared_type.tp_vectorcall_offset = offsetof(Prepared, vectorcall);
  g_prepared_type.tp_call = PyVectorcall_Call;
  g_prepared_type.tp_dealloc = [](PyObject* o) { PyObject_Free(o); };
  if (PyType_Ready(&g_prepared_type) < 0) return nullptr;
  return PyModule_Create(&g_module);
}
