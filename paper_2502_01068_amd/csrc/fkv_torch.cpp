// Native call path of binding.py: one function per wrapper that checks torch tensors against the host
// descriptor, allocates missing outputs, finds the current stream and makes the library call.
//
// A call at the sizes where launches count (one decode step, a short prompt) was bound by the Python
// around it: of 12 and 32 us per decode and compress call, 7.5 and 18 went into attribute reads, size
// checks, argument conversion and torch.empty.  Here a decode call is issued in 4.1 us and a compress call in 12.7, launches included.
//
// Every function returns None for anything it does not recognise as a correct call (wrong type, size, device, count,
// a call the library refuses): the Python wrapper then makes the call itself, whose checks name the
// mistake.  Nothing has been enqueued in that case, since the library validates before its first launch.  A failed
// HIP call is raised from here: launches before it may have been enqueued, so the call is not made again.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "fastkv_select.h"

namespace {

struct Api {
  decltype(&fkv_score_window) score_window;
  decltype(&fkv_score_heads) score_heads;
  decltype(&fkv_select_topk) select_topk;
  decltype(&fkv_gather_rows) gather_rows;
  decltype(&fkv_gather_kv) gather_kv;
  decltype(&fkv_gather_kv_per_head) gather_kv_per_head;
  decltype(&fkv_compress_kv) compress_kv;
  decltype(&fkv_compress_kv_paged) compress_kv_paged;
  decltype(&fkv_decode_attention) decode_attention;
  decltype(&fkv_decode_attention_paged) decode_attention_paged;
  decltype(&fkv_window_output) window_output;
  decltype(&fkv_score_window_output) score_window_output;
} api;

PyTypeObject *shape_type = nullptr;
PyObject *error_type = nullptr;
PyObject *key_k_out, *key_v_out, *key_idx_kv, *key_x_out, *key_idx_tsp;

// The fixed head of every call: context handle and device, descriptor, and the sizes that follow from it.
struct Call {
  fkv_ctx *ctx = nullptr;
  int dev = -1;
  const fkv_shape *shape = nullptr;
  int64_t total = 0, sum_p = 0, q_win = 0, q_dec = 0, kv = 0;
  int64_t n_seq = 0, hq = 0, hkv = 0, d = 0;
  void *stream = nullptr;

  bool open(PyObject *const *args) {
    ctx = static_cast<fkv_ctx *>(PyLong_AsVoidPtr(args[0]));
    dev = (int)PyLong_AsLong(args[1]);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    if (ctx == nullptr || shape_type == nullptr || !PyObject_TypeCheck(args[2], shape_type)) return false;
    Py_buffer buf;
    if (PyObject_GetBuffer(args[2], &buf, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return false; }
    shape = buf.len >= (Py_ssize_t)sizeof(fkv_shape) ? static_cast<const fkv_shape *>(buf.buf) : nullptr;
    PyBuffer_Release(&buf);  // the caller holds the object for the length of the call
    if (shape == nullptr || shape->n_seq < 1 || shape->n_seq > FKV_MAX_SEQS || shape->cu_seqlens == nullptr) return false;
    if (c10::hip::current_device() != dev) return false;
    n_seq = shape->n_seq, hq = shape->n_q_heads, hkv = shape->n_kv_heads, d = shape->head_dim;
    total = shape->cu_seqlens[n_seq];
    sum_p = total - n_seq * shape->window;
    if (hq < 1 || hkv < 1 || d < 1 || shape->window < 1 || sum_p < 0) return false;
    q_dec = n_seq * hq * d;
    q_win = q_dec * shape->window;
    kv = total * hkv * d;
    stream = c10::hip::getCurrentHIPStream((c10::DeviceIndex)dev).stream();
    return true;
  }
};

enum Kind { kAny, kBf16, kF32, kI32 };
bool kind_ok(Kind kind, at::ScalarType t) {
  switch (kind) {
    case kBf16: return t == at::kBFloat16 || t == at::kShort || t == at::kUInt16;
    case kF32: return t == at::kFloat;
    case kI32: return t == at::kInt;
    default: return true;
  }
}

// The tensor behind `o` if it is on the context's GPU, contiguous, of the kind and long enough.
const at::Tensor *tensor(const Call &c, PyObject *o, Kind kind, int64_t numel) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.get_device() != c.dev || t.layout() != at::kStrided || !t.is_contiguous() ||
      !kind_ok(kind, t.scalar_type()) || t.numel() < numel)
    return nullptr;
  return &t;
}

// An output the caller passed, or a new one.
bool output(const Call &c, PyObject *o, Kind kind, int64_t numel, at::IntArrayRef sizes, at::ScalarType dtype, at::Tensor &out) {
  if (o != nullptr && o != Py_None) {
    const at::Tensor *t = tensor(c, o, kind, numel);
    if (t == nullptr) return false;
    out = *t;
    return true;
  }
  out = at::empty(sizes, at::TensorOptions().dtype(dtype).device(c10::Device(c10::kCUDA, (c10::DeviceIndex)c.dev)));
  return true;
}

// Per-sequence counts: one int for all sequences or a list / tuple of them.
struct Counts {
  int32_t v[FKV_MAX_SEQS];
  int64_t sum = 0;
  bool read(const Call &c, PyObject *o) {
    if (PyLong_CheckExact(o)) {
      const long x = PyLong_AsLong(o);
      if (PyErr_Occurred() || x < 0 || x > INT32_MAX) { PyErr_Clear(); return false; }
      for (int64_t b = 0; b < c.n_seq; ++b) v[b] = (int32_t)x;
      sum = x * c.n_seq;
      return sum <= INT32_MAX;
    }
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
    if (PySequence_Fast_GET_SIZE(o) != c.n_seq) return false;
    PyObject **items = PySequence_Fast_ITEMS(o);
    for (int64_t b = 0; b < c.n_seq; ++b) {
      if (!PyLong_CheckExact(items[b])) return false;
      const long x = PyLong_AsLong(items[b]);
      if (PyErr_Occurred() || x < 0 || x > INT32_MAX) { PyErr_Clear(); return false; }
      v[b] = (int32_t)x;
      sum += x;
    }
    return sum <= INT32_MAX;
  }
};

struct HipFailure { const char *where; };

// False if the library refuses the call.
template <typename F>
bool call(const char *where, F &&f) {
  int status;
  {
    struct NoGil {
      PyThreadState *state = PyEval_SaveThread();
      ~NoGil() { PyEval_RestoreThread(state); }
    } no_gil;
    status = f();
  }
  if (status == FKV_EHIP) throw HipFailure{where};
  return status == FKV_OK;
}

PyObject *none() { Py_RETURN_NONE; }
PyObject *wrap(const at::Tensor &t) { return THPVariable_Wrap(t); }
PyObject *wrap_or_none(const at::Tensor &t) { return t.defined() ? THPVariable_Wrap(t) : none(); }
float *f32(const at::Tensor &t) { return t.defined() ? static_cast<float *>(t.data_ptr()) : nullptr; }
int32_t *i32(const at::Tensor &t) { return static_cast<int32_t *>(t.data_ptr()); }

// C++ exceptions of torch (an allocation that fails, for one) become a fallback to the Python wrapper, which
// then meets the same condition.
template <PyObject *(*F)(PyObject *const *), Py_ssize_t kArgs>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != kArgs) return none();
  try {
    return F(args);
  } catch (const HipFailure &e) {
    if (PyObject *error = PyObject_CallFunction(error_type, "is", (int)FKV_EHIP, e.where)) {
      PyErr_SetObject(error_type, error);
      Py_DECREF(error);
    }
    return nullptr;
  } catch (...) {
    PyErr_Clear();
    return none();
  }
}

// (ctx, dev, shape, q_win, k, scores_group, scores_tsp, want_tsp)
PyObject *score_window(PyObject *const *a) {
  Call c;
  if (!c.open(a)) return none();
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_win), *k = tensor(c, a[4], kBf16, c.kv);
  at::Tensor sg, st;
  if (!q || !k || !output(c, a[5], kF32, c.hkv * c.sum_p, {c.hkv, c.sum_p}, at::kFloat, sg)) return none();
  if ((a[6] != Py_None || a[7] == Py_True) && !output(c, a[6], kF32, c.sum_p, {c.sum_p}, at::kFloat, st)) return none();
  if (!call("fkv_score_window", [&] {
        return api.score_window(c.ctx, c.shape, q->data_ptr(), k->data_ptr(), f32(sg), f32(st), c.stream);
      }))
    return none();
  return Py_BuildValue("(NN)", wrap(sg), wrap_or_none(st));
}

// (ctx, dev, shape, q_win, k, scores_head)
PyObject *score_heads(PyObject *const *a) {
  Call c;
  if (!c.open(a)) return none();
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_win), *k = tensor(c, a[4], kBf16, c.kv);
  at::Tensor sh;
  if (!q || !k || !output(c, a[5], kF32, c.hq * c.sum_p, {c.hq, c.sum_p}, at::kFloat, sh)) return none();
  if (!call("fkv_score_heads", [&] {
        return api.score_heads(c.ctx, c.shape, q->data_ptr(), k->data_ptr(), f32(sh), c.stream);
      }))
    return none();
  return wrap(sh);
}

// (ctx, dev, shape, scores, k_per_seq, idx_out)
PyObject *select_topk(PyObject *const *a) {
  Call c;
  Counts n;
  if (!c.open(a) || !n.read(c, a[4])) return none();
  const at::Tensor *s = tensor(c, a[3], kF32, 0);
  if (!s || s->dim() < 1 || s->dim() > 2 || s->size(-1) != c.sum_p) return none();
  const int64_t rows = s->dim() == 1 ? 1 : s->size(0);
  at::Tensor idx;
  if (rows > INT32_MAX || !output(c, a[5], kI32, rows * n.sum, {rows, n.sum}, at::kInt, idx)) return none();
  if (!call("fkv_select_topk", [&] {
        return api.select_topk(c.ctx, c.shape, f32(*s), (int32_t)rows, n.v, i32(idx), c.stream);
      }))
    return none();
  return wrap(idx);
}

// (ctx, dev, shape, x, idx, k_per_seq, out)
PyObject *gather_rows(PyObject *const *a) {
  Call c;
  Counts n;
  if (!c.open(a) || !n.read(c, a[5])) return none();
  const at::Tensor *x = tensor(c, a[3], kAny, 0), *idx = tensor(c, a[4], kI32, n.sum);
  if (!x || !idx || x->dim() < 1 || x->size(0) != c.total) return none();
  const size_t row_bytes = x->stride(0) * x->element_size();
  at::Tensor out;
  c10::DimVector sizes(x->sizes().begin(), x->sizes().end());
  sizes[0] = n.sum;
  if (!output(c, a[6], kAny, 0, sizes, x->scalar_type(), out) || out.nbytes() < n.sum * row_bytes) return none();
  if (!call("fkv_gather_rows", [&] {
        return api.gather_rows(c.ctx, c.shape, x->data_ptr(), row_bytes, i32(*idx), n.v, out.data_ptr(), c.stream);
      }))
    return none();
  return wrap(out);
}

// (ctx, dev, shape, k, v, idx, budget, k_out, v_out), one copy per KV head or per query head
template <bool kPerHead>
PyObject *gather_kv(PyObject *const *a) {
  Call c;
  Counts n;
  if (!c.open(a) || !n.read(c, a[6])) return none();
  const int64_t heads = kPerHead ? c.hq : c.hkv;
  const bool has_v = a[4] != Py_None;
  const at::Tensor *k = tensor(c, a[3], kBf16, c.kv), *v = has_v ? tensor(c, a[4], kBf16, c.kv) : nullptr;
  const at::Tensor *idx = tensor(c, a[5], kI32, heads * n.sum);
  at::Tensor ko, vo;
  if (!k || !idx || (has_v && !v) || (!has_v && a[8] != Py_None)) return none();
  const int64_t sizes[3] = {heads, n.sum, c.d};
  if (!output(c, a[7], kBf16, heads * n.sum * c.d, sizes, k->scalar_type(), ko)) return none();
  if (has_v && !output(c, a[8], kBf16, heads * n.sum * c.d, sizes, v->scalar_type(), vo)) return none();
  const auto fn = kPerHead ? api.gather_kv_per_head : api.gather_kv;
  if (!call(kPerHead ? "fkv_gather_kv_per_head" : "fkv_gather_kv", [&] {
        return fn(c.ctx, c.shape, k->data_ptr(), has_v ? v->data_ptr() : nullptr, i32(*idx), n.v, ko.data_ptr(),
                  has_v ? vo.data_ptr() : nullptr, c.stream);
      }))
    return none();
  return Py_BuildValue("(NN)", wrap(ko), wrap_or_none(vo));
}

// (ctx, dev, shape, q_win, k, v, budget, x, k_tsp, out)
PyObject *compress_kv(PyObject *const *a) {
  Call c;
  Counts nb, nt;
  if (!c.open(a) || !nb.read(c, a[6])) return none();
  const bool tsp = a[7] != Py_None;
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_win), *k = tensor(c, a[4], kBf16, c.kv), *v = tensor(c, a[5], kBf16, c.kv);
  const at::Tensor *x = tsp ? tensor(c, a[7], kAny, 0) : nullptr;
  if (!q || !k || !v || (tsp && (!x || x->dim() < 1 || x->size(0) != c.total || !nt.read(c, a[8])))) return none();
  PyObject *dict = a[9] == Py_None ? nullptr : a[9];
  if (dict != nullptr && !PyDict_CheckExact(dict)) return none();
  auto item = [&](PyObject *key) { return dict ? PyDict_GetItem(dict, key) : nullptr; };
  auto missing = [&](PyObject *key) { return dict != nullptr && (item(key) == nullptr || item(key) == Py_None); };
  if (missing(key_k_out) || missing(key_v_out) || missing(key_idx_kv) || (tsp && (missing(key_x_out) || missing(key_idx_tsp)))) return none();
  const int64_t kv_sizes[3] = {c.hkv, nb.sum, c.d}, n_kv = c.hkv * nb.sum * c.d;
  at::Tensor ko, vo, ik, xo, it;
  if (!output(c, item(key_k_out), kBf16, n_kv, kv_sizes, k->scalar_type(), ko)) return none();
  if (!output(c, item(key_v_out), kBf16, n_kv, kv_sizes, v->scalar_type(), vo)) return none();
  if (!output(c, item(key_idx_kv), kI32, c.hkv * nb.sum, {c.hkv, nb.sum}, at::kInt, ik)) return none();
  size_t row_bytes = 0;
  if (tsp) {
    row_bytes = x->stride(0) * x->element_size();
    c10::DimVector sizes(x->sizes().begin(), x->sizes().end());
    sizes[0] = nt.sum;
    if (!output(c, item(key_x_out), kAny, 0, sizes, x->scalar_type(), xo) || xo.nbytes() < nt.sum * row_bytes) return none();
    if (!output(c, item(key_idx_tsp), kI32, nt.sum, {nt.sum}, at::kInt, it)) return none();
  }
  if (!call("fkv_compress_kv", [&] {
        return api.compress_kv(c.ctx, c.shape, q->data_ptr(), k->data_ptr(), v->data_ptr(), nb.v, ko.data_ptr(), vo.data_ptr(), i32(ik),
                               tsp ? x->data_ptr() : nullptr, row_bytes, tsp ? nt.v : nullptr, tsp ? xo.data_ptr() : nullptr,
                               tsp ? i32(it) : nullptr, c.stream);
      }))
    return none();
  if (dict != nullptr) {
    Py_INCREF(dict);
    return dict;
  }
  PyObject *out = PyDict_New();
  if (out == nullptr) return nullptr;
  auto put = [&](PyObject *key, const at::Tensor &t) {
    PyObject *o = wrap(t);
    const int rc = o == nullptr ? -1 : PyDict_SetItem(out, key, o);
    Py_XDECREF(o);
    return rc == 0;
  };
  if (!put(key_k_out, ko) || !put(key_v_out, vo) || !put(key_idx_kv, ik) || (tsp && (!put(key_x_out, xo) || !put(key_idx_tsp, it)))) {
    Py_DECREF(out);
    return nullptr;
  }
  return out;
}

// Page pools [n_pages][page_size][Hkv][d] and their block table [n_seq][max_pages].
struct Pages {
  const at::Tensor *k = nullptr, *v = nullptr, *table = nullptr;
  bool read(const Call &c, PyObject *ok, PyObject *ov, PyObject *ot) {
    k = tensor(c, ok, kBf16, 0);
    v = tensor(c, ov, kBf16, 0);
    table = tensor(c, ot, kI32, 0);
    return k && v && table && k->dim() == 4 && k->size(2) == c.hkv && k->size(3) == c.d && v->sizes() == k->sizes() &&
           table->dim() == 2 && table->size(0) == c.n_seq && table->size(1) <= INT32_MAX && k->size(1) <= INT32_MAX;
  }
};

// (ctx, dev, shape, q_win, k, v, budget, block_table, k_pages, v_pages, idx_kv)
PyObject *compress_kv_paged(PyObject *const *a) {
  Call c;
  Counts n;
  Pages p;
  if (!c.open(a) || !n.read(c, a[6]) || !p.read(c, a[8], a[9], a[7])) return none();
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_win), *k = tensor(c, a[4], kBf16, c.kv), *v = tensor(c, a[5], kBf16, c.kv);
  at::Tensor idx;
  if (!q || !k || !v || !output(c, a[10], kI32, c.hkv * n.sum, {c.hkv, n.sum}, at::kInt, idx)) return none();
  if (!call("fkv_compress_kv_paged", [&] {
        return api.compress_kv_paged(c.ctx, c.shape, q->data_ptr(), k->data_ptr(), v->data_ptr(), n.v, i32(*p.table), (int32_t)p.table->size(1),
                                     (int32_t)p.k->size(1), p.k->size(0), p.k->data_ptr(), p.v->data_ptr(), i32(idx), c.stream);
      }))
    return none();
  return wrap(idx);
}

// (ctx, dev, shape, q, k, v, n_per_seq, layout, out)
PyObject *decode_attention(PyObject *const *a) {
  Call c;
  Counts n;
  if (!c.open(a) || !n.read(c, a[6]) || !PyUnicode_Check(a[7])) return none();
  int32_t layout;
  if (PyUnicode_CompareWithASCIIString(a[7], "compact") == 0) layout = FKV_KV_COMPACT;
  else if (PyUnicode_CompareWithASCIIString(a[7], "token_major") == 0) layout = FKV_KV_TOKEN_MAJOR;
  else return none();
  const int64_t n_cache = n.sum * c.hkv * c.d;
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_dec), *k = tensor(c, a[4], kBf16, n_cache), *v = tensor(c, a[5], kBf16, n_cache);
  at::Tensor out;
  if (!q || !k || !v || !output(c, a[8], kF32, c.q_dec, {c.n_seq, c.hq, c.d}, at::kFloat, out)) return none();
  if (!call("fkv_decode_attention", [&] {
        return api.decode_attention(c.ctx, c.shape, q->data_ptr(), k->data_ptr(), v->data_ptr(), layout, n.v, f32(out), c.stream);
      }))
    return none();
  return wrap(out);
}

// (ctx, dev, shape, q, k_pages, v_pages, block_table, n_per_seq, out)
PyObject *decode_attention_paged(PyObject *const *a) {
  Call c;
  Counts n;
  Pages p;
  if (!c.open(a) || !n.read(c, a[7]) || !p.read(c, a[4], a[5], a[6])) return none();
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_dec);
  at::Tensor out;
  if (!q || !output(c, a[8], kF32, c.q_dec, {c.n_seq, c.hq, c.d}, at::kFloat, out)) return none();
  if (!call("fkv_decode_attention_paged", [&] {
        return api.decode_attention_paged(c.ctx, c.shape, q->data_ptr(), p.k->data_ptr(), p.v->data_ptr(), i32(*p.table), (int32_t)p.table->size(1),
                                          (int32_t)p.k->size(1), p.k->size(0), n.v, f32(out), c.stream);
      }))
    return none();
  return wrap(out);
}

// (ctx, dev, shape, q_win, k, v, out)
PyObject *window_output(PyObject *const *a) {
  Call c;
  if (!c.open(a)) return none();
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_win), *k = tensor(c, a[4], kBf16, c.kv), *v = tensor(c, a[5], kBf16, c.kv);
  at::Tensor out;
  if (!q || !k || !v || !output(c, a[6], kF32, c.q_win, {c.n_seq, c.shape->window, c.hq, c.d}, at::kFloat, out)) return none();
  if (!call("fkv_window_output", [&] {
        return api.window_output(c.ctx, c.shape, q->data_ptr(), k->data_ptr(), v->data_ptr(), f32(out), c.stream);
      }))
    return none();
  return wrap(out);
}

// (ctx, dev, shape, q_win, k, v, scores_group, scores_tsp, out, want_tsp)
PyObject *score_window_output(PyObject *const *a) {
  Call c;
  if (!c.open(a)) return none();
  const at::Tensor *q = tensor(c, a[3], kBf16, c.q_win), *k = tensor(c, a[4], kBf16, c.kv), *v = tensor(c, a[5], kBf16, c.kv);
  at::Tensor sg, st, out;
  if (!q || !k || !v || !output(c, a[6], kF32, c.hkv * c.sum_p, {c.hkv, c.sum_p}, at::kFloat, sg)) return none();
  if ((a[7] != Py_None || a[9] == Py_True) && !output(c, a[7], kF32, c.sum_p, {c.sum_p}, at::kFloat, st)) return none();
  if (!output(c, a[8], kF32, c.q_win, {c.n_seq, c.shape->window, c.hq, c.d}, at::kFloat, out)) return none();
  if (!call("fkv_score_window_output", [&] {
        return api.score_window_output(c.ctx, c.shape, q->data_ptr(), k->data_ptr(), v->data_ptr(), f32(sg), f32(st), f32(out), c.stream);
      }))
    return none();
  return Py_BuildValue("(NNN)", wrap(sg), wrap_or_none(st), wrap(out));
}

// bind(shape type, error type, {name: address}): the library the calls go to.
PyObject *bind(PyObject *, PyObject *args) {
  PyObject *type, *error, *addresses;
  if (!PyArg_ParseTuple(args, "O!O!O!", &PyType_Type, &type, &PyType_Type, &error, &PyDict_Type, &addresses)) return nullptr;
  bool ok = true;
  auto get = [&](auto &slot, const char *name) {
    PyObject *o = PyDict_GetItemString(addresses, name);
    void *p = o ? PyLong_AsVoidPtr(o) : nullptr;
    if (p == nullptr) ok = false;
    slot = reinterpret_cast<std::decay_t<decltype(slot)>>(p);
  };
  get(api.score_window, "fkv_score_window");
  get(api.score_heads, "fkv_score_heads");
  get(api.select_topk, "fkv_select_topk");
  get(api.gather_rows, "fkv_gather_rows");
  get(api.gather_kv, "fkv_gather_kv");
  get(api.gather_kv_per_head, "fkv_gather_kv_per_head");
  get(api.compress_kv, "fkv_compress_kv");
  get(api.compress_kv_paged, "fkv_compress_kv_paged");
  get(api.decode_attention, "fkv_decode_attention");
  get(api.decode_attention_paged, "fkv_decode_attention_paged");
  get(api.window_output, "fkv_window_output");
  get(api.score_window_output, "fkv_score_window_output");
  if (!ok) {
    shape_type = nullptr;
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: a function address is missing");
    return nullptr;
  }
  Py_INCREF(type);
  Py_INCREF(error);
  error_type = error;
  shape_type = reinterpret_cast<PyTypeObject *>(type);
  Py_RETURN_NONE;
}

#define FKV_METHOD(name, fn, n) \
  {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(guarded<fn, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    FKV_METHOD("score_window", score_window, 8),
    FKV_METHOD("score_heads", score_heads, 6),
    FKV_METHOD("select_topk", select_topk, 6),
    FKV_METHOD("gather_rows", gather_rows, 7),
    FKV_METHOD("gather_kv", gather_kv<false>, 9),
    FKV_METHOD("gather_kv_per_head", gather_kv<true>, 9),
    FKV_METHOD("compress_kv", compress_kv, 10),
    FKV_METHOD("compress_kv_paged", compress_kv_paged, 11),
    FKV_METHOD("decode_attention", decode_attention, 9),
    FKV_METHOD("decode_attention_paged", decode_attention_paged, 9),
    FKV_METHOD("window_output", window_output, 7),
    FKV_METHOD("score_window_output", score_window_output, 10),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  key_k_out = PyUnicode_InternFromString("k_out");
  key_v_out = PyUnicode_InternFromString("v_out");
  key_idx_kv = PyUnicode_InternFromString("idx_kv");
  key_x_out = PyUnicode_InternFromString("x_out");
  key_idx_tsp = PyUnicode_InternFromString("idx_tsp");
  if (!key_k_out || !key_v_out || !key_idx_kv || !key_x_out || !key_idx_tsp) return nullptr;
  return PyModule_Create(&module);
}
