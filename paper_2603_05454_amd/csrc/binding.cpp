// Native argument marshalling of the Python binding: each function takes the
// tensors of the Python call of the same name, checks what a plain pointer would
// hide (device, element type, shape, layout) and calls the C entry point on the
// current stream.  It answers with the call's status, or with None when any
// argument is not in its ordinary form - the caller then takes the general path
// in Python, which raises the error or handles the rarer form.
//
// Why: through ctypes a call cost 9-18 us on the host (attribute reads, checks and
// conversions of up to 20 arguments in the interpreter), more than many of
// the kernels behind it take; here it is 4-10 us, most of it the launch itself.
#include <Python.h>
#include <hip/hip_runtime_api.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <chrono>

#include "binding_workspace.h"
#include "lsp.h"

namespace {

// Entry points of the loaded liblsp.so (addresses handed over once by bind()).
struct Entry {
  decltype(&lsp_attn_workspace_bytes) attn_workspace_bytes;
  decltype(&lsp_attn_step) attn_step;
  decltype(&lsp_attn_step_layers) attn_step_layers;
  decltype(&lsp_confidence_workspace_bytes) confidence_workspace_bytes;
  decltype(&lsp_confidence) confidence;
  decltype(&lsp_lm_head_confidence_workspace_bytes) lm_head_confidence_workspace_bytes;
  decltype(&lsp_lm_head_confidence) lm_head_confidence;
  decltype(&lsp_commit) commit;
  decltype(&lsp_flip_update) flip_update;
  decltype(&lsp_poll_lengths) poll_lengths;
  decltype(&lsp_commit_step) commit_step;
  decltype(&lsp_poll_progress) poll_progress;
} g;
constexpr int kEntries = 12;

const at::Tensor *tensor(PyObject *o) { return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }
const at::Tensor *device_tensor(PyObject *o) {
  const at::Tensor *t = tensor(o);
  return t && t->is_cuda() ? t : nullptr;
}
// a contiguous device tensor of this element type and, where given, shape
const at::Tensor *plain(PyObject *o, at::ScalarType type, int64_t d0 = -1, int64_t d1 = -1) {
  const at::Tensor *t = device_tensor(o);
  if (!t || t->scalar_type() != type || !t->is_contiguous()) return nullptr;
  if (d0 < 0) return t;
  if (d1 < 0) return t->dim() == 1 && t->size(0) == d0 ? t : nullptr;
  return t->dim() == 2 && t->size(0) == d0 && t->size(1) == d1 ? t : nullptr;
}
bool element_type(const at::Tensor &t, int32_t &type) {
  if (t.scalar_type() == at::kBFloat16) type = LSP_BF16;
  else if (t.scalar_type() == at::kFloat) type = LSP_F32;
  else return false;
  return true;
}
template <typename T>
T *data(const at::Tensor *t) {
  return t ? static_cast<T *>(t->mutable_data_ptr()) : nullptr;
}
int64_t bytes_of(const at::Tensor *t) { return t ? int64_t(t->nbytes()) : 0; }
void *stream() { return c10::hip::getCurrentHIPStream().stream(); }
bool shape4(const at::Tensor &t, int64_t a, int64_t b, int64_t c, int64_t d) {
  return t.dim() == 4 && t.size(0) == a && t.size(1) == b && t.size(2) == c && t.size(3) == d;
}
bool strides3(const at::Tensor &t, int64_t (&s)[3]) {
  if (t.stride(3) != 1) return false;
  for (int k = 0; k < 3; ++k) s[k] = t.stride(k);
  return true;
}
bool same_strides(const at::Tensor &a, const at::Tensor &b) { return a.strides() == b.strides(); }

// false for what is not a number by itself (the general path may still make one of it)
bool number(PyObject *o, float &x) {
  x = float(PyFloat_AsDouble(o));
  if (!PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

bool integer(PyObject *o, long &x) {
  x = o ? PyLong_AsLong(o) : 0;
  if (!PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}
struct Object {  // a reference of one's own
  PyObject *o;
  explicit Object(PyObject *p) : o(p) {}
  ~Object() { Py_XDECREF(o); }
  Object(const Object &) = delete;
};
// The memory of a ctypes object, held while this lives.
struct Memory {
  Py_buffer view = {};
  Memory() = default;
  ~Memory() { PyBuffer_Release(&view); }
  Memory(const Memory &) = delete;
  bool of(PyObject *o, size_t bytes) {
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0) return size_t(view.len) >= bytes;
    PyErr_Clear();
    return false;
  }
};
// a list of N tables of `layers` pointers each
template <int N>
bool tables(PyObject *list, Memory (&tab)[N], long layers) {
  if (!list) PyErr_Clear();
  if (!list || !PyList_Check(list) || PyList_GET_SIZE(list) != N) return false;
  for (int k = 0; k < N; ++k)
    if (!tab[k].of(PyList_GET_ITEM(list, k), size_t(layers) * sizeof(void *))) return false;
  return true;
}

// The entry point itself runs without the interpreter lock: a launch waits for a full queue, and a kernel's first one
// loads its code.  What it reads of Python's is held by the caller's references meanwhile.
template <typename... P, typename... A>
int32_t unlocked(int32_t (*entry)(P...), A... args) {
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = entry(args...);
  Py_END_ALLOW_THREADS;
  return rc;
}
template <typename... P, typename... A>
PyObject *status(int32_t (*entry)(P...), A... args) {
  return PyLong_FromLong(unlocked(entry, args...));
}
#define ORDINARY(cond) \
  if (!(cond)) Py_RETURN_NONE
#define ARGUMENTS(count)                                                              \
  if (n != count) {                                                                   \
    PyErr_Format(PyExc_TypeError, "%s: %d arguments expected, got %zd", __func__, count, n); \
    return nullptr;                                                                   \
  }

PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(kEntries);
  void *p[kEntries];
  for (int k = 0; k < kEntries; ++k) p[k] = PyLong_AsVoidPtr(a[k]);
  if (PyErr_Occurred()) return nullptr;
  g.attn_workspace_bytes = reinterpret_cast<decltype(g.attn_workspace_bytes)>(p[0]);
  g.attn_step = reinterpret_cast<decltype(g.attn_step)>(p[1]);
  g.attn_step_layers = reinterpret_cast<decltype(g.attn_step_layers)>(p[2]);
  g.confidence_workspace_bytes = reinterpret_cast<decltype(g.confidence_workspace_bytes)>(p[3]);
  g.confidence = reinterpret_cast<decltype(g.confidence)>(p[4]);
  g.lm_head_confidence_workspace_bytes = reinterpret_cast<decltype(g.lm_head_confidence_workspace_bytes)>(p[5]);
  g.lm_head_confidence = reinterpret_cast<decltype(g.lm_head_confidence)>(p[6]);
  g.commit = reinterpret_cast<decltype(g.commit)>(p[7]);
  g.flip_update = reinterpret_cast<decltype(g.flip_update)>(p[8]);
  g.poll_lengths = reinterpret_cast<decltype(g.poll_lengths)>(p[9]);
  g.commit_step = reinterpret_cast<decltype(g.commit_step)>(p[10]);
  g.poll_progress = reinterpret_cast<decltype(g.poll_progress)>(p[11]);
  Py_RETURN_NONE;
}

// (q, k_suf, v_suf, k_cache, v_cache, prefix_len, suffix_len, scale, out, workspace)
PyObject *attn_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(10);
  const at::Tensor *q = device_tensor(a[0]), *ks = device_tensor(a[1]), *vs = device_tensor(a[2]), *kc = device_tensor(a[3]),
                   *vc = device_tensor(a[4]), *out = device_tensor(a[8]);
  ORDINARY(q && ks && vs && kc && vc && out && q->dim() == 4 && ks->dim() == 4 && kc->dim() == 4);
  const int64_t B = q->size(0), S = q->size(1), Hq = q->size(2), D = q->size(3), Hkv = ks->size(2), C = kc->size(1);
  const auto type = q->scalar_type();
  ORDINARY(ks->scalar_type() == type && vs->scalar_type() == type && kc->scalar_type() == type && vc->scalar_type() == type &&
           out->scalar_type() == type);
  ORDINARY(shape4(*ks, B, S, Hkv, D) && shape4(*vs, B, S, Hkv, D) && shape4(*kc, B, C, Hkv, D) && shape4(*vc, B, C, Hkv, D) &&
           shape4(*out, B, S, Hq, D) && same_strides(*ks, *vs) && same_strides(*kc, *vc));
  const at::Tensor *pl = plain(a[5], at::kInt, B), *sl = plain(a[6], at::kInt, B);
  ORDINARY(pl && sl);
  lsp_attn_desc d = {};
  ORDINARY(element_type(*q, d.dtype));
  d.B = int32_t(B); d.S = int32_t(S); d.Hq = int32_t(Hq); d.Hkv = int32_t(Hkv); d.D = int32_t(D); d.C = int32_t(C);
  ORDINARY(number(a[7], d.scale));
  ORDINARY(strides3(*q, d.q_stride) && strides3(*ks, d.kv_suf_stride) && strides3(*kc, d.cache_stride) && strides3(*out, d.o_stride));
  const Workspace work(g.attn_workspace_bytes(&d), device_tensor(a[9]));
  return status(g.attn_step, &d, q->const_data_ptr(), ks->const_data_ptr(), vs->const_data_ptr(), kc->const_data_ptr(),
                vc->const_data_ptr(), data<int32_t>(pl), data<int32_t>(sl), data<void>(out), work.at, work.bytes, stream());
}

// (table descriptor, layers, list of six tables, prefix_len, suffix_len, scale, workspace or None)
PyObject *attn_step_layers(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(7);
  Memory desc, tab[6];
  long layers;
  ORDINARY(integer(a[1], layers) && layers > 0 && desc.of(a[0], sizeof(lsp_attn_desc)) && tables(a[2], tab, layers));
  lsp_attn_desc own = *static_cast<const lsp_attn_desc *>(desc.view.buf);
  ORDINARY(number(a[5], own.scale));
  const at::Tensor *pl = plain(a[3], at::kInt, own.B), *sl = plain(a[4], at::kInt, own.B);
  ORDINARY(pl && sl);
  const Workspace work(g.attn_workspace_bytes(&own), device_tensor(a[6]));
  auto in = [&](int k) { return static_cast<const void *const *>(tab[k].view.buf); };
  return status(g.attn_step_layers, &own, int32_t(layers), in(0), in(1), in(2), in(3), in(4), data<int32_t>(pl), data<int32_t>(sl),
                static_cast<void *const *>(tab[5].view.buf), work.at, work.bytes, stream());
}

struct ConfOut {
  int32_t *id;
  float *prob, *margin;
};
bool conf_out(PyObject *o, int64_t B, int64_t S, ConfOut &r) {
  if (!PyTuple_Check(o) || PyTuple_GET_SIZE(o) != 3) return false;
  const at::Tensor *id = plain(PyTuple_GET_ITEM(o, 0), at::kInt, B, S), *prob = plain(PyTuple_GET_ITEM(o, 1), at::kFloat, B, S),
                   *margin = plain(PyTuple_GET_ITEM(o, 2), at::kFloat, B, S);
  if (!id || !prob || !margin) return false;
  r = {data<int32_t>(id), data<float>(prob), data<float>(margin)};
  return true;
}

// (logits, suffix_len or None, out, workspace or None)
PyObject *confidence(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(4);
  const at::Tensor *z = device_tensor(a[0]);
  int32_t type;
  ORDINARY(z && z->dim() == 3 && z->stride(2) == 1 && element_type(*z, type));
  const int64_t B = z->size(0), S = z->size(1), V = z->size(2);
  const at::Tensor *sl = a[1] == Py_None ? nullptr : plain(a[1], at::kInt, B);
  ORDINARY(sl || a[1] == Py_None);
  ConfOut o;
  ORDINARY(conf_out(a[2], B, S, o));
  const at::Tensor *ws = a[3] == Py_None ? nullptr : device_tensor(a[3]);
  ORDINARY(ws ? ws->is_contiguous() : a[3] == Py_None);
  // few long rows need one, which the general path allocates; one that is not aligned is found out by the call, before any launch
  ORDINARY(B * S >= 128 || bytes_of(ws) >= int64_t(g.confidence_workspace_bytes(int32_t(B), int32_t(S), int32_t(V))));
  const int32_t rc = unlocked(g.confidence, type, z->const_data_ptr(), int32_t(B), int32_t(S), int32_t(V), z->stride(1), z->stride(0),
                              data<int32_t>(sl), o.id, o.prob, o.margin, data<void>(ws), size_t(bytes_of(ws)), stream());
  ORDINARY(rc != LSP_ERR_WORKSPACE);
  return PyLong_FromLong(rc);
}

// (hidden, weight, suffix_len or None, out, workspace)
PyObject *lm_head_confidence(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(5);
  const at::Tensor *h = device_tensor(a[0]), *w = device_tensor(a[1]);
  int32_t type;
  ORDINARY(h && w && h->dim() == 3 && w->dim() == 2 && h->stride(2) == 1 && w->stride(1) == 1 && element_type(*h, type));
  const int64_t B = h->size(0), S = h->size(1), K = h->size(2), V = w->size(0);
  ORDINARY(w->size(1) == K && w->scalar_type() == h->scalar_type());
  const at::Tensor *sl = a[2] == Py_None ? nullptr : plain(a[2], at::kInt, B);
  ORDINARY(sl || a[2] == Py_None);
  ConfOut o;
  ORDINARY(conf_out(a[3], B, S, o));
  const at::Tensor *ws = device_tensor(a[4]);
  ORDINARY(ws && bytes_of(ws) >= int64_t(g.lm_head_confidence_workspace_bytes(int32_t(B), int32_t(S), int32_t(V))));
  return status(g.lm_head_confidence, type, h->const_data_ptr(), w->const_data_ptr(), int32_t(B), int32_t(S), int32_t(K), int32_t(V),
                h->stride(1), h->stride(0), w->stride(0), data<int32_t>(sl), o.id, o.prob, o.margin,
                data<void>(ws), size_t(bytes_of(ws)), stream());
}

// int32[4] of host memory, as lsp_poll_lengths wants it
int32_t *host_words(PyObject *o) {
  const at::Tensor *t = tensor(o);
  return t && t->is_cpu() && t->scalar_type() == at::kInt && t->is_contiguous() && t->numel() >= 4 ? data<int32_t>(t) : nullptr;
}

PyObject *k_mask, *k_raw, *k_snapped, *k_len, *k_flags, *k_tau;  // keys of commit's result
// attributes of a layer table: the tables, then numbers
PyObject *k_arrays, *k_numbers[9];
constexpr const char *kNumbers[9] = {"kv_dtype", "B", "S", "Hkv", "D", "C", "n", "suf_bs", "cache_bs"};

// (margin, top1_id, bitmap, prefix_len, suffix_len, tokens or None, layer table or None, out,
//  (V, tau, window, min_commit, snap_enabled, adaptive, alpha, beta, max_commit, C))
// STEP: and (base_prefix_len, last_id, counters, window_lo, window_hi, step_counts or None)
template <bool STEP>
PyObject *commit(PyObject *, PyObject *const *a, Py_ssize_t n) {
  constexpr int kArguments = STEP ? 10 : 9;
  ARGUMENTS(kArguments);
  ORDINARY(PyDict_Check(a[7]) && PyDict_GET_SIZE(a[7]) == 6 && PyTuple_Check(a[8]) && PyTuple_GET_SIZE(a[8]) == 10);
  const at::Tensor *margin = device_tensor(a[0]);
  ORDINARY(margin && margin->dim() == 2);
  const int64_t B = margin->size(0), S = margin->size(1);
  margin = plain(a[0], at::kFloat, B, S);
  const at::Tensor *id = plain(a[1], at::kInt, B, S), *pl = plain(a[3], at::kInt, B), *sl = plain(a[4], at::kInt, B);
  const at::Tensor *bm = device_tensor(a[2]);
  ORDINARY(margin && id && pl && sl && bm && bm->is_contiguous() && (bm->scalar_type() == at::kInt || bm->scalar_type() == at::kUInt32));
  const at::Tensor *tokens = a[5] == Py_None ? nullptr : device_tensor(a[5]);
  ORDINARY(a[5] == Py_None || (tokens && tokens->dim() == 2 && plain(a[5], at::kInt, B, tokens->size(1))));
  long i[10];
  double f[10];
  for (int k = 0; k < 10; ++k) {
    PyObject *x = PyTuple_GET_ITEM(a[8], k);
    if (k == 1 || k == 6 || k == 7) f[k] = PyFloat_AsDouble(x);
    else i[k] = PyLong_AsLong(x);
  }
  if (PyErr_Occurred()) {  // a number of an unusual type
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  ORDINARY(bm->numel() >= (i[0] + 31) / 32);
  lsp_commit_desc d = {};
  d.B = int32_t(B); d.S = int32_t(S); d.V = int32_t(i[0]); d.tau = float(f[1]); d.window = int32_t(i[2]); d.min_commit = int32_t(i[3]);
  d.snap_enabled = int32_t(i[4]); d.adaptive = i[5] != 0; d.alpha = float(f[6]); d.beta = float(f[7]); d.max_commit = int32_t(i[8]);
  d.T = tokens ? int32_t(tokens->size(1)) : 0;
  Memory tab[4];
  if (a[6] != Py_None) {
    long t[9];
    for (int k = 0; k < 9; ++k) {
      Object x(PyObject_GetAttr(a[6], k_numbers[k]));
      ORDINARY(integer(x.o, t[k]));
    }
    Object arrays(PyObject_GetAttr(a[6], k_arrays));
    ORDINARY(t[1] == B && t[2] == S && t[6] > 0 && tables(arrays.o, tab, t[6]));
    d.kv_dtype = int32_t(t[0]); d.Hkv = int32_t(t[3]); d.D = int32_t(t[4]); d.C = int32_t(t[5]); d.num_layers = int32_t(t[6]);
    d.suf_batch_stride = t[7]; d.cache_batch_stride = t[8];
  } else {
    d.C = int32_t(i[9]);
  }
  auto per_sequence = [&](PyObject *key, at::ScalarType type) -> const at::Tensor * {
    PyObject *o = PyDict_GetItemWithError(a[7], key);
    return o ? plain(o, type, B) : nullptr;
  };
  PyObject *mask_o = PyDict_GetItemWithError(a[7], k_mask);
  const at::Tensor *mask = mask_o ? plain(mask_o, at::kByte, B, S) : nullptr, *raw = per_sequence(k_raw, at::kInt),
                   *snapped = per_sequence(k_snapped, at::kInt), *len = per_sequence(k_len, at::kInt),
                   *flags = per_sequence(k_flags, at::kInt), *tau = per_sequence(k_tau, at::kFloat);
  if (PyErr_Occurred()) return nullptr;
  ORDINARY(mask && raw && snapped && len && flags && tau);
  if constexpr (STEP) {
    ORDINARY(PyTuple_Check(a[9]) && PyTuple_GET_SIZE(a[9]) == 6);
    PyObject *const *x = &PyTuple_GET_ITEM(a[9], 0);
    const at::Tensor *last = device_tensor(x[1]);
    ORDINARY(last && last->dim() == 2);
    const int64_t G = last->size(1);
    last = plain(x[1], at::kInt, B, G);
    const at::Tensor *base = plain(x[0], at::kInt, B), *counters = plain(x[2], at::kLong, 4),
                     *steps = x[5] == Py_None ? nullptr : plain(x[5], at::kInt, B, 2);
    ORDINARY(base && last && counters && (steps || x[5] == Py_None));
    const long lo = PyLong_AsLong(x[3]), hi = PyLong_AsLong(x[4]);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
    return status(g.commit_step, &d, data<float>(margin), data<int32_t>(id), data<uint32_t>(bm), static_cast<const void *const *>(tab[0].view.buf),
                  static_cast<const void *const *>(tab[1].view.buf), static_cast<void *const *>(tab[2].view.buf),
                  static_cast<void *const *>(tab[3].view.buf), data<int32_t>(tokens), data<int32_t>(pl), data<int32_t>(sl), data<uint8_t>(mask),
                  data<int32_t>(raw), data<int32_t>(snapped), data<int32_t>(len), data<int32_t>(flags), data<float>(tau), int32_t(G),
                  data<int32_t>(base), data<int32_t>(last), data<int64_t>(counters), int32_t(lo), int32_t(hi), data<int32_t>(steps), stream());
  }
  return status(g.commit, &d, data<float>(margin), data<int32_t>(id), data<uint32_t>(bm), static_cast<const void *const *>(tab[0].view.buf),
                static_cast<const void *const *>(tab[1].view.buf), static_cast<void *const *>(tab[2].view.buf),
                static_cast<void *const *>(tab[3].view.buf), data<int32_t>(tokens), data<int32_t>(pl), data<int32_t>(sl), data<uint8_t>(mask),
                data<int32_t>(raw), data<int32_t>(snapped), data<int32_t>(len),
                data<int32_t>(flags), data<float>(tau), nullptr, 0, stream());
}

// (top1_id, prefix_len, suffix_len, base_prefix_len, last_id, counters, window_lo, window_hi, step_counts or None)
PyObject *flip_update(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(9);
  const at::Tensor *id = device_tensor(a[0]), *last = device_tensor(a[4]);
  ORDINARY(id && id->dim() == 2 && last && last->dim() == 2);
  const int64_t B = id->size(0), S = id->size(1), G = last->size(1);
  id = plain(a[0], at::kInt, B, S);
  last = plain(a[4], at::kInt, B, G);
  const at::Tensor *pl = plain(a[1], at::kInt, B), *sl = plain(a[2], at::kInt, B), *base = plain(a[3], at::kInt, B),
                   *counters = plain(a[5], at::kLong, 4), *steps = a[8] == Py_None ? nullptr : plain(a[8], at::kInt, B, 2);
  ORDINARY(id && last && pl && sl && base && counters && (steps || a[8] == Py_None));
  const long lo = PyLong_AsLong(a[6]), hi = PyLong_AsLong(a[7]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  return status(g.flip_update, data<int32_t>(id), int32_t(B), int32_t(S), int32_t(G), data<int32_t>(pl), data<int32_t>(sl),
                data<int32_t>(base), data<int32_t>(last), data<int64_t>(counters), int32_t(lo), int32_t(hi),
                data<int32_t>(steps), stream());
}

struct Unlocked {  // the interpreter lock is given back until the end of the scope, also by an exception
  PyThreadState *state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
// (suffix_len, commit_len or None, host): launches lsp_poll_lengths and waits; host is pinned memory of the caller's own.
// Answers (left, stalled), or the status of a failed launch.
PyObject *poll_lengths(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(3);
  const at::Tensor *sl = device_tensor(a[0]);
  ORDINARY(sl && sl->dim() == 1);
  const int64_t B = sl->size(0);
  sl = plain(a[0], at::kInt, B);
  const at::Tensor *len = a[1] == Py_None ? nullptr : plain(a[1], at::kInt, B);
  int32_t *h = host_words(a[2]);
  ORDINARY(sl && (len || a[1] == Py_None) && h);
  __atomic_store_n(h + 2, 0, __ATOMIC_RELAXED);
  const int32_t rc = unlocked(g.poll_lengths, data<int32_t>(sl), data<int32_t>(len), int32_t(B), h, stream());
  if (rc != LSP_OK) return PyLong_FromLong(rc);
  {
    // the flag comes some microseconds before the runtime would tell; a long step is left to the runtime
    Unlocked without_lock;
    const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(2);
    while (!__atomic_load_n(h + 2, __ATOMIC_ACQUIRE))
      if (std::chrono::steady_clock::now() > until) {
        c10::hip::getCurrentHIPStream().synchronize();
        break;
      }
  }
  return Py_BuildValue("(ii)", int(h[0]), int(h[1]));
}
constexpr int kProgressWords = 12;
uint64_t *progress_words(PyObject *o) {
  const at::Tensor *t = tensor(o);
  return t && t->is_cpu() && t->scalar_type() == at::kLong && t->is_contiguous() && t->numel() >= kProgressWords ? data<uint64_t>(t) : nullptr;
}
// (suffix_len, commit_len or None, prefix_len, base_prefix_len, counters, host, call): launches lsp_poll_progress.
PyObject *poll_start(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(7);
  const at::Tensor *sl = device_tensor(a[0]);
  ORDINARY(sl && sl->dim() == 1);
  const int64_t B = sl->size(0);
  sl = plain(a[0], at::kInt, B);
  const at::Tensor *len = a[1] == Py_None ? nullptr : plain(a[1], at::kInt, B), *pl = plain(a[2], at::kInt, B),
                   *base = plain(a[3], at::kInt, B), *counters = plain(a[4], at::kLong, 4);
  uint64_t *h = progress_words(a[5]);
  long call;
  ORDINARY(sl && (len || a[1] == Py_None) && pl && base && counters && h && integer(a[6], call));
  return status(g.poll_progress, data<int32_t>(sl), data<int32_t>(len), data<int32_t>(pl), data<int32_t>(base), data<int64_t>(counters),
                int32_t(B), uint32_t(call), h, stream());
}
// (host, call): waits up to 2 ms for that call's words and answers their lower halves, or None: the words come some microseconds before the
// runtime would tell, and a longer step is left to the runtime.
PyObject *poll_wait(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(2);
  const uint64_t *h = progress_words(a[0]);
  long call;
  ORDINARY(h && integer(a[1], call));
  uint64_t got[kProgressWords];
  auto all = [&] {
    bool here = true;
    for (int k = 0; k < kProgressWords; ++k) {
      got[k] = __atomic_load_n(h + k, __ATOMIC_ACQUIRE);
      here = here && uint32_t(got[k] >> 32) == uint32_t(call);
    }
    return here;
  };
  bool here;
  {
    Unlocked without_lock;
    const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(2);
    while (!(here = all()) && std::chrono::steady_clock::now() < until) {
    }
  }
  ORDINARY(here);
  auto wide = [&](int k) { return (long long)(uint64_t(uint32_t(got[k + 1])) << 32 | uint32_t(got[k])); };
  return Py_BuildValue("(iiLLLLL)", int(uint32_t(got[0])), int(uint32_t(got[1])), wide(2), wide(4), wide(6), wide(8), wide(10));
}
// Addresses of a list of device tensors that share shape, strides and element type, as bytes.
PyObject *addresses(PyObject *, PyObject *const *a, Py_ssize_t n) {
  ARGUMENTS(1);
  ORDINARY(PyList_Check(a[0]) && PyList_GET_SIZE(a[0]) > 0);
  const Py_ssize_t count = PyList_GET_SIZE(a[0]);
  Object bytes(PyBytes_FromStringAndSize(nullptr, count * Py_ssize_t(sizeof(void *))));
  if (!bytes.o) return nullptr;
  auto *out = reinterpret_cast<void **>(PyBytes_AS_STRING(bytes.o));
  const at::Tensor *first = device_tensor(PyList_GET_ITEM(a[0], 0));
  ORDINARY(first);
  for (Py_ssize_t k = 0; k < count; ++k) {
    const at::Tensor *t = device_tensor(PyList_GET_ITEM(a[0], k));
    ORDINARY(t && t->scalar_type() == first->scalar_type() && t->sizes() == first->sizes() && t->strides() == first->strides());
    out[k] = t->mutable_data_ptr();
  }
  Py_INCREF(bytes.o);
  return bytes.o;
}

// No C++ exception may reach the interpreter: torch throws where a tensor has no strides or no
// storage (sparse, batched by vmap), there is no device or a subclass written in Python raises (the error is then
// set as well), and the general path meets the same and raises it.
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  try {
    return F(self, a, n);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyMethodDef fast(const char *name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<F>)), METH_FASTCALL, nullptr};
}
PyMethodDef methods[] = {fast<bind>("bind"), fast<attn_step>("attn_step"), fast<attn_step_layers>("attn_step_layers"),
                         fast<confidence>("confidence"), fast<lm_head_confidence>("lm_head_confidence"), fast<commit<false>>("commit"), fast<commit<true>>("commit_step"),
                         fast<flip_update>("flip_update"), fast<poll_lengths>("poll_lengths"),
                         fast<poll_start>("poll_start"), fast<poll_wait>("poll_wait"), fast<addresses>("addresses"), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  k_mask = PyUnicode_InternFromString("stable_mask");
  k_raw = PyUnicode_InternFromString("raw_boundary");
  k_snapped = PyUnicode_InternFromString("snapped_boundary");
  k_len = PyUnicode_InternFromString("commit_len");
  k_flags = PyUnicode_InternFromString("status_flags");
  k_tau = PyUnicode_InternFromString("tau_used");
  k_arrays = PyUnicode_InternFromString("arrays");
  for (int k = 0; k < 9; ++k) k_numbers[k] = PyUnicode_InternFromString(kNumbers[k]);
  return PyModule_Create(&module);
}
