// Argument marshalling of the Python binding: checks the tensors of a call (device, contiguity, type, shape), takes their
// pointers and the current stream, and calls the C ABI without the GIL.  No step of the method happens here.
//
// Native because a small launch is shorter than the same checks in Python: twelve to twenty attribute look-ups and tuple
// comparisons per call cost 5 to 14 us, next to 3 us for a launch (hf_pool_keys 8.2 -> 3.0 us per call, a two-call step of a
// small stream 25 -> 7 us).  The entry points come as addresses from the library that the binding loaded; this file links
// against Python and torch only.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <string>
#include <vector>

#include "hf.h"

namespace {

#define HF_ENTRIES(X)                                                                                                      \
  X(hf_last_error) X(hf_state_bytes) X(hf_select_k) X(hf_state_init) X(hf_state_fold_linear) X(hf_absorb_evicted)           \
  X(hf_state_planes) X(hf_absorb_evicted_planes) X(hf_window_evict) X(hf_block_select) X(hf_block_select_cached)            \
  X(hf_block_select_static) X(hf_hybrid_attn_fwd) X(hf_hybrid_attn_fwd_split) X(hf_hybrid_attn_fwd_planes) X(hf_pool_keys)  \
  X(hf_select_attn_fwd) X(hf_step_fwd) X(hf_hybrid_attn_fwd_save) X(hf_rope_window_indices) X(hf_rope_tables)               \
  X(hf_rope_append_keys) X(hf_rope_apply) X(hf_stream_open_chunk) X(hf_stream_step) X(hf_ring_open_chunk) X(hf_ring_step)   \
  X(hf_ring_last_step) X(hf_hybrid_attn_bwd) X(hf_hybrid_attn_bwd_saved)

#define HF_POINTER(name) decltype(&::name) name = nullptr;
struct {
  HF_ENTRIES(HF_POINTER)
} lib;
PyObject* error_class = nullptr;   // HFError(code, message)

struct Raised {};                  // the Python error is set

template <class... A> [[noreturn]] void raise(PyObject* type, const char* format, A... a) {
  PyErr_Format(type, format, a...);
  throw Raised();
}

void check(int code) {
  if (code == HF_OK) return;
  PyObject* e = PyObject_CallFunction(error_class, "is", code, lib.hf_last_error());
  if (e) {
    PyErr_SetObject(error_class, e);
    Py_DECREF(e);
  }
  throw Raised();
}

// the binding's class of a structure
template <class T> struct Class { static PyTypeObject* type; };
template <class T> PyTypeObject* Class<T>::type = nullptr;

// the memory of a ctypes structure
template <class T> struct Struct {
  Py_buffer b;
  Struct(PyObject* o, const char* name) {
    if (!PyObject_TypeCheck(o, Class<T>::type)) raise(PyExc_TypeError, "%s must be an %s structure, got %s", name, name, Py_TYPE(o)->tp_name);
    if (PyObject_GetBuffer(o, &b, PyBUF_WRITABLE) < 0) throw Raised();
  }
  Struct(const Struct&) = delete;
  ~Struct() { PyBuffer_Release(&b); }
  T* get() const { return static_cast<T*>(b.buf); }
  T* operator->() const { return get(); }
};

typedef std::initializer_list<int64_t> Shape;

std::string text(at::IntArrayRef s) {
  std::string r = "(";
  for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
  return r + (s.size() == 1 ? ",)" : ")");
}

const char* dtype_name(at::ScalarType t) {
  switch (t) {
    case at::kBFloat16: return "torch.bfloat16";
    case at::kFloat: return "torch.float32";
    case at::kInt: return "torch.int32";
    case at::kByte: return "torch.uint8";
    default: return c10::toString(t);
  }
}

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s must be a GPU tensor", name);
  return THPVariable_Unpack(o);
}

int64_t length(PyObject* o, const char* name, int dim, int dims = 4) {
  const at::Tensor& t = tensor(o, name);
  if (t.dim() != dims) raise(PyExc_ValueError, "%s must have %d dimensions, got %d", name, dims, (int)t.dim());
  return t.size(dim);
}

void* ptr(PyObject* o, const char* name, at::ScalarType type) {
  if (o == Py_None) return nullptr;   // (the library says where NULL is not allowed)
  const at::Tensor& t = tensor(o, name);
  if (!t.is_cuda()) raise(PyExc_TypeError, "%s must be a GPU tensor", name);
  if (!t.is_contiguous()) raise(PyExc_ValueError, "%s must be contiguous", name);
  if (t.scalar_type() != type) raise(PyExc_TypeError, "%s must be %s, got %s", name, dtype_name(type), dtype_name(t.scalar_type()));
  return t.data_ptr();
}

void* ptr(PyObject* o, const char* name, at::ScalarType type, Shape shape) {
  void* p = ptr(o, name, type);
  if (o == Py_None) return p;
  const at::IntArrayRef got = THPVariable_Unpack(o).sizes(), want(shape.begin(), shape.size());
  if (got != want) raise(PyExc_ValueError, "%s must have shape %s, got %s", name, text(want).c_str(), text(got).c_str());
  return p;
}

float* f32(PyObject* o, const char* name, Shape shape) { return static_cast<float*>(ptr(o, name, at::kFloat, shape)); }
int32_t* i32(PyObject* o, const char* name, Shape shape) { return static_cast<int32_t*>(ptr(o, name, at::kInt, shape)); }
void* bytes(PyObject* o, const char* name) { return ptr(o, name, at::kByte); }
size_t size_of(PyObject* o) { return o == Py_None ? 0 : (size_t)THPVariable_Unpack(o).numel(); }   // after bytes()

int narrow(PyObject* n) {   // takes the reference
  if (!n) throw Raised();
  const long v = PyLong_AsLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw Raised();
  if (v != (long)(int)v) raise(PyExc_OverflowError, "%ld does not fit in 32 bits", v);
  return (int)v;
}

int to_int(PyObject* o) { return narrow(PyNumber_Long(o)); }     // what int() takes
int index(PyObject* o) { return narrow(PyNumber_Index(o)); }     // whole numbers only

bool equals(PyObject* o, int64_t v) {
  PyObject* n = PyLong_FromLongLong(v);
  if (!n) throw Raised();
  const int same = PyObject_RichCompareBool(o, n, Py_EQ);
  Py_DECREF(n);
  if (same < 0) throw Raised();
  return same;
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

int cdiv(int a, int b) { return (a + b - 1) / b; }

struct Config : Struct<hf_config> {
  at::ScalarType type;
  int64_t B, H, D;
  explicit Config(PyObject* o) : Struct(o, "hf_config") {
    type = get()->dtype == HF_BF16 ? at::kBFloat16 : at::kFloat;
    B = get()->batch;
    H = get()->heads;
    D = get()->head_dim;
    if (get()->block_q < 1 || get()->block_kv < 1) {   // (t_m and t_n divide by them): the library's own error
      size_t n = 0;
      check(lib.hf_state_bytes(get(), &n));
    }
  }
  void* tokens(PyObject* o, const char* name, int64_t n) const { return ptr(o, name, type, {B, H, n, D}); }
  float* table(PyObject* o, const char* name, int64_t n) const { return f32(o, name, {n, D / 2}); }
  float* state(PyObject* o, const char* name) const {
    size_t n = 0;
    check(lib.hf_state_bytes(get(), &n));
    return f32(o, name, {(int64_t)(n / 4)});
  }
  int t_m(int n_q) const { return cdiv(n_q, get()->block_q); }
  int t_n(int n_kv) const { return cdiv(n_kv, get()->block_kv); }
  int select_k(int n_kv) const {
    int32_t k = 0;
    check(lib.hf_select_k(get(), n_kv, &k));
    return k;
  }
  // valid tokens of a window tensor: its length when packed, the caller's n_kv in a cache buffer
  int kv_len(int64_t held, PyObject* n_kv) const {
    if (get()->kv_capacity > 0) {
      if (n_kv == Py_None) raise(PyExc_ValueError, "n_kv must be given when cfg.kv_capacity is set");
      if (held != get()->kv_capacity) raise(PyExc_ValueError, "K_win must hold kv_capacity=%d tokens per head", (int)get()->kv_capacity);
      return to_int(n_kv);
    }
    if (n_kv != Py_None && !equals(n_kv, held)) raise(PyExc_ValueError, "n_kv differs from the packed window length");
    return (int)held;
  }
};

// the call itself, without the GIL.  A type, not a function: a braced list is evaluated in its order, so of several bad arguments
// the first is reported, and the stream is asked for behind the checks
struct call {
  template <class F, class... A> call(F f, A... a) {
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = f(a...);
    Py_END_ALLOW_THREADS
    check(code);
  }
};

typedef PyObject* const* Args;
PyObject* none() { Py_RETURN_NONE; }

PyObject* state_init(Args a) {   // cfg, state
  const Config c(a[0]);
  call{lib.hf_state_init, c.get(), c.state(a[1], "state"), stream()};
  return none();
}

PyObject* state_fold_linear(Args a) {   // cfg, state_in, W, state_out
  const Config c(a[0]);
  call{lib.hf_state_fold_linear, c.get(), c.state(a[1], "state_in"), f32(a[2], "W", {c.H, c.D, c.D}), c.state(a[3], "state_out"), stream()};
  return none();
}

PyObject* state_planes(Args a) {   // cfg, state, planes_out
  const Config c(a[0]);
  call{lib.hf_state_planes, c.get(), c.state(a[1], "state"), bytes(a[2], "planes_out"), stream()};
  return none();
}

PyObject* absorb_evicted(Args a) {   // cfg, state, K_ev, V_ev, rope_cos, rope_sin, workspace
  const Config c(a[0]);
  const int n = (int)length(a[2], "K_ev", 2);
  call{lib.hf_absorb_evicted, c.get(), c.state(a[1], "state"), c.tokens(a[2], "K_ev", n), c.tokens(a[3], "V_ev", n), n,
       c.table(a[4], "rope_cos", n), c.table(a[5], "rope_sin", n), bytes(a[6], "workspace"), size_of(a[6]), stream()};
  return none();
}

PyObject* absorb_evicted_planes(Args a) {   // cfg, state, K_ev, V_ev, planes_out, rope_cos, rope_sin, workspace
  const Config c(a[0]);
  const int n = (int)length(a[2], "K_ev", 2);
  call{lib.hf_absorb_evicted_planes, c.get(), c.state(a[1], "state"), c.tokens(a[2], "K_ev", n), c.tokens(a[3], "V_ev", n), n,
       c.table(a[5], "rope_cos", n), c.table(a[6], "rope_sin", n), bytes(a[7], "workspace"), size_of(a[7]),
       bytes(a[4], "planes_out"), stream()};
  return none();
}

PyObject* window_evict(Args a) {   // cfg, K_win, V_win, n_evict, state, rope_cos, rope_sin, workspace, n_sink, n_kv
  const Config c(a[0]);
  const int64_t held = length(a[1], "K_win", 2);
  const int n_kv = c.kv_len(held, a[9]), n = to_int(a[3]);
  call{lib.hf_window_evict, c.get(), c.tokens(a[1], "K_win", held), c.tokens(a[2], "V_win", held), n_kv, to_int(a[8]), n,
       c.state(a[4], "state"), c.table(a[5], "rope_cos", n), c.table(a[6], "rope_sin", n),
       bytes(a[7], "workspace"), size_of(a[7]), stream()};
  return none();
}

PyObject* block_select(Args a) {   // cfg, Q, K_win, n_cached or None, block_idx, scores, workspace, n_kv
  const Config c(a[0]);
  const int n_q = (int)length(a[1], "Q", 2);
  const int64_t held = length(a[2], "K_win", 2);
  const int n_kv = c.kv_len(held, a[7]), k = c.select_k(n_kv);
  void* ws = bytes(a[6], "workspace");
  const void *q = c.tokens(a[1], "Q", n_q), *kw = c.tokens(a[2], "K_win", held);
  int32_t* idx = i32(a[4], "block_idx", {c.B, c.H, c.t_m(n_q), k});
  float* sc = f32(a[5], "scores", {c.B, c.H, c.t_m(n_q), c.t_n(n_kv)});
  if (a[3] == Py_None) call{lib.hf_block_select, c.get(), q, n_q, kw, n_kv, idx, sc, ws, size_of(a[6]), stream()};
  else call{lib.hf_block_select_cached, c.get(), q, n_q, kw, n_kv, to_int(a[3]), idx, sc, ws, size_of(a[6]), stream()};
  return none();
}

PyObject* block_select_static(Args a) {   // cfg, Q, K_win, block_idx, scores, n_kv
  const Config c(a[0]);
  const int n_q = (int)length(a[1], "Q", 2);
  const int64_t held = length(a[2], "K_win", 2);
  const int n_kv = c.kv_len(held, a[5]), k = c.select_k(n_kv);
  call{lib.hf_block_select_static, c.get(), c.tokens(a[1], "Q", n_q), n_q, c.tokens(a[2], "K_win", held), n_kv,
       i32(a[3], "block_idx", {c.B, c.H, c.t_m(n_q), k}), f32(a[4], "scores", {c.B, c.H, c.t_m(n_q), c.t_n(n_kv)}), stream()};
  return none();
}

// Q, K_win, V_win and an optional block list, as every attention call takes them
struct Attn {
  int n_q, n_kv, k = 0;
  int64_t held;
  const void *q, *kw, *vw, *q_hist;
  const int32_t* idx;
  Attn(const Config& c, PyObject* Q, PyObject* K, PyObject* V, PyObject* block_idx, PyObject* Q_hist, PyObject* n_kv_arg) {
    n_q = (int)length(Q, "Q", 2);
    held = length(K, "K_win", 2);
    n_kv = c.kv_len(held, n_kv_arg);
    if (block_idx != Py_None) {
      if (tensor(block_idx, "block_idx").dim() != 4) raise(PyExc_ValueError, "block_idx must be [B, H, T_m, k]");
      k = (int)THPVariable_Unpack(block_idx).size(3);
    }
    q = c.tokens(Q, "Q", n_q);
    q_hist = c.tokens(Q_hist, "Q_hist", n_q);
    kw = c.tokens(K, "K_win", held);
    vw = c.tokens(V, "V_win", held);
    idx = i32(block_idx, "block_idx", {c.B, c.H, c.t_m(n_q), k});
  }
};

PyObject* hybrid_attn_fwd(Args a) {   // cfg, Q, K_win, V_win, block_idx, state, O, workspace, rope_cos_q, rope_sin_q, Q_hist, n_kv
  const Config c(a[0]);
  const Attn t(c, a[1], a[2], a[3], a[4], a[10], a[11]);
  const float *st = c.state(a[5], "state"), *cs = c.table(a[8], "rope_cos_q", t.n_q), *sn = c.table(a[9], "rope_sin_q", t.n_q);
  void *o = c.tokens(a[6], "O", t.n_q), *ws = bytes(a[7], "workspace");
  if (a[10] == Py_None)
    call{lib.hf_hybrid_attn_fwd, c.get(), t.q, t.n_q, t.kw, t.vw, t.n_kv, t.idx, t.k, st, cs, sn, o, ws, size_of(a[7]), stream()};
  else
    call{lib.hf_hybrid_attn_fwd_split, c.get(), t.q, t.q_hist, t.n_q, t.kw, t.vw, t.n_kv, t.idx, t.k, st, cs, sn, o, ws,
         size_of(a[7]), stream()};
  return none();
}

PyObject* hybrid_attn_fwd_planes(Args a) {   // cfg, Q, K_win, V_win, block_idx, state, planes, O, rope_cos_q, rope_sin_q, Q_hist, n_kv
  const Config c(a[0]);
  const Attn t(c, a[1], a[2], a[3], a[4], a[10], a[11]);
  call{lib.hf_hybrid_attn_fwd_planes, c.get(), t.q, t.q_hist, t.n_q, t.kw, t.vw, t.n_kv, t.idx, t.k, c.state(a[5], "state"),
       bytes(a[6], "planes"), c.table(a[8], "rope_cos_q", t.n_q), c.table(a[9], "rope_sin_q", t.n_q), c.tokens(a[7], "O", t.n_q),
       stream()};
  return none();
}

PyObject* hybrid_attn_fwd_save(Args a) {   // cfg, Q, K_win, V_win, block_idx, state, O, O_local_out, lse2_out, workspace, cos, sin, Q_hist, n_kv
  const Config c(a[0]);
  const Attn t(c, a[1], a[2], a[3], a[4], a[12], a[13]);
  call{lib.hf_hybrid_attn_fwd_save, c.get(), t.q, t.q_hist, t.n_q, t.kw, t.vw, t.n_kv, t.idx, t.k, c.state(a[5], "state"),
       c.table(a[10], "rope_cos_q", t.n_q), c.table(a[11], "rope_sin_q", t.n_q), c.tokens(a[6], "O", t.n_q),
       c.tokens(a[7], "O_local_out", t.n_q), f32(a[8], "lse2_out", {c.B * c.H, t.n_q}),
       bytes(a[9], "workspace"), size_of(a[9]), stream()};
  return none();
}

PyObject* pool_keys(Args a) {   // cfg, K_win, pooled_K, n_cached_kv_blocks, n_kv
  const Config c(a[0]);
  const int64_t held = length(a[1], "K_win", 2);
  const int n_kv = c.kv_len(held, a[4]);
  call{lib.hf_pool_keys, c.get(), c.tokens(a[1], "K_win", held), n_kv, index(a[3]), bytes(a[2], "pooled_K"), stream()};
  return none();
}

// the list that a selecting launch writes has to hold exactly what it chooses
int32_t* list_out(const Config& c, PyObject* o, int n_q, int n_kv) {
  if (tensor(o, "block_idx_out").dim() != 4) raise(PyExc_ValueError, "block_idx_out must be [B, H, T_m, k]");
  const int k = c.select_k(n_kv);
  if (THPVariable_Unpack(o).size(3) != k) raise(PyExc_ValueError, "block_idx_out must hold hf_select_k(cfg, n_kv) entries per row");
  return i32(o, "block_idx_out", {c.B, c.H, c.t_m(n_q), k});
}

PyObject* select_attn_fwd(Args a) {   // cfg, Q, K_win, V_win, pooled_K, state, planes, O, block_idx_out, scores, cos, sin, Q_hist, n_kv
  const Config c(a[0]);
  const Attn t(c, a[1], a[2], a[3], Py_None, a[12], a[13]);
  int32_t* idx = list_out(c, a[8], t.n_q, t.n_kv);
  call{lib.hf_select_attn_fwd, c.get(), t.q, t.q_hist, t.n_q, t.kw, t.vw, t.n_kv, bytes(a[4], "pooled_K"), c.state(a[5], "state"),
       bytes(a[6], "planes"), c.table(a[10], "rope_cos_q", t.n_q), c.table(a[11], "rope_sin_q", t.n_q), c.tokens(a[7], "O", t.n_q),
       idx, f32(a[9], "scores", {c.B, c.H, c.t_m(t.n_q), c.t_n(t.n_kv)}), stream()};
  return none();
}

// cfg, Q, K_win, V_win, pooled_K, state_in, planes, O, block_idx_out, K_ev, V_ev, state_out, planes_out, workspace, scores, cos,
// sin, Q_hist, n_kv, n_ev
PyObject* step_fwd(Args a) {
  const Config c(a[0]);
  const Attn t(c, a[1], a[2], a[3], Py_None, a[17], a[18]);
  int32_t* idx = list_out(c, a[8], t.n_q, t.n_kv);
  const int ev_stride = (int)length(a[9], "K_ev", 2), n_ev = a[19] == Py_None ? ev_stride : to_int(a[19]);
  call{lib.hf_step_fwd, c.get(), t.q, t.q_hist, t.n_q, t.kw, t.vw, t.n_kv, bytes(a[4], "pooled_K"), c.state(a[5], "state_in"),
       bytes(a[6], "planes"), c.table(a[15], "rope_cos_q", t.n_q), c.table(a[16], "rope_sin_q", t.n_q), c.tokens(a[7], "O", t.n_q),
       idx, f32(a[14], "scores", {c.B, c.H, c.t_m(t.n_q), c.t_n(t.n_kv)}), c.tokens(a[9], "K_ev", ev_stride),
       c.tokens(a[10], "V_ev", ev_stride), n_ev, ev_stride, c.state(a[11], "state_out"), bytes(a[12], "planes_out"),
       bytes(a[13], "workspace"),
       size_of(a[13]), stream()};
  return none();
}

PyObject* rope_window_indices(Args a) {   // i_newest, n_frames, t0
  const int n = index(a[1]);
  std::vector<int32_t> out(n > 0 ? n : 1);   // (an empty one has no address: the library would name that, not the number)
  check(lib.hf_rope_window_indices(to_int(a[0]), n, to_int(a[2]), out.data()));
  PyObject* list = PyList_New(n);
  if (!list) throw Raised();
  for (int i = 0; i < n; ++i) PyList_SET_ITEM(list, i, PyLong_FromLong(out[i]));
  return list;
}

PyObject* rope_tables(Args a) {   // frame_idx, height, width, pairs, cos_out, sin_out, theta, temporal_only
  auto ints = [](PyObject* o) {
    PyObject* s = PySequence_Fast(o, "a sequence of integers is needed");
    if (!s) throw Raised();
    std::vector<int32_t> v((size_t)PySequence_Fast_GET_SIZE(s));
    try {
      for (size_t i = 0; i < v.size(); ++i) v[i] = to_int(PySequence_Fast_GET_ITEM(s, (Py_ssize_t)i));
    } catch (Raised&) {
      Py_DECREF(s);
      throw;
    }
    Py_DECREF(s);
    return v;
  };
  const std::vector<int32_t> frames = ints(a[0]), pairs = ints(a[3]);
  if (pairs.size() != 3) raise(PyExc_ValueError, "pairs must be three numbers");
  const int height = to_int(a[1]), width = to_int(a[2]);
  const double theta = PyFloat_AsDouble(a[6]);
  if (theta == -1.0 && PyErr_Occurred()) throw Raised();
  const int temporal = PyObject_IsTrue(a[7]);
  if (temporal < 0) throw Raised();
  const int64_t rows = (int64_t)frames.size() * height * width, cols = (int64_t)pairs[0] + pairs[1] + pairs[2];
  call{lib.hf_rope_tables, frames.data(), (int)frames.size(), height, width, pairs[0], pairs[1], pairs[2], theta, temporal,
       f32(a[4], "cos_out", {rows, cols}), f32(a[5], "sin_out", {rows, cols}), stream()};
  return none();
}

PyObject* rope_append_keys(Args a) {   // cfg, K_new, rope_cos, rope_sin, K_win, first, pooled_K, n_kv
  const Config c(a[0]);
  const int n = (int)length(a[1], "K_new", 2);
  const int64_t held = length(a[4], "K_win", 2);
  const int n_kv = c.kv_len(held, a[7]);
  call{lib.hf_rope_append_keys, c.get(), c.tokens(a[1], "K_new", n), n, c.table(a[2], "rope_cos", n), c.table(a[3], "rope_sin", n),
       c.tokens(a[4], "K_win", held), index(a[5]), n_kv, bytes(a[6], "pooled_K"), stream()};
  return none();
}

PyObject* rope_apply(Args a) {   // cfg, X, rope_cos, rope_sin, Y
  const Config c(a[0]);
  const int n = (int)length(a[1], "X", 2);
  call{lib.hf_rope_apply, c.get(), c.tokens(a[1], "X", n), n, c.table(a[2], "rope_cos", n), c.table(a[3], "rope_sin", n),
       c.tokens(a[4], "Y", n), stream()};
  return none();
}

PyObject* stream_open_chunk(Args a) {   // cfg, win, n_chunk, K_win, V_win, state, rope_cos_ev, rope_sin_ev, workspace
  const Config c(a[0]);
  const Struct<hf_window> win(a[1], "hf_window");
  const int cap = c->kv_capacity, n = to_int(a[2]);
  const int64_t over = (int64_t)win->n_tokens + n > cap ? (int64_t)win->n_tokens + n - cap : 0;
  int32_t first = -1, n_ev = -1;
  call{lib.hf_stream_open_chunk, c.get(), win.get(), n, c.tokens(a[3], "K_win", cap), c.tokens(a[4], "V_win", cap),
       c.state(a[5], "state"), c.table(a[6], "rope_cos_ev", over), c.table(a[7], "rope_sin_ev", over),
       bytes(a[8], "workspace"), size_of(a[8]), &first,
       &n_ev, stream()};
  return Py_BuildValue("ii", first, n_ev);
}

PyObject* stream_step(Args a) {   // cfg, win, Q, K_win, V_win, step_in_chunk, block_idx, state, O, workspace, cos, sin, Q_hist
  const Config c(a[0]);
  const Struct<hf_window> win(a[1], "hf_window");
  const int cap = c->kv_capacity, n_q = (int)length(a[2], "Q", 2), k = c.select_k(win->n_tokens);
  call{lib.hf_stream_step, c.get(), win.get(), c.tokens(a[2], "Q", n_q), c.tokens(a[12], "Q_hist", n_q), n_q,
       c.tokens(a[3], "K_win", cap), c.tokens(a[4], "V_win", cap), to_int(a[5]), i32(a[6], "block_idx", {c.B, c.H, c.t_m(n_q), k}),
       c.state(a[7], "state"), c.table(a[10], "rope_cos_q", n_q), c.table(a[11], "rope_sin_q", n_q), c.tokens(a[8], "O", n_q),
       bytes(a[9], "workspace"),
       size_of(a[9]), stream()};
  return none();
}

PyObject* ring_open_chunk(Args a) {   // cfg, ring, K_cache, V_cache, state, rope_cos_ev, rope_sin_ev, workspace
  const Config c(a[0]);
  const Struct<hf_ring> ring(a[1], "hf_ring");
  const int cap = c->kv_capacity, n = ring->n_chunk;
  int32_t first = -1, n_ev = -1;
  call{lib.hf_ring_open_chunk, c.get(), ring.get(), c.tokens(a[2], "K_cache", cap), c.tokens(a[3], "V_cache", cap),
       c.state(a[4], "state"), c.table(a[5], "rope_cos_ev", n), c.table(a[6], "rope_sin_ev", n),
       bytes(a[7], "workspace"), size_of(a[7]), &first, &n_ev,
       stream()};
  return Py_BuildValue("ii", first, n_ev);
}

PyObject* ring_step(Args a) {   // cfg, ring, Q, K_cache, V_cache, step_in_chunk, block_idx, state, O, workspace, cos, sin, Q_hist
  const Config c(a[0]);
  const Struct<hf_ring> ring(a[1], "hf_ring");
  const int cap = c->kv_capacity, n_q = ring->n_chunk, k = c.select_k(ring->n_sink + ring->n_filled * ring->n_chunk);
  call{lib.hf_ring_step, c.get(), ring.get(), c.tokens(a[2], "Q", n_q), c.tokens(a[12], "Q_hist", n_q),
       c.tokens(a[3], "K_cache", cap), c.tokens(a[4], "V_cache", cap), to_int(a[5]),
       i32(a[6], "block_idx", {c.B, c.H, c.t_m(n_q), k}), c.state(a[7], "state"), c.table(a[10], "rope_cos_q", n_q),
       c.table(a[11], "rope_sin_q", n_q), c.tokens(a[8], "O", n_q), bytes(a[9], "workspace"), size_of(a[9]), stream()};
  return none();
}

// cfg, ring, Q, K_cache, V_cache, step_in_chunk, block_idx, state, O, workspace, state_out, step_workspace, rope_cos_q,
// rope_sin_q, Q_hist, rope_cos_ev, rope_sin_ev
PyObject* ring_last_step(Args a) {
  const Config c(a[0]);
  const Struct<hf_ring> ring(a[1], "hf_ring");
  const int cap = c->kv_capacity, n_q = ring->n_chunk, k = c.select_k(ring->n_sink + ring->n_filled * ring->n_chunk);
  int32_t done = 0;
  call{lib.hf_ring_last_step, c.get(), ring.get(), c.tokens(a[2], "Q", n_q), c.tokens(a[14], "Q_hist", n_q),
       c.tokens(a[3], "K_cache", cap), c.tokens(a[4], "V_cache", cap), index(a[5]),
       i32(a[6], "block_idx", {c.B, c.H, c.t_m(n_q), k}), c.state(a[7], "state"), c.table(a[12], "rope_cos_q", n_q),
       c.table(a[13], "rope_sin_q", n_q), c.tokens(a[8], "O", n_q), bytes(a[9], "workspace"),
       size_of(a[9]), c.state(a[10], "state_out"),
       c.table(a[15], "rope_cos_ev", n_q), c.table(a[16], "rope_sin_ev", n_q), bytes(a[11], "step_workspace"),
       size_of(a[11]), &done, stream()};
  return PyBool_FromLong(done);
}

PyObject* hybrid_attn_bwd(Args a) {   // cfg, Q, K_win, V_win, block_idx, state, dO, dQ, dK, dV, workspace, cos, sin, Q_hist, dQ_hist, n_kv
  const Config c(a[0]);
  const Attn t(c, a[1], a[2], a[3], a[4], a[13], a[15]);
  call{lib.hf_hybrid_attn_bwd, c.get(), t.q, t.q_hist, t.n_q, t.kw, t.vw, t.n_kv, t.idx, t.k, c.state(a[5], "state"),
       c.table(a[11], "rope_cos_q", t.n_q), c.table(a[12], "rope_sin_q", t.n_q), c.tokens(a[6], "dO", t.n_q),
       c.tokens(a[7], "dQ", t.n_q), c.tokens(a[14], "dQ_hist", t.n_q), c.tokens(a[8], "dK", t.held), c.tokens(a[9], "dV", t.held),
       bytes(a[10], "workspace"),
       size_of(a[10]), stream()};
  return none();
}

// cfg, Q, K_win, V_win, block_idx, state, dO, O_local, lse2, dQ, dK, dV, workspace, cos, sin, Q_hist, dQ_hist, n_kv
PyObject* hybrid_attn_bwd_saved(Args a) {
  const Config c(a[0]);
  const Attn t(c, a[1], a[2], a[3], a[4], a[15], a[17]);
  call{lib.hf_hybrid_attn_bwd_saved, c.get(), t.q, t.q_hist, t.n_q, t.kw, t.vw, t.n_kv, t.idx, t.k, c.state(a[5], "state"),
       c.table(a[13], "rope_cos_q", t.n_q), c.table(a[14], "rope_sin_q", t.n_q), c.tokens(a[6], "dO", t.n_q),
       c.tokens(a[7], "O_local", t.n_q), f32(a[8], "lse2", {c.B * c.H, t.n_q}), c.tokens(a[9], "dQ", t.n_q),
       c.tokens(a[16], "dQ_hist", t.n_q), c.tokens(a[10], "dK", t.held), c.tokens(a[11], "dV", t.held),
       bytes(a[12], "workspace"), size_of(a[12]), stream()};
  return none();
}

// bind(addresses by name, HFError, hf_config, hf_window, hf_ring)
PyObject* bind(Args a) {
  if (!PyDict_Check(a[0])) raise(PyExc_TypeError, "bind takes a dict of addresses");
  auto address = [&](const char* name) -> void* {
    PyObject* v = PyDict_GetItemString(a[0], name);
    if (!v) raise(PyExc_KeyError, "no address for %s", name);
    void* p = PyLong_AsVoidPtr(v);
    if (!p) raise(PyExc_ValueError, "no address for %s", name);
    return p;
  };
  auto structure = [](PyObject* o) {   // (kept for good, like the module)
    if (!PyType_Check(o)) raise(PyExc_TypeError, "bind takes the structures' classes");
    Py_INCREF(o);
    return reinterpret_cast<PyTypeObject*>(o);
  };
#define HF_TAKE(name) lib.name = reinterpret_cast<decltype(lib.name)>(address(#name));
  HF_ENTRIES(HF_TAKE)
  Class<hf_config>::type = structure(a[2]);
  Class<hf_window>::type = structure(a[3]);
  Class<hf_ring>::type = structure(a[4]);
  Py_INCREF(a[1]);
  Py_XDECREF(error_class);
  error_class = a[1];
  return none();
}

PyObject* entry_names(Args) {
  PyObject* list = PyList_New(0);
#define HF_NAME(name)                               \
  if (list) {                                       \
    PyObject* s = PyUnicode_FromString(#name);      \
    if (s) PyList_Append(list, s);                  \
    Py_XDECREF(s);                                  \
  }
  HF_ENTRIES(HF_NAME)
  return list;
}

template <PyObject* (*F)(Args), int N> PyObject* method(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != N) return PyErr_Format(PyExc_TypeError, "%d arguments needed, got %d", N, (int)n);
  try {
    return F(args);
  } catch (Raised&) {
    return nullptr;
  } catch (std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

#define HF_METHOD(name, n) {#name, (PyCFunction)(void*)(&method<name, n>), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    HF_METHOD(bind, 5), HF_METHOD(entry_names, 0), HF_METHOD(state_init, 2), HF_METHOD(state_fold_linear, 4),
    HF_METHOD(state_planes, 3), HF_METHOD(absorb_evicted, 7), HF_METHOD(absorb_evicted_planes, 8), HF_METHOD(window_evict, 10),
    HF_METHOD(block_select, 8), HF_METHOD(block_select_static, 6), HF_METHOD(hybrid_attn_fwd, 12),
    HF_METHOD(hybrid_attn_fwd_planes, 12), HF_METHOD(hybrid_attn_fwd_save, 14), HF_METHOD(pool_keys, 5),
    HF_METHOD(select_attn_fwd, 14), HF_METHOD(step_fwd, 20), HF_METHOD(rope_window_indices, 3), HF_METHOD(rope_tables, 8),
    HF_METHOD(rope_append_keys, 8), HF_METHOD(rope_apply, 5), HF_METHOD(stream_open_chunk, 9), HF_METHOD(stream_step, 13),
    HF_METHOD(ring_open_chunk, 8), HF_METHOD(ring_step, 13), HF_METHOD(ring_last_step, 17), HF_METHOD(hybrid_attn_bwd, 16),
    HF_METHOD(hybrid_attn_bwd_saved, 18), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "argument marshalling of the hf library", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
