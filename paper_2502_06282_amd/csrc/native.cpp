// Python calls of libjakiro_verify, marshalled natively: one C function per call that a decoding loop makes, taking
// torch tensors and plain numbers positionally (binding.py gives them their names, defaults and documentation).
//
// Why it exists: most of the library's calls run for 3 - 40 us on the GPU, and a loop that issues them one by one
// is bound by its own host work.  Marshalled through ctypes (current stream 2.7 us, torch.empty 1.7 us an output, the
// call itself 3 - 4 us) an attention call of one layer cost 14 us of host time, growing and cutting a tree of depth
// six 87 us, with the GPU idle for most of it.  Here a call costs its allocations and its launches.
//
// Nothing is computed here: shapes and types are checked, outputs allocated from torch's caching allocator, and the
// C ABI is called on torch's current stream (or the given one).  Allocating and launching both may wait (for memory, for
// room in a full queue): they run without the interpreter lock, released once per call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <atomic>
#include <functional>
#include <mutex>
#include <string>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime.h>
#include <torch/csrc/autograd/python_variable.h>

#include "jk_internal.h"

namespace {

PyObject* g_error_class = nullptr;  // binding.JakiroError

// Thrown where a Python exception has been set.
struct PyFailure {};

[[noreturn]] void fail(PyObject* type, const char* what) {
  PyErr_SetString(type, what);
  throw PyFailure{};
}
[[noreturn]] void fail_status(int status, const char* where) {
  PyObject* e = g_error_class ? PyObject_CallFunction(g_error_class, "is", status, where) : nullptr;
  if (e) {
    PyErr_SetObject(g_error_class, e);
    Py_DECREF(e);
  } else if (!PyErr_Occurred()) {
    PyErr_SetString(PyExc_RuntimeError, where);
  }
  throw PyFailure{};
}
void check(int status, const char* where) {
  if (status != JK_OK) fail_status(status, where);
}

// Other Python threads run while this one allocates or launches.  (Nothing in the scope may touch a Python object; the
// tensors of the arguments are kept alive by the caller's references.)
class Unlocked {
 public:
  Unlocked() : state_(PyEval_SaveThread()) {}
  ~Unlocked() { PyEval_RestoreThread(state_); }
  Unlocked(const Unlocked&) = delete;
  Unlocked& operator=(const Unlocked&) = delete;

 private:
  PyThreadState* state_;
};
template <class F>
int unlocked(F f) {
  Unlocked u;
  return f();
}

// ------------------------------------------------------------------ arguments
struct Args {
  PyObject* const* a;
  Py_ssize_t n, at = 0;
  PyObject* next() {
    if (at >= n) fail(PyExc_TypeError, "too few arguments");
    return a[at++];
  }
  const at::Tensor& tensor() {
    PyObject* o = next();
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch tensor");
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda()) fail(PyExc_TypeError, "expected a tensor in device memory");
    return t;
  }
  const at::Tensor* optional_tensor() {
    if (at < n && a[at] == Py_None) {
      ++at;
      return nullptr;
    }
    return &tensor();
  }
  long long integer() {
    PyObject* o = next();
    PyObject* as_int = PyNumber_Index(o);
    if (!as_int) {  // what int() takes
      PyErr_Clear();
      as_int = PyNumber_Long(o);
    }
    if (!as_int) throw PyFailure{};
    const long long v = PyLong_AsLongLong(as_int);
    Py_DECREF(as_int);
    if (v == -1 && PyErr_Occurred()) throw PyFailure{};
    return v;
  }
  int32_t i32() {
    const long long v = integer();
    if (v < INT32_MIN || v > INT32_MAX) fail(PyExc_OverflowError, "value does not fit 32 bits");
    return (int32_t)v;
  }
  float real() {
    const double v = PyFloat_AsDouble(next());
    if (v == -1.0 && PyErr_Occurred()) throw PyFailure{};
    return (float)v;
  }
  bool truth() {
    const int v = PyObject_IsTrue(next());
    if (v < 0) throw PyFailure{};
    return v != 0;
  }
};

void* ptr(const at::Tensor& t) { return t.data_ptr(); }
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
size_t bytes_of(const at::Tensor& t) { return t.nbytes(); }
bool is_i32(const at::Tensor& t) { return t.scalar_type() == at::kInt && t.is_contiguous(); }
bool is_f32(const at::Tensor& t) { return t.scalar_type() == at::kFloat && t.is_contiguous(); }
bool is_bf16(const at::Tensor& t) { return t.scalar_type() == at::kBFloat16 && t.is_contiguous(); }
void dims(const at::Tensor& t, int n, const char* what) {
  if (t.dim() != n) fail(PyExc_ValueError, what);
}

at::Tensor empty(at::IntArrayRef size, at::ScalarType type, const at::Tensor& like) {
  return at::Tensor(at::detail::empty_cuda(size, type, like.device(), std::nullopt));
}
PyObject* wrap(at::Tensor t) {
  PyObject* o = THPVariable_Wrap(std::move(t));
  if (!o) throw PyFailure{};
  return o;
}
template <class... T>
PyObject* pack(T... t) {  // a tuple of new references
  PyObject* r = PyTuple_New(sizeof...(t));
  if (!r) throw PyFailure{};
  Py_ssize_t i = 0;
  (PyTuple_SET_ITEM(r, i++, t), ...);
  return r;
}
PyObject* none() {
  Py_INCREF(Py_None);
  return Py_None;
}

// The hipStream_t to launch on: torch's current stream, or the given torch.cuda.Stream.  The first use on a device
// also runs jk_init there (a short synchronous probe), unless that stream is being captured into a graph.
void* stream_handle(PyObject* stream) {
  static std::atomic<bool> initialised[64];
  void* handle = nullptr;
  if (stream == nullptr || stream == Py_None) {
    handle = c10::hip::getCurrentHIPStream().stream();
  } else {
    PyObject* h = PyObject_GetAttrString(stream, "cuda_stream");
    if (!h) throw PyFailure{};
    handle = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (PyErr_Occurred()) throw PyFailure{};
  }
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) fail_status(JK_ERR_HIP, "hipGetDevice");
  if (dev >= 0 && dev < 64 && !initialised[dev]) {  // (two threads at once: both probe, with the same result)
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    void* current = c10::hip::getCurrentHIPStream().stream();
    if (hipStreamIsCapturing(static_cast<hipStream_t>(current), &st) != hipSuccess)
      fail_status(JK_ERR_HIP, "hipStreamIsCapturing");
    if (st == hipStreamCaptureStatusNone) {
      check(unlocked([&] { return jk_init(handle); }), "jk_init");
      initialised[dev] = true;
    }
  }
  return handle;
}

// ------------------------------------------------------------------ a call marshalled once
// launch() issues exactly that one library call: what a decoding loop, or a HIP-graph capture of it, calls per step.
struct PreparedCall {
  PyObject_HEAD
  std::function<int(void*)>* call;
  const char* where;
  PyObject* keep;  // references to every tensor the call points to
};

void prepared_dealloc(PyObject* o) {
  PreparedCall* p = reinterpret_cast<PreparedCall*>(o);
  delete p->call;
  Py_XDECREF(p->keep);
  Py_TYPE(o)->tp_free(o);
}
PyObject* prepared_launch(PyObject* o, PyObject* const* a, Py_ssize_t n, PyObject* names) {
  PyObject* stream = nullptr;
  const Py_ssize_t named = names ? PyTuple_GET_SIZE(names) : 0;
  if (n + named > 1 || (named && PyUnicode_CompareWithASCIIString(PyTuple_GET_ITEM(names, 0), "stream") != 0)) {
    PyErr_SetString(PyExc_TypeError, "launch(stream=None)");
    return nullptr;
  }
  if (n + named == 1) stream = a[0];
  PreparedCall* p = reinterpret_cast<PreparedCall*>(o);
  try {
    void* on = stream_handle(stream);
    check(unlocked([&] { return (*p->call)(on); }), p->where);
  } catch (const PyFailure&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
  Py_RETURN_NONE;
}
PyMethodDef prepared_methods[] = {
    {"launch", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(prepared_launch)),
     METH_FASTCALL | METH_KEYWORDS,
     "launch(stream=None): issue the call on `stream` (default: torch's current stream)"},
    {nullptr, nullptr, 0, nullptr}};
PyTypeObject prepared_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* prepared(std::function<int(void*)> call, const char* where, const Args& args) {
  PreparedCall* p = PyObject_New(PreparedCall, &prepared_type);
  if (!p) throw PyFailure{};
  p->call = new std::function<int(void*)>(std::move(call));
  p->where = where;
  p->keep = PyTuple_New(args.n);
  if (!p->keep) {
    Py_DECREF(p);
    throw PyFailure{};
  }
  for (Py_ssize_t i = 0; i < args.n; ++i) {
    Py_INCREF(args.a[i]);
    PyTuple_SET_ITEM(p->keep, i, args.a[i]);
  }
  return reinterpret_cast<PyObject*>(p);
}

// ------------------------------------------------------------------ attention
struct Attention {
  jk_attn_desc d;
  jk_paged_kv pages;
  bool paged;
  const void *q, *k, *v, *kt, *vt;
  const int32_t *parent, *plen;
  int32_t max_prefix;
  void *out, *ws;
  size_t ws_bytes;
  int operator()(void* stream) const {
    return paged ? jk_tree_verify_attention_paged(&d, &pages, q, k, v, kt, vt, parent, plen, max_prefix, out, ws, ws_bytes, stream)
                 : jk_tree_verify_attention(&d, q, k, v, kt, vt, parent, plen, max_prefix, out, ws, ws_bytes, stream);
  }
  const char* where() const { return paged ? "jk_tree_verify_attention_paged" : "jk_tree_verify_attention"; }
};

void head_dim_innermost(const at::Tensor& t) {
  if (t.dim() > 0 && t.size(-1) > 1 && t.stride(-1) != 1)
    fail(PyExc_ValueError, "head_dim must be the contiguous innermost axis");
}

// (q, k, v, table or None, k_tree, v_tree, parent, prefix_len, max_prefix_len or None, scale, out or None, workspace)
Attention read_attention(Args& a, at::Tensor* new_out) {
  Attention c{};
  const at::Tensor& q = a.tensor();
  const at::Tensor* k = a.optional_tensor();
  const at::Tensor* v = a.optional_tensor();
  const at::Tensor* table = a.optional_tensor();
  const at::Tensor &kt = a.tensor(), &vt = a.tensor(), &parent = a.tensor(), &plen = a.tensor();
  c.paged = table != nullptr;
  if (!c.paged && k && k->size(1) == 0) k = v = nullptr;  // an empty cache has no meaningful strides
  if (a.at < a.n && a.a[a.at] == Py_None) {
    ++a.at;
    c.max_prefix = k ? (int32_t)k->size(1) : 0;
  } else {
    c.max_prefix = a.i32();
  }
  const float scale = a.real();
  const at::Tensor* out = a.optional_tensor();
  const at::Tensor& ws = a.tensor();
  if (k) {
    if (!v) fail(PyExc_ValueError, "k_cache without v_cache");
    if (k->strides() != v->strides() || k->sizes() != v->sizes())
      fail(PyExc_ValueError, c.paged ? "K and V pools must share strides" : "k_cache and v_cache must share shape and strides");
  }
  if (kt.strides() != vt.strides() || kt.sizes() != vt.sizes())
    fail(PyExc_ValueError, "k_tree and v_tree must share shape and strides");
  if (parent.scalar_type() != at::kInt || plen.scalar_type() != at::kInt)
    fail(PyExc_TypeError, "parent and prefix_len must be int32");
  if (!parent.is_contiguous() || !plen.is_contiguous())
    fail(PyExc_ValueError, "parent and prefix_len must be contiguous");
  dims(q, 4, "q must be [B, T, Hq, D]");
  dims(kt, 4, "k_tree must be [B, T, Hkv, D]");
  if (!out) {
    if (!new_out) fail(PyExc_TypeError, "out is required");
    Unlocked u;
    *new_out = empty(q.sizes(), q.scalar_type(), q);
    out = new_out;
  }
  dims(*out, 4, "out must be [B, T, Hq, D]");
  jk_attn_desc& d = c.d;
  d.dtype = q.scalar_type() == at::kBFloat16 ? JK_BF16 : JK_F32;
  if (d.dtype == JK_F32 && q.scalar_type() != at::kFloat) fail(PyExc_TypeError, "q must be bfloat16 or float32");
  head_dim_innermost(q);
  if (k) head_dim_innermost(*k);
  head_dim_innermost(kt);
  head_dim_innermost(*out);
  d.batch = (int32_t)q.size(0); d.n_tree = (int32_t)q.size(1); d.n_q_heads = (int32_t)q.size(2);
  d.n_kv_heads = (int32_t)kt.size(2); d.head_dim = (int32_t)q.size(3);
  d.q_stride_b = q.stride(0); d.q_stride_t = q.stride(1); d.q_stride_h = q.stride(2);
  if (k) {
    dims(*k, 4, "caches and pools have four axes");
    d.kc_stride_b = c.paged ? 0 : k->stride(0);
    d.kc_stride_l = k->stride(1); d.kc_stride_h = k->stride(2);
  }
  d.kt_stride_b = kt.stride(0); d.kt_stride_t = kt.stride(1); d.kt_stride_h = kt.stride(2);
  d.o_stride_b = out->stride(0); d.o_stride_t = out->stride(1); d.o_stride_h = out->stride(2);
  d.scale = scale;
  if (c.paged) {
    if (!k) fail(PyExc_TypeError, "a paged call needs its pools");
    dims(*table, 2, "block_table must be [B, max_blocks]");
    c.pages.block_table = static_cast<const int32_t*>(ptr(table));
    c.pages.max_blocks = (int32_t)table->size(1);
    c.pages.page_size = (int32_t)k->size(1);
    c.pages.n_pages = (int32_t)k->size(0);
    c.pages.page_stride = k->stride(0);
  }
  c.q = ptr(q); c.k = ptr(k); c.v = ptr(v); c.kt = ptr(kt); c.vt = ptr(vt);
  c.parent = static_cast<const int32_t*>(ptr(parent)); c.plen = static_cast<const int32_t*>(ptr(plen));
  c.out = ptr(out); c.ws = ptr(ws); c.ws_bytes = bytes_of(ws);
  return c;
}
PyObject* attention(Args& a) {
  at::Tensor made;
  const Attention c = read_attention(a, &made);
  void* stream = stream_handle(a.next());
  const int st = unlocked([&] { return c(stream); });
  if (st != JK_OK) {
    if (jk_tree_verify_attention_workspace(&c.d, c.max_prefix) == 0) fail_status(JK_ERR_UNSUPPORTED, "jk_tree_verify_attention_workspace");
    fail_status(st, c.where());
  }
  if (made.defined()) return wrap(std::move(made));
  PyObject* out = a.a[10];
  Py_INCREF(out);
  return out;
}
PyObject* prepare_attention(Args& a) {
  const Attention c = read_attention(a, nullptr);
  return prepared(c, c.where(), a);
}

// ------------------------------------------------------------------ acceptance
struct Accept {
  int32_t b, n, v, depth, mode;
  float temperature;
  const int32_t *tokens, *parent, *draft_row;
  const float *logits, *draft, *uniforms;
  int64_t draft_rows;
  int32_t *path, *len, *bonus;
  void* ws;
  size_t ws_bytes;
  int operator()(void* stream) const {
    return draft_row ? jk_accept_path_rows(b, n, v, depth, tokens, parent, logits, mode, temperature, draft, draft_rows, draft_row,
                                           uniforms, path, len, bonus, ws, ws_bytes, stream)
                     : jk_accept_path(b, n, v, depth, tokens, parent, logits, mode, temperature, draft, uniforms, path, len, bonus,
                                      ws, ws_bytes, stream);
  }
  const char* where() const { return draft_row ? "jk_accept_path_rows" : "jk_accept_path"; }
};

// (tokens, parent, logits, mode, temperature, draft or None, draft_row or None, uniforms or None)
Accept read_accept(Args& a, const at::Tensor** tokens_out) {
  Accept c{};
  const at::Tensor &tokens = a.tensor(), &parent = a.tensor(), &logits = a.tensor();
  c.mode = a.i32();
  c.temperature = a.real();
  const at::Tensor* draft = a.optional_tensor();
  const at::Tensor* row = a.optional_tensor();
  const at::Tensor* uniforms = a.optional_tensor();
  dims(tokens, 2, "tree_tokens must be [B, N]");
  if (!is_i32(tokens) || !is_i32(parent) || (row && !is_i32(*row)))
    fail(PyExc_TypeError, row ? "tree_tokens, parent and q_row must be contiguous int32" : "tree_tokens and parent must be contiguous int32");
  if (!is_f32(logits) || (draft && !is_f32(*draft)) || (uniforms && !is_f32(*uniforms)))
    fail(PyExc_TypeError, "logits, draft_probs and uniforms must be contiguous float32");
  c.b = (int32_t)tokens.size(0); c.n = (int32_t)tokens.size(1); c.v = (int32_t)logits.size(-1);
  if (logits.dim() != 3 || logits.size(0) != c.b || logits.size(1) != c.n + 1)
    fail(PyExc_ValueError, "target_logits must be [B, N+1, V]");
  if (row) {
    if (!draft || draft->size(-1) != c.v || row->dim() != 2 || row->size(0) != c.b || row->size(1) != c.n)
      fail(PyExc_ValueError, "q_all [n_rows, V], q_row [B, N]");
    c.draft_rows = draft->numel() / c.v;
  }
  c.tokens = static_cast<const int32_t*>(ptr(tokens)); c.parent = static_cast<const int32_t*>(ptr(parent));
  c.logits = static_cast<const float*>(ptr(logits)); c.draft = static_cast<const float*>(ptr(draft));
  c.draft_row = static_cast<const int32_t*>(ptr(row)); c.uniforms = static_cast<const float*>(ptr(uniforms));
  *tokens_out = &tokens;
  return c;
}
// ... , max_depth or None, workspace, stream
PyObject* accept(Args& a) {
  const at::Tensor* tokens;
  Accept c = read_accept(a, &tokens);
  if (a.at < a.n && a.a[a.at] == Py_None) {
    ++a.at;
    c.depth = c.n;
  } else {
    c.depth = a.i32();
  }
  const at::Tensor& ws = a.tensor();
  c.ws = ptr(ws); c.ws_bytes = bytes_of(ws);
  void* stream = stream_handle(a.next());
  at::Tensor path, len, bonus;
  const int st = unlocked([&] {
    path = empty({c.b, c.depth}, at::kInt, *tokens); len = empty({c.b}, at::kInt, *tokens); bonus = empty({c.b}, at::kInt, *tokens);
    c.path = static_cast<int32_t*>(ptr(path)); c.len = static_cast<int32_t*>(ptr(len)); c.bonus = static_cast<int32_t*>(ptr(bonus));
    return c(stream);
  });
  if (st != JK_OK) {
    if (jk_accept_path_workspace(c.b, c.n, c.v, c.mode) == 0) fail_status(JK_ERR_UNSUPPORTED, "jk_accept_path_workspace");
    fail_status(st, c.where());
  }
  return pack(wrap(std::move(path)), wrap(std::move(len)), wrap(std::move(bonus)));
}
// ... , out_path, out_accept_len, out_bonus_token, workspace
PyObject* prepare_accept(Args& a) {
  const at::Tensor* tokens;
  Accept c = read_accept(a, &tokens);
  const at::Tensor &path = a.tensor(), &len = a.tensor(), &bonus = a.tensor(), &ws = a.tensor();
  c.depth = (int32_t)path.size(1);
  c.path = static_cast<int32_t*>(ptr(path)); c.len = static_cast<int32_t*>(ptr(len)); c.bonus = static_cast<int32_t*>(ptr(bonus));
  c.ws = ptr(ws); c.ws_bytes = bytes_of(ws);
  return prepared(c, c.where(), a);
}

// ------------------------------------------------------------------ commit
// One layer, or all layers of a model (the four pointers are then device tables), contiguous or paged caches.
struct Commit {
  jk_attn_desc d;
  jk_paged_kv pages;
  bool paged;
  int32_t layers;
  void *kt, *vt, *kc, *vc;
  const int32_t *path, *len;
  int32_t depth, capacity, advance;
  int32_t* plen;
  int operator()(void* stream) const {
    if (layers == 0) return jk_commit_path(&d, kt, vt, kc, vc, path, len, depth, capacity, plen, advance, stream);
    auto in = [](void* p) { return static_cast<const void* const*>(p); };
    auto io = [](void* p) { return static_cast<void* const*>(p); };
    if (paged)
      return jk_commit_path_layers_paged(&d, &pages, layers, in(kt), in(vt), io(kc), io(vc), path, len, depth, plen, advance, stream);
    return jk_commit_path_layers(&d, layers, in(kt), in(vt), io(kc), io(vc), path, len, depth, capacity, plen, advance, stream);
  }
  const char* where() const {
    return layers == 0 ? "jk_commit_path" : paged ? "jk_commit_path_layers_paged" : "jk_commit_path_layers";
  }
};
// (k_tree, v_tree, k_cache, v_cache, block_table or None, path, accept_len, prefix_len, advance, n_layers, then, with
// n_layers > 0, the four device tables of layer pointers)
Commit read_commit(Args& a) {
  Commit c{};
  const at::Tensor &kt = a.tensor(), &vt = a.tensor(), &kc = a.tensor(), &vc = a.tensor();
  const at::Tensor* table = a.optional_tensor();
  const at::Tensor &path = a.tensor(), &len = a.tensor(), &plen = a.tensor();
  c.advance = a.truth() ? 1 : 0;
  c.layers = a.i32();
  dims(kt, 4, "k_tree must be [B, T, Hkv, D]");
  dims(kc, 4, "caches and pools have four axes");
  dims(path, 2, "path must be [B, max_depth]");
  c.d.dtype = kt.scalar_type() == at::kBFloat16 ? JK_BF16 : JK_F32;
  if (c.d.dtype == JK_F32 && kt.scalar_type() != at::kFloat) fail(PyExc_TypeError, "k_tree must be bfloat16 or float32");
  if (vt.strides() != kt.strides() || vc.strides() != kc.strides()) fail(PyExc_ValueError, "K and V must share strides");
  head_dim_innermost(kt);
  head_dim_innermost(kc);
  c.paged = table != nullptr;
  jk_attn_desc& d = c.d;
  d.batch = (int32_t)kt.size(0); d.n_tree = (int32_t)kt.size(1); d.n_q_heads = d.n_kv_heads = (int32_t)kt.size(2);
  d.head_dim = (int32_t)kt.size(3);
  d.kc_stride_b = c.paged ? 0 : kc.stride(0); d.kc_stride_l = kc.stride(1); d.kc_stride_h = kc.stride(2);
  d.kt_stride_b = kt.stride(0); d.kt_stride_t = kt.stride(1); d.kt_stride_h = kt.stride(2);
  if (c.paged) {
    dims(*table, 2, "block_table must be [B, max_blocks]");
    c.pages = {static_cast<const int32_t*>(ptr(table)), (int32_t)table->size(1), (int32_t)kc.size(1), (int32_t)kc.size(0), kc.stride(0)};
  }
  c.kt = ptr(kt); c.vt = ptr(vt); c.kc = ptr(kc); c.vc = ptr(vc);
  c.path = static_cast<const int32_t*>(ptr(path)); c.len = static_cast<const int32_t*>(ptr(len));
  c.plen = static_cast<int32_t*>(ptr(plen));
  c.depth = (int32_t)path.size(1); c.capacity = (int32_t)kc.size(1);
  if (c.layers > 0) {
    c.kt = ptr(a.tensor()); c.vt = ptr(a.tensor()); c.kc = ptr(a.tensor()); c.vc = ptr(a.tensor());
  }
  return c;
}
PyObject* commit(Args& a) {  // ... , stream
  const Commit c = read_commit(a);
  void* stream = stream_handle(a.next());
  check(unlocked([&] { return c(stream); }), c.where());
  return none();
}
PyObject* prepare_commit(Args& a) {  // ... (and whatever else is to be kept alive)
  const Commit c = read_commit(a);
  return prepared(c, c.where(), a);
}

// ------------------------------------------------------------------ draft heads
struct Heads {
  jk_draft_heads_desc d;
  const void *f, *w;
  const float* s;
  float *logits, *probs, *topp;
  int32_t* topk;
  void* ws;
  size_t ws_bytes;
  int operator()(void* stream) const { return jk_draft_heads(&d, f, s, w, logits, probs, topk, topp, ws, ws_bytes, stream); }
};
// (f_top, s_top, w_head, mode, temperature, top_k, alpha, beta)
Heads read_heads(Args& a, const at::Tensor** f_out) {
  Heads c{};
  const at::Tensor &f = a.tensor(), &s = a.tensor(), &w = a.tensor();
  dims(f, 3, "f_top must be [R, 2, d]");
  dims(w, 2, "w_head must be [V, d]");
  if (f.size(1) != 2 || s.dim() != 2 || s.size(0) != f.size(0) || s.size(1) != 2 || w.size(1) != f.size(2))
    fail(PyExc_ValueError, "f_top [R,2,d], s_top [R,2], w_head [V,d]");
  if (!is_bf16(f) || !is_bf16(w)) fail(PyExc_TypeError, "f_top and w_head must be contiguous bfloat16");
  if (!is_f32(s)) fail(PyExc_TypeError, "s_top, logits, draft_probs and topk_probs must be contiguous float32");
  c.d.rows = (int32_t)f.size(0); c.d.d_model = (int32_t)f.size(2); c.d.vocab = (int32_t)w.size(0);
  c.d.mode = a.i32(); c.d.temperature = a.real(); c.d.top_k = a.i32(); c.d.alpha = a.real(); c.d.beta = a.real();
  c.f = ptr(f); c.s = static_cast<const float*>(ptr(s)); c.w = ptr(w);
  *f_out = &f;
  return c;
}
// ... , want_probs, out_probs or None, stream -> (logits, probs or None, topk_tokens, topk_probs)
PyObject* heads(Args& a) {
  const at::Tensor* f;
  Heads c = read_heads(a, &f);
  const bool want = a.truth();
  const at::Tensor* given = a.optional_tensor();
  const int64_t R = c.d.rows, V = c.d.vocab, K = c.d.top_k;
  if (given && (given->dim() != 3 || given->size(0) != R || given->size(1) != 2 || given->size(2) != V))
    fail(PyExc_ValueError, "out_probs must be [R, 2, V]");
  if (given && !is_f32(*given)) fail(PyExc_TypeError, "s_top, logits, draft_probs and topk_probs must be contiguous float32");
  if (K < 0) fail(PyExc_RuntimeError, "top_k must not be negative");
  const size_t need = jk::draft_heads_call_bytes(c.d.rows, c.d.d_model, c.d.vocab);
  if (need == 0) fail_status(JK_ERR_UNSUPPORTED, "jk_draft_heads_workspace");
  void* stream = stream_handle(a.next());
  at::Tensor logits, probs, tk, tp, ws;
  check(unlocked([&] {
          logits = empty({R, 2, V}, at::kFloat, *f);
          if (!given && want) probs = empty({R, 2, V}, at::kFloat, *f);
          tk = empty({R, 2, K}, at::kInt, *f); tp = empty({R, 2, K}, at::kFloat, *f); ws = empty({(int64_t)need}, at::kByte, *f);
          c.logits = static_cast<float*>(ptr(logits));
          c.probs = static_cast<float*>(given ? ptr(given) : probs.defined() ? ptr(probs) : nullptr);
          c.topk = static_cast<int32_t*>(ptr(tk)); c.topp = static_cast<float*>(ptr(tp));
          c.ws = ptr(ws); c.ws_bytes = need;
          return c(stream);
        }),
        "jk_draft_heads");
  PyObject* p;
  if (given) {
    p = a.a[9];
    Py_INCREF(p);
  } else {
    p = probs.defined() ? wrap(std::move(probs)) : none();
  }
  return pack(wrap(std::move(logits)), p, wrap(std::move(tk)), wrap(std::move(tp)));
}
// ... , logits, draft_probs or None, topk_tokens, topk_probs, workspace
PyObject* prepare_heads(Args& a) {
  const at::Tensor* f;
  Heads c = read_heads(a, &f);
  const at::Tensor& logits = a.tensor();
  const at::Tensor* probs = a.optional_tensor();
  const at::Tensor &tk = a.tensor(), &tp = a.tensor(), &ws = a.tensor();
  if (!is_f32(logits) || (probs && !is_f32(*probs)) || !is_f32(tp))
    fail(PyExc_TypeError, "s_top, logits, draft_probs and topk_probs must be contiguous float32");
  if (!is_i32(tk)) fail(PyExc_TypeError, "topk_tokens must be contiguous int32");
  c.logits = static_cast<float*>(ptr(logits)); c.probs = static_cast<float*>(ptr(probs));
  c.topk = static_cast<int32_t*>(ptr(tk)); c.topp = static_cast<float*>(ptr(tp));
  c.ws = ptr(ws); c.ws_bytes = bytes_of(ws);
  return prepared(c, "jk_draft_heads", a);
}

// ------------------------------------------------------------------ router and experts
struct Moe {
  jk_moe_desc d;
  const void *u, *cen, *gate, *up, *down;
  void *f_top, *f_mix, *ws;
  float* s_top;
  int32_t* idx;
  size_t ws_bytes;
  int operator()(void* stream) const { return jk_moe_experts(&d, u, cen, gate, up, down, f_top, s_top, idx, f_mix, ws, ws_bytes, stream); }
};
// (u, centroids, w_gate, w_up, w_down)
Moe read_moe(Args& a, const at::Tensor** u_out) {
  Moe c{};
  const at::Tensor &u = a.tensor(), &cen = a.tensor(), &gate = a.tensor(), &up = a.tensor(), &down = a.tensor();
  dims(u, 2, "u must be [R, d]");
  dims(gate, 3, "w_gate must be [N, F, d]");
  const int64_t d = u.size(1), n = gate.size(0), f = gate.size(1);
  if (gate.size(2) != d || cen.dim() != 2 || cen.size(0) != n || cen.size(1) != d || up.sizes() != gate.sizes() || down.dim() != 3 ||
      down.size(0) != n || down.size(1) != d || down.size(2) != f)
    fail(PyExc_ValueError, "u [R,d], centroids [N,d], w_gate/w_up [N,F,d], w_down [N,d,F]");
  for (const at::Tensor* t : {&u, &cen, &gate, &up, &down})
    if (!is_bf16(*t)) fail(PyExc_TypeError, "features and weights must be contiguous bfloat16");
  c.d.rows = (int32_t)u.size(0); c.d.d_model = (int32_t)d; c.d.d_ff = (int32_t)f; c.d.n_experts = (int32_t)n;
  c.u = ptr(u); c.cen = ptr(cen); c.gate = ptr(gate); c.up = ptr(up); c.down = ptr(down);
  *u_out = &u;
  return c;
}
// ... , want_mix, stream -> (f_top, s_top, expert_idx, f_mix or None)
PyObject* moe(Args& a) {
  const at::Tensor* u;
  Moe c = read_moe(a, &u);
  const bool want = a.truth();
  const int64_t R = c.d.rows, d = c.d.d_model;
  const size_t need = jk::moe_experts_call_bytes(c.d);
  if (need == 0) fail_status(JK_ERR_UNSUPPORTED, "jk_moe_experts_workspace");
  void* stream = stream_handle(a.next());
  at::Tensor f, s, idx, mix, ws;
  check(unlocked([&] {
          f = empty({R, 2, d}, at::kBFloat16, *u); s = empty({R, 2}, at::kFloat, *u); idx = empty({R, 2}, at::kInt, *u);
          if (want) mix = empty({R, d}, at::kBFloat16, *u);
          ws = empty({(int64_t)need}, at::kByte, *u);
          c.f_top = ptr(f); c.s_top = static_cast<float*>(ptr(s)); c.idx = static_cast<int32_t*>(ptr(idx));
          c.f_mix = want ? ptr(mix) : nullptr; c.ws = ptr(ws); c.ws_bytes = need;
          return c(stream);
        }),
        "jk_moe_experts");
  return pack(wrap(std::move(f)), wrap(std::move(s)), wrap(std::move(idx)), want ? wrap(std::move(mix)) : none());
}
// ... , f_top, s_top, expert_idx, f_mix or None, workspace
PyObject* prepare_moe(Args& a) {
  const at::Tensor* u;
  Moe c = read_moe(a, &u);
  const at::Tensor &f = a.tensor(), &s = a.tensor(), &idx = a.tensor();
  const at::Tensor* mix = a.optional_tensor();
  const at::Tensor& ws = a.tensor();
  if (!is_bf16(f) || (mix && !is_bf16(*mix))) fail(PyExc_TypeError, "features and weights must be contiguous bfloat16");
  if (s.scalar_type() != at::kFloat || idx.scalar_type() != at::kInt) fail(PyExc_TypeError, "s_top float32, expert_idx int32");
  c.f_top = ptr(f); c.s_top = static_cast<float*>(ptr(s)); c.idx = static_cast<int32_t*>(ptr(idx)); c.f_mix = ptr(mix);
  c.ws = ptr(ws); c.ws_bytes = bytes_of(ws);
  return prepared(c, "jk_moe_experts", a);
}

// ------------------------------------------------------------------ linear
// (x, w, residual or None, fp32 result, stream)
PyObject* linear(Args& a) {
  const at::Tensor &x = a.tensor(), &w = a.tensor();
  const at::Tensor* res = a.optional_tensor();
  const bool f32 = a.truth();
  dims(x, 2, "x must be [m, k]");
  dims(w, 2, "w must be [n, k]");
  if (!is_bf16(x) || !is_bf16(w) || (res && !is_bf16(*res))) fail(PyExc_TypeError, "x, w and residual must be contiguous bfloat16");
  const int64_t m = x.size(0), k = x.size(1), n = w.size(0);
  if (w.size(1) != k || (res && (res->dim() != 2 || res->size(0) != m || res->size(1) != n)))
    fail(PyExc_ValueError, "x [m,k], w [n,k], residual [m,n]");
  const size_t need = jk::linear_call_bytes((int)m, (int)n, (int)k);
  if (need == 0) fail_status(JK_ERR_UNSUPPORTED, "jk_linear_workspace");
  void* stream = stream_handle(a.next());
  at::Tensor out, ws;
  check(unlocked([&] {
          out = empty({m, n}, f32 ? at::kFloat : at::kBFloat16, x);
          // (most products write nothing to a workspace: no allocation for one)
          const bool used = jk::linear_call_writes((int)m, (int)n, (int)k);
          if (used) ws = empty({(int64_t)need}, at::kByte, x);
          return jk::linear_call((int32_t)m, (int32_t)n, (int32_t)k, ptr(x), ptr(w), ptr(res), f32 ? nullptr : ptr(out),
                                 f32 ? static_cast<float*>(ptr(out)) : nullptr, used ? ptr(ws) : nullptr, stream);
        }),
        "jk_linear");
  return wrap(std::move(out));
}

// ------------------------------------------------------------------ draft tree
struct TreeState {
  jk_tree_state s;
  int32_t batch;
};
TreeState read_tree_state(Args& a) {  // (tokens, parent, score, q_row, n_nodes)
  const at::Tensor &tok = a.tensor(), &par = a.tensor(), &sc = a.tensor(), &qr = a.tensor(), &n = a.tensor();
  dims(tok, 2, "tree state arrays must be [batch, max_nodes]");
  TreeState t;
  t.s = {static_cast<int32_t*>(ptr(tok)), static_cast<int32_t*>(ptr(par)), static_cast<float*>(ptr(sc)),
         static_cast<int32_t*>(ptr(qr)), static_cast<int32_t*>(ptr(n)), (int32_t)tok.size(1)};
  t.batch = (int32_t)tok.size(0);
  return t;
}
struct Candidates {
  const at::Tensor *front, *tok, *p;
  int32_t n_front, k;
};
Candidates read_candidates(Args& a, int32_t batch) {  // (frontier_in or None, cand_tokens, cand_probs)
  Candidates c;
  c.front = a.optional_tensor();
  c.tok = &a.tensor();
  c.p = &a.tensor();
  if (c.front) dims(*c.front, 2, "frontier_in must be [B, n_front]");
  c.n_front = c.front ? (int32_t)c.front->size(1) : 1;
  dims(*c.tok, 3, "cand_tokens / cand_probs must be [B*n_front, 2, k]");
  if (c.tok->size(0) != (int64_t)batch * c.n_front || c.tok->size(1) != 2 || c.p->sizes() != c.tok->sizes())
    fail(PyExc_ValueError, "cand_tokens / cand_probs must be [B*n_front, 2, k]");
  if (!is_i32(*c.tok) || !is_f32(*c.p)) fail(PyExc_TypeError, "cand_tokens contiguous int32, cand_probs contiguous float32");
  if (c.front && !is_i32(*c.front)) fail(PyExc_TypeError, "frontier_in contiguous int32");
  c.k = (int32_t)c.tok->size(2);
  return c;
}
const int32_t* ints(const at::Tensor* t) { return static_cast<const int32_t*>(ptr(t)); }

PyObject* tree_grow(Args& a) {  // state, candidates, width, q_row_base, stream -> frontier
  const TreeState t = read_tree_state(a);
  const Candidates c = read_candidates(a, t.batch);
  const int32_t width = a.i32(), base = a.i32();
  void* stream = stream_handle(a.next());
  at::Tensor out;
  check(unlocked([&] {
          out = empty({t.batch, width > 0 ? width : 0}, at::kInt, *c.tok);
          return jk_tree_grow(&t.s, t.batch, c.n_front, c.k, width, base, ints(c.front), ints(c.tok), static_cast<const float*>(ptr(c.p)),
                              static_cast<int32_t*>(ptr(out)), stream);
        }),
        "jk_tree_grow");
  return wrap(std::move(out));
}
PyObject* tree_grow_tail(Args& a) {  // state, candidates, k1, k2, width, q_row_base, stream
  const TreeState t = read_tree_state(a);
  const Candidates c = read_candidates(a, t.batch);
  const int32_t k1 = a.i32(), k2 = a.i32(), width = a.i32(), base = a.i32();
  void* stream = stream_handle(a.next());
  check(unlocked([&] {
          return jk_tree_grow_tail(&t.s, t.batch, c.n_front, c.k, k1, k2, width, base, ints(c.front), ints(c.tok),
                                   static_cast<const float*>(ptr(c.p)), stream);
        }),
        "jk_tree_grow_tail");
  return none();
}
PyObject* tree_fill_static(Args& a) {  // state, candidates, slot, expert, rank, next or None, q_row_base, stream -> (frontier or None, ids)
  const TreeState t = read_tree_state(a);
  const Candidates c = read_candidates(a, t.batch);
  const at::Tensor &slot = a.tensor(), &expert = a.tensor(), &rank = a.tensor();
  const at::Tensor* next = a.optional_tensor();
  const int32_t base = a.i32(), n_new = (int32_t)slot.numel(), n_next = next ? (int32_t)next->numel() : 0;
  void* stream = stream_handle(a.next());
  at::Tensor ids, out;
  check(unlocked([&] {
          ids = empty({t.batch, n_new}, at::kInt, *c.tok);
          if (n_next) out = empty({t.batch, n_next}, at::kInt, *c.tok);
          return jk_tree_fill_static(&t.s, t.batch, c.n_front, c.k, base, ints(c.front), ints(c.tok), static_cast<const float*>(ptr(c.p)),
                                     ints(&slot), ints(&expert), ints(&rank), n_new, ints(next), n_next,
                                     n_next ? static_cast<int32_t*>(ptr(out)) : nullptr, static_cast<int32_t*>(ptr(ids)), stream);
        }),
        "jk_tree_fill_static");
  return pack(n_next ? wrap(std::move(out)) : none(), wrap(std::move(ids)));
}
// Whether an operation on t would run its device kernel and nothing else: a tensor with the dispatch keys of an ordinary one, and nobody who
// intercepts, records, transforms or traces what this thread does (function and dispatch modes, transforms and tracing have keys of their
// own in the thread's set; inference mode takes one away).
bool ordinary(const at::Tensor& t) {
  constexpr auto backend = c10::BackendComponent::CUDABit;
  static const c10::DispatchKeySet plain = c10::DispatchKeySet(c10::DispatchKey::CUDA) | c10::getAutocastRelatedKeySetFromBackend(backend) |
                                           c10::getAutogradRelatedKeySetFromBackend(backend);
  return t.key_set() == plain && c10::impl::tls_local_dispatch_key_set().included_.add(c10::DispatchKey::ADInplaceOrView) == c10::default_included_set &&
         !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::hasCallbacks();
}
// n_nodes -> whether it was cleared here, as zero_ would have.  (zero_ takes 3.6 us of a thread, TreeState.reset with this 2.8.)
PyObject* tree_reset(Args& a) {
  PyObject* o = a.next();
  bool plain = THPVariable_CheckExact(o);
  if (plain) {
    const at::Tensor& n = THPVariable_Unpack(o);
    plain = ordinary(n) && is_i32(n) && n.numel() > 0 && n.numel() <= INT32_MAX && n.get_device() == c10::hip::current_device();
    if (plain) {
      int32_t* counts = static_cast<int32_t*>(ptr(n));
      const int batch = (int)n.numel();
      void* stream = stream_handle(nullptr);
      check(unlocked([&] { return jk::launch_tree_reset(counts, batch, static_cast<hipStream_t>(stream)) == hipSuccess ? JK_OK : JK_ERR_HIP; }), "tree_reset");
      n.unsafeGetTensorImpl()->bump_version();
    }
  }
  return PyBool_FromLong(plain);
}
PyObject* tree_finalize(Args& a) {  // state, n_keep, stream -> (tokens, parent, q_row, old_index, n_valid)
  const Py_ssize_t first = a.at;
  const TreeState t = read_tree_state(a);
  const at::Tensor& like = THPVariable_Unpack(a.a[first]);
  const int32_t keep = a.i32();
  void* stream = stream_handle(a.next());
  at::Tensor o[4], n;
  check(unlocked([&] {
          n = empty({t.batch}, at::kInt, like);
          for (at::Tensor& x : o) x = empty({t.batch, keep > 0 ? keep : 0}, at::kInt, like);
          auto out = [&](int i) { return static_cast<int32_t*>(ptr(o[i])); };
          return jk_tree_finalize(&t.s, t.batch, keep, out(0), out(1), out(2), out(3), static_cast<int32_t*>(ptr(n)), stream);
        }),
        "jk_tree_finalize");
  return pack(wrap(std::move(o[0])), wrap(std::move(o[1])), wrap(std::move(o[2])), wrap(std::move(o[3])), wrap(std::move(n)));
}
PyObject* gather_draft_probs(Args& a) {  // q_all, q_row, stream
  const at::Tensor &q = a.tensor(), &row = a.tensor();
  if (!is_f32(q) || !is_i32(row)) fail(PyExc_TypeError, "q_all contiguous float32, q_row contiguous int32");
  dims(row, 2, "q_row must be [B, N]");
  const int64_t V = q.size(-1), B = row.size(0), N = row.size(1);
  void* stream = stream_handle(a.next());
  at::Tensor out;
  check(unlocked([&] {
          out = empty({B, N, V}, at::kFloat, q);
          return jk_gather_draft_probs((int32_t)B, (int32_t)N, (int32_t)V, static_cast<const float*>(ptr(q)), V ? q.numel() / V : 0,
                                       ints(&row), static_cast<float*>(ptr(out)), stream);
        }),
        "jk_gather_draft_probs");
  return wrap(std::move(out));
}

PyObject* stream_of(Args& a) { return PyLong_FromVoidPtr(stream_handle(a.next())); }

// ------------------------------------------------------------------ module
template <PyObject* (*F)(Args&)>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args args{a, n};
  try {
    return F(args);
  } catch (const PyFailure&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}
template <PyObject* (*F)(Args&)>
constexpr PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<F>)), METH_FASTCALL, nullptr};
}
PyObject* set_error_class(PyObject*, PyObject* cls) {
  Py_INCREF(cls);
  Py_XSETREF(g_error_class, cls);
  Py_RETURN_NONE;
}
PyMethodDef methods[] = {
    method<attention>("attention"), method<prepare_attention>("prepare_attention"),
    method<accept>("accept"), method<prepare_accept>("prepare_accept"),
    method<commit>("commit"), method<prepare_commit>("prepare_commit"),
    method<heads>("draft_heads"), method<prepare_heads>("prepare_draft_heads"),
    method<moe>("moe_experts"), method<prepare_moe>("prepare_moe_experts"),
    method<linear>("linear"), method<tree_grow>("tree_grow"), method<tree_grow_tail>("tree_grow_tail"),
    method<tree_fill_static>("tree_fill_static"), method<tree_finalize>("tree_finalize"), method<tree_reset>("tree_reset"),
    method<gather_draft_probs>("gather_draft_probs"), method<stream_of>("stream_handle"),
    {"set_error_class", set_error_class, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "native call marshalling of libjakiro_verify", -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  prepared_type.tp_name = "paper_2502_06282_amd._native.PreparedCall";
  prepared_type.tp_basicsize = sizeof(PreparedCall);
  prepared_type.tp_dealloc = prepared_dealloc;
  prepared_type.tp_flags = Py_TPFLAGS_DEFAULT;
  prepared_type.tp_doc = "A library call with its arguments marshalled once: launch(stream=None) issues it";
  prepared_type.tp_methods = prepared_methods;
  if (PyType_Ready(&prepared_type) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  Py_INCREF(&prepared_type);
  if (PyModule_AddObject(m, "PreparedCall", reinterpret_cast<PyObject*>(&prepared_type)) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
