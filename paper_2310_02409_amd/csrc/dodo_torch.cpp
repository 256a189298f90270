// The binding's calls on plain arguments, in native code: checks, allocation of missing results, current stream, library
// call.  A call costs 1 us or less beyond its kernel launch (3.3 to 4.2 us) and its allocations (0.8 us each), where
// attribute look-ups, ctypes conversions and the interpreter took 3 to 4.5 us.
//
// Every function takes the positional arguments of the Python function of the same name and returns its result, or None
// where an argument is not in the plain form -- exact tensors on the GPU, contiguous, of the expected types and shapes,
// whole numbers that fit -- and the Python function then does the call itself, with its own checks and errors.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cmath>
#include <initializer_list>
#include <limits>

#include "dodo.h"

namespace {

// entry points of the library that the binding has loaded, and the Python function that raises its error
struct Entries {
  decltype(&dodo_score) score = nullptr;
  decltype(&dodo_select_topk) select_topk = nullptr;
  decltype(&dodo_gather_nuggets) gather = nullptr;
  decltype(&dodo_nugget_attention_workspace_bytes) attention_ws = nullptr;
  decltype(&dodo_nugget_attention_workspace_bytes_grouped) attention_ws_grouped = nullptr;
  decltype(&dodo_nugget_attention) attention = nullptr;
  decltype(&dodo_nugget_attention_indexed) attention_indexed = nullptr;
  decltype(&dodo_nugget_attention_cached) attention_cached = nullptr;
  decltype(&dodo_stream_append) stream_append = nullptr;
  decltype(&dodo_score_mlp_workspace_bytes) score_mlp_ws = nullptr;
  decltype(&dodo_score_mlp) score_mlp = nullptr;
  decltype(&dodo_threshold_from_sample_workspace_bytes) threshold_ws = nullptr;
  decltype(&dodo_threshold_from_sample) threshold = nullptr;
  decltype(&dodo_select_threshold) select_threshold = nullptr;
  decltype(&dodo_segment_plan) segment_plan = nullptr;
  decltype(&dodo_nugget_attention_segments) attention_segments = nullptr;
  decltype(&dodo_ste_score_grad_workspace_bytes) ste_ws = nullptr;
  decltype(&dodo_ste_score_grad) ste = nullptr;
} L;
PyObject* raise_error = nullptr;

struct NotPlain {};  // thrown and caught inside this file: the caller is told None

void require(bool ok) {
  if (!ok) throw NotPlain{};
}

// A tensor in the plain form: of torch's own class, strided, on the GPU, contiguous, no wrapper of a transform.
const at::Tensor& tensor(PyObject* o) {
  require(THPVariable_CheckExact(o));
  const at::Tensor& t = THPVariable_Unpack(o);
  using K = c10::DispatchKey;
  require(t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() && t.has_storage() &&
          !t.key_set().has_any(c10::DispatchKeySet({K::Python, K::FuncTorchBatched, K::FuncTorchGradWrapper, K::Functionalize,
                                                    K::Conjugate, K::Negative, K::ZeroTensor})));
  return t;
}
at::Tensor optional_tensor(PyObject* o) { return o == Py_None ? at::Tensor() : tensor(o); }
const at::Tensor& int32_tensor(PyObject* o) {
  const at::Tensor& t = tensor(o);
  require(t.scalar_type() == at::kInt);
  return t;
}
int64_t whole(PyObject* o) {
  require(PyLong_CheckExact(o));
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  require(overflow == 0);
  return v;
}
int32_t int32(int64_t v) {
  require(v >= std::numeric_limits<int32_t>::min() && v <= std::numeric_limits<int32_t>::max());
  return static_cast<int32_t>(v);
}
double real(PyObject* o) {
  require(PyFloat_CheckExact(o));
  return PyFloat_AS_DOUBLE(o);
}
bool truth(PyObject* o) {
  require(o == Py_True || o == Py_False);
  return o == Py_True;
}
int dtype_code(const at::Tensor& t) {
  require(t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16);
  return t.scalar_type() == at::kFloat ? DODO_DTYPE_F32 : DODO_DTYPE_BF16;
}
void* ptr(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
int32_t* iptr(const at::Tensor& t) { return static_cast<int32_t*>(ptr(t)); }
float* fptr(const at::Tensor& t) { return static_cast<float*>(ptr(t)); }
size_t bytes_of(const at::Tensor& ws) { return ws.defined() ? static_cast<size_t>(ws.numel()) : 0; }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }
PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }

// an argument that is handed back is the caller's own object
PyObject* same_or_new(PyObject* given, const at::Tensor& t) {
  if (given == Py_None) return wrap(t);
  Py_INCREF(given);
  return given;
}

struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// Runs `call` -- the allocation of missing results, then the library call -- without the interpreter lock, as torch's own
// functions and a call through ctypes do (an allocation may wait for the device, for another thread's or for an allocator that
// needs the interpreter); raises the binding's error if it fails.
template <class F>
bool run(const char* where, F call) {
  int rc;
  {
    Unlocked u;
    rc = call();
  }
  if (rc == 0) return true;
  PyObject* r = PyObject_CallFunction(raise_error, "is", rc, where);
  Py_XDECREF(r);
  return false;
}

// C++ exceptions end here: what is not plain is left to Python, and so is what torch refuses (an allocation that fails
// is then asked for again, and reported, there).
template <class F>
PyObject* guarded(PyObject* const* a, Py_ssize_t given, Py_ssize_t expected, F body) {
  if (given != expected || raise_error == nullptr) Py_RETURN_NONE;
  try {
    return body(a);
  } catch (const NotPlain&) {
  } catch (const std::exception&) {
  }
  PyErr_Clear();
  Py_RETURN_NONE;
}

PyObject* score(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 4, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &hidden = tensor(a[0]), &w = tensor(a[1]);
    const float bias = static_cast<float>(real(a[2]));
    at::Tensor scores = optional_tensor(a[3]);
    require(hidden.dim() == 2 && w.dim() == 1 && w.size(0) == hidden.size(1) && w.scalar_type() == hidden.scalar_type());
    const int code = dtype_code(hidden);
    const int64_t N = hidden.size(0);
    require(!scores.defined() || (scores.scalar_type() == at::kFloat && scores.numel() == N));
    const int32_t d = int32(hidden.size(1));
    if (!run("dodo_score", [&] {
          if (!scores.defined()) scores = at::empty({N}, hidden.options().dtype(at::kFloat));
          return L.score(ptr(hidden), ptr(w), bias, code, N, d, hidden.stride(0), fptr(scores), stream());
        }))
      return nullptr;
    return same_or_new(a[3], scores);
  });
}

// (one_workgroup: sequences up to this length get no workspace of their own)
PyObject* select_topk(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 10, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &scores = tensor(a[0]), &cu_seqlens = int32_tensor(a[1]), &cu_nuggets = int32_tensor(a[2]);
    const int32_t max_n = int32(whole(a[3])), max_k = int32(whole(a[4]));
    const int64_t total = whole(a[5]), flags = whole(a[6]);
    at::Tensor idx = optional_tensor(a[7]), ws = optional_tensor(a[8]);
    require(scores.scalar_type() == at::kFloat && cu_seqlens.numel() == cu_nuggets.numel() && flags >= 0 && flags <= 0x7fffffff);
    require(ws.defined() || max_n <= whole(a[9]));
    require(cu_seqlens.numel() >= 1 && total >= 0);
    require(!idx.defined() || (idx.scalar_type() == at::kInt && idx.numel() >= total));
    const int32_t B = int32(cu_seqlens.numel() - 1);
    if (!run("dodo_select_topk", [&] {
          if (!idx.defined()) idx = at::empty({total}, cu_seqlens.options().device(scores.device()));
          return L.select_topk(fptr(scores), iptr(cu_seqlens), iptr(cu_nuggets), B, max_n, max_k, static_cast<uint32_t>(flags),
                               iptr(idx), ptr(ws), bytes_of(ws), stream());
        }))
      return nullptr;
    return same_or_new(a[7], idx);
  });
}

PyObject* gather_nuggets(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 9, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &K = tensor(a[0]), &V = tensor(a[1]), &idx = tensor(a[2]), &cu_seqlens = tensor(a[3]), &cu_nuggets = tensor(a[4]);
    const int64_t total = whole(a[5]), layout = whole(a[6]);
    at::Tensor Kn = optional_tensor(a[7]), Vn = optional_tensor(a[8]);
    require(K.dim() == 3 && V.sizes() == K.sizes() && V.strides() == K.strides() && V.scalar_type() == K.scalar_type());
    require(total >= 0 && (layout == DODO_LAYOUT_TOKEN_MAJOR || layout == DODO_LAYOUT_HEAD_MAJOR) && cu_seqlens.numel() >= 1);
    const int code = dtype_code(K);
    const int64_t h_kv = K.size(1), d_h = K.size(2);
    const bool token = layout == DODO_LAYOUT_TOKEN_MAJOR;
    const int64_t shape[3] = {token ? total : h_kv, token ? h_kv : total, d_h};
    require((!Kn.defined() || Kn.sizes() == at::IntArrayRef(shape)) && (!Vn.defined() || Vn.sizes() == at::IntArrayRef(shape)));
    const int32_t B = int32(cu_seqlens.numel() - 1), h = int32(h_kv), dh = int32(d_h);
    if (!run("dodo_gather_nuggets", [&] {
          if (!Kn.defined()) Kn = at::empty(shape, K.options());
          if (!Vn.defined()) Vn = at::empty(shape, K.options());
          return L.gather(ptr(K), ptr(V), code, iptr(idx), iptr(cu_seqlens), iptr(cu_nuggets), B, total, h, dh, K.stride(0), ptr(Kn),
                          ptr(Vn), static_cast<int>(layout), stream());
        }))
      return nullptr;
    PyObject* k = same_or_new(a[7], Kn);
    PyObject* v = same_or_new(a[8], Vn);
    if (k == nullptr || v == nullptr) {
      Py_XDECREF(k);
      Py_XDECREF(v);
      return nullptr;
    }
    PyObject* both = PyTuple_New(2);
    PyTuple_SET_ITEM(both, 0, k);
    PyTuple_SET_ITEM(both, 1, v);
    return both;
  });
}

// What the attention calls share: scale, results and workspace, and the pair that they return.
struct AttentionArgs {
  const at::Tensor &Q, &cu_q;
  int32_t H, d_h, B, max_q, max_k, max_local;
  int code;
  float scale;
  bool want;
  at::Tensor O, lse, ws;
  PyObject *O_given, *lse_given;

  AttentionArgs(PyObject* q, PyObject* cu, PyObject* mq, PyObject* mk, PyObject* ml, PyObject* softmax_scale, PyObject* o, PyObject* l,
                PyObject* want_lse, PyObject* w)
      : Q(tensor(q)), cu_q(tensor(cu)), O(optional_tensor(o)), lse(optional_tensor(l)), ws(optional_tensor(w)), O_given(o), lse_given(l) {
    require(Q.dim() == 3 && cu_q.numel() >= 1 && Q.size(2) > 0);
    H = int32(Q.size(1));
    d_h = int32(Q.size(2));
    B = int32(cu_q.numel() - 1);
    max_q = int32(whole(mq));
    max_k = int32(whole(mk));
    max_local = int32(whole(ml));
    code = dtype_code(Q);
    scale = static_cast<float>(softmax_scale == Py_None ? 1.0 / std::sqrt(static_cast<double>(d_h)) : real(softmax_scale));
    want = truth(want_lse);
  }
  // Missing results, and a workspace by the rule of _attention_workspace
  void allocate(size_t need, bool grouped) {
    if (!O.defined()) O = at::empty_like(Q);
    if (!lse.defined() && want) lse = at::empty({Q.size(0), Q.size(1)}, Q.options().dtype(at::kFloat));
    const bool block = code == DODO_DTYPE_BF16 && max_q >= DODO_ATTENTION_BLOCK_MIN_Q;
    if (need == 0 || ws.defined() || (!grouped && !block && 2ll * B * H * max_q > 256)) return;
    if (block) {
      ws = at::empty({static_cast<int64_t>(need)}, Q.options().dtype(at::kByte));
      return;
    }
    ws = at::zeros({static_cast<int64_t>(need)}, Q.options().dtype(at::kByte));
  }
  PyObject* result() const {
    PyObject* o = same_or_new(O_given, O);
    if (o == nullptr) return nullptr;
    PyObject* l = Py_None;
    if (lse.defined()) l = same_or_new(lse_given, lse); else Py_INCREF(l);
    if (l == nullptr) {
      Py_DECREF(o);
      return nullptr;
    }
    PyObject* both = PyTuple_New(2);
    PyTuple_SET_ITEM(both, 0, o);
    PyTuple_SET_ITEM(both, 1, l);
    return both;
  }
};

PyObject* nugget_attention(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 17, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &Kn = tensor(a[1]), &Vn = tensor(a[2]), &Kl = tensor(a[3]), &Vl = tensor(a[4]), &cu_n = tensor(a[6]), &cu_l = tensor(a[7]);
    const int64_t layout = whole(a[12]);
    require(Kl.dim() >= 2 && Kn.dim() >= 2 && (layout == DODO_LAYOUT_TOKEN_MAJOR || layout == DODO_LAYOUT_HEAD_MAJOR));
    AttentionArgs p(a[0], a[5], a[8], a[9], a[10], a[11], a[13], a[14], a[15], a[16]);
    const int32_t H_kv = int32(Kl.size(1));
    const int64_t Kt = Kn.size(layout == DODO_LAYOUT_TOKEN_MAJOR ? 0 : 1);
    if (!run("dodo_nugget_attention", [&] {
          p.allocate(L.attention_ws_grouped(p.B, p.H, H_kv, p.d_h, p.max_q, p.max_k, p.max_local, p.code),
                     p.code == DODO_DTYPE_BF16 && static_cast<int64_t>(p.H) * p.max_q >= 4ll * H_kv);
          return L.attention(ptr(p.Q), ptr(Kn), ptr(Vn), ptr(Kl), ptr(Vl), iptr(p.cu_q), iptr(cu_n), iptr(cu_l), p.B, p.H, H_kv, p.d_h,
                             p.max_q, p.max_k, p.max_local, Kt, p.scale, p.code, static_cast<int>(layout), ptr(p.O), fptr(p.lse),
                             ptr(p.ws), bytes_of(p.ws), stream());
        }))
      return nullptr;
    return p.result();
  });
}

PyObject* nugget_attention_indexed(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 19, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &K = tensor(a[1]), &V = tensor(a[2]), &idx = tensor(a[3]), &cu_s = tensor(a[4]), &Kl = tensor(a[5]),
                     &Vl = tensor(a[6]), &cu_n = tensor(a[8]), &cu_l = tensor(a[9]);
    require(K.dim() == 3 && V.dim() == 3 && K.strides() == V.strides() && K.stride(2) == 1 && K.stride(1) == K.size(2));
    const int32_t max_n = int32(whole(a[13]));
    AttentionArgs p(a[0], a[7], a[10], a[11], a[12], a[14], a[15], a[16], a[17], a[18]);
    const int32_t H_kv = int32(K.size(1));
    if (!run("dodo_nugget_attention_indexed", [&] {
          p.allocate(L.attention_ws(p.B, p.H, p.d_h, p.max_q, p.max_k, p.max_local, p.code), false);
          return L.attention_indexed(ptr(p.Q), ptr(K), ptr(V), iptr(idx), iptr(cu_s), ptr(Kl), ptr(Vl), iptr(p.cu_q), iptr(cu_n),
                                     iptr(cu_l), p.B, p.H, H_kv, p.d_h, p.max_q, p.max_k, p.max_local, max_n, K.stride(0), p.scale,
                                     p.code, ptr(p.O), fptr(p.lse), ptr(p.ws), bytes_of(p.ws), stream());
        }))
      return nullptr;
    return p.result();
  });
}

PyObject* nugget_attention_cached(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 18, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &Kn = tensor(a[1]), &Vn = tensor(a[2]), &Kl = tensor(a[3]), &Vl = tensor(a[4]), &start = tensor(a[6]),
                     &len = tensor(a[7]), &cu_l = tensor(a[8]);
    const int64_t layout = whole(a[13]);
    require(Kl.dim() >= 2 && Kn.dim() >= 2 && (layout == DODO_LAYOUT_TOKEN_MAJOR || layout == DODO_LAYOUT_HEAD_MAJOR));
    AttentionArgs p(a[0], a[5], a[9], a[10], a[11], a[12], a[14], a[15], a[16], a[17]);
    const int32_t H_kv = int32(Kl.size(1));
    const int64_t Kt = Kn.size(layout == DODO_LAYOUT_TOKEN_MAJOR ? 0 : 1);
    if (!run("dodo_nugget_attention_cached", [&] {
          p.allocate(L.attention_ws_grouped(p.B, p.H, H_kv, p.d_h, p.max_q, p.max_k, p.max_local, p.code),
                     p.code == DODO_DTYPE_BF16 && static_cast<int64_t>(p.H) * p.max_q >= 4ll * H_kv);
          return L.attention_cached(ptr(p.Q), ptr(Kn), ptr(Vn), ptr(Kl), ptr(Vl), iptr(p.cu_q), iptr(start), iptr(len), iptr(cu_l), p.B,
                                    p.H, H_kv, p.d_h, p.max_q, p.max_k, p.max_local, Kt, p.scale, p.code, static_cast<int>(layout),
                                    ptr(p.O), fptr(p.lse), ptr(p.ws), bytes_of(p.ws), stream());
        }))
      return nullptr;
    return p.result();
  });
}

PyObject* nugget_attention_segments(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 19, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &Kn = tensor(a[1]), &Vn = tensor(a[2]), &K = tensor(a[3]), &V = tensor(a[4]), &nug_start = tensor(a[6]),
                     &nug_len = tensor(a[7]), &loc_start = tensor(a[8]), &loc_len = tensor(a[9]);
    const int64_t layout = whole(a[14]);
    require(K.dim() >= 2 && Kn.dim() >= 2 && (layout == DODO_LAYOUT_TOKEN_MAJOR || layout == DODO_LAYOUT_HEAD_MAJOR));
    AttentionArgs p(a[0], a[5], a[10], a[11], a[12], a[13], a[15], a[16], a[17], a[18]);
    const int32_t H_kv = int32(K.size(1));
    const int64_t Kt = Kn.size(layout == DODO_LAYOUT_TOKEN_MAJOR ? 0 : 1);
    if (!run("dodo_nugget_attention_segments", [&] {
          p.allocate(L.attention_ws_grouped(p.B, p.H, H_kv, p.d_h, p.max_q, p.max_k, p.max_local, p.code),
                     p.code == DODO_DTYPE_BF16 && static_cast<int64_t>(p.H) * p.max_q >= 4ll * H_kv);
          return L.attention_segments(ptr(p.Q), ptr(Kn), ptr(Vn), ptr(K), ptr(V), iptr(p.cu_q), iptr(nug_start), iptr(nug_len),
                                      iptr(loc_start), iptr(loc_len), p.B, p.H, H_kv, p.d_h, p.max_q, p.max_k, p.max_local, Kt, p.scale,
                                      p.code, static_cast<int>(layout), ptr(p.O), fptr(p.lse), ptr(p.ws), bytes_of(p.ws), stream());
        }))
      return nullptr;
    return p.result();
  });
}

// (True: done)
PyObject* stream_append(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 8, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &scores = tensor(a[0]), &lam = tensor(a[1]), &K_rows = tensor(a[2]), &V_rows = tensor(a[3]), &counts = tensor(a[4]),
                     &Kn = tensor(a[5]), &Vn = tensor(a[6]);
    const at::Tensor dropped = optional_tensor(a[7]);
    require(K_rows.dim() == 3 && Kn.dim() == 4 && V_rows.strides() == K_rows.strides());
    require(Kn.size(0) == K_rows.size(0) && Kn.size(2) == K_rows.size(1) && Kn.size(3) == K_rows.size(2));
    const int code = dtype_code(K_rows);
    const int32_t B = int32(K_rows.size(0)), h = int32(K_rows.size(1)), dh = int32(K_rows.size(2)), cap = int32(Kn.size(1));
    require(K_rows.stride(2) == 1 && K_rows.stride(1) == dh);
    if (!run("dodo_stream_append", [&] {
          return L.stream_append(fptr(scores), fptr(lam), ptr(K_rows), ptr(V_rows), code, B, h, dh, K_rows.stride(0), cap, iptr(counts),
                                 iptr(dropped), ptr(Kn), ptr(Vn), stream());
        }))
      return nullptr;
    Py_RETURN_TRUE;
  });
}

PyObject* score_mlp(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 8, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &hidden = tensor(a[0]), &W1 = tensor(a[1]), &b1 = tensor(a[2]), &w2 = tensor(a[3]);
    const float b2 = static_cast<float>(real(a[4]));
    const int act = int32(whole(a[5]));
    at::Tensor out = optional_tensor(a[6]), ws = optional_tensor(a[7]);
    require(hidden.dim() == 2 && W1.dim() == 2 && b1.dim() == 1 && w2.dim() == 1);
    const int64_t N = hidden.size(0);
    const int32_t d = int32(hidden.size(1)), d_hid = int32(W1.size(0));
    require(W1.size(1) == d && b1.size(0) == d_hid && w2.size(0) == d_hid && b1.scalar_type() == at::kFloat);
    require(W1.scalar_type() == hidden.scalar_type() && w2.scalar_type() == hidden.scalar_type());
    const int code = dtype_code(hidden);
    if (!run("dodo_score_mlp", [&] {
          if (!out.defined()) out = at::empty({N}, hidden.options().dtype(at::kFloat));
          const size_t need = ws.defined() ? 0 : L.score_mlp_ws(code, N, d, d_hid);
          if (need > 0) ws = at::empty({static_cast<int64_t>(need)}, hidden.options().dtype(at::kByte));
          return L.score_mlp(ptr(hidden), ptr(W1), fptr(b1), ptr(w2), b2, act, code, N, d, d_hid, hidden.stride(0), fptr(out), ptr(ws),
                             bytes_of(ws), stream());
        }))
      return nullptr;
    return same_or_new(a[6], out);
  });
}

// a tuple of the tensors, in order
PyObject* tuple_of(std::initializer_list<const at::Tensor*> tensors) {
  PyObject* all = PyTuple_New(static_cast<Py_ssize_t>(tensors.size()));
  if (all == nullptr) return nullptr;
  Py_ssize_t i = 0;
  for (const at::Tensor* t : tensors) {
    PyObject* o = wrap(*t);
    if (o == nullptr) {
      Py_DECREF(all);
      return nullptr;
    }
    PyTuple_SET_ITEM(all, i++, o);
  }
  return all;
}

// (one_workgroup: samples up to this length get no workspace of their own)
PyObject* threshold_from_sample(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 6, [](PyObject* const* a) -> PyObject* {
    const at::Tensor& sample = tensor(a[0]);
    const int64_t num = whole(a[1]), den = whole(a[2]), one_workgroup = whole(a[5]);
    at::Tensor out = optional_tensor(a[3]), ws = optional_tensor(a[4]);
    require(sample.scalar_type() == at::kFloat);
    const int64_t count = sample.numel();
    if (!run("dodo_threshold_from_sample", [&] {
          if (!out.defined()) out = at::empty({1}, sample.options());
          const size_t need = ws.defined() || count <= one_workgroup ? 0 : L.threshold_ws(count);
          if (need > 0) ws = at::empty({static_cast<int64_t>(need)}, sample.options().dtype(at::kByte));
          return L.threshold(fptr(sample), count, num, den, fptr(out), ptr(ws), bytes_of(ws), stream());
        }))
      return nullptr;
    return same_or_new(a[3], out);
  });
}

PyObject* select_threshold(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 3, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &scores = tensor(a[0]), &cu_seqlens = tensor(a[1]), &lam = tensor(a[2]);
    require(scores.scalar_type() == at::kFloat && lam.scalar_type() == at::kFloat && cu_seqlens.numel() >= 1);
    const int32_t B = int32(cu_seqlens.numel() - 1);
    at::Tensor counts, cu_nuggets, idx;
    if (!run("dodo_select_threshold", [&] {
          const auto ints = scores.options().dtype(at::kInt);
          counts = at::empty({B}, ints);
          cu_nuggets = at::empty({static_cast<int64_t>(B) + 1}, ints);
          idx = at::empty({std::max<int64_t>(1, scores.numel())}, ints);
          return L.select_threshold(fptr(scores), iptr(cu_seqlens), B, fptr(lam), iptr(counts), iptr(cu_nuggets), iptr(idx), stream());
        }))
      return nullptr;
    return tuple_of({&counts, &cu_nuggets, &idx});
  });
}

PyObject* segment_plan(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 6, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &idx = tensor(a[0]), &cu_seqlens = tensor(a[1]), &cu_nuggets = tensor(a[2]);
    const int32_t seg_len = int32(whole(a[3])), tau = int32(whole(a[4])), capacity = int32(whole(a[5]));
    require(cu_seqlens.numel() >= 1 && capacity >= 0);
    const int32_t B = int32(cu_seqlens.numel() - 1);
    at::Tensor cu_q, nug_start, nug_len, loc_start, loc_len, count;
    if (!run("dodo_segment_plan", [&] {
          const auto ints = cu_seqlens.options().dtype(at::kInt);
          cu_q = at::empty({static_cast<int64_t>(capacity) + 1}, ints);
          for (at::Tensor* t : {&nug_start, &nug_len, &loc_start, &loc_len}) *t = at::empty({capacity}, ints);
          count = at::empty({1}, ints);
          return L.segment_plan(iptr(idx), iptr(cu_seqlens), iptr(cu_nuggets), B, seg_len, tau, capacity, iptr(cu_q), iptr(nug_start),
                                iptr(nug_len), iptr(loc_start), iptr(loc_len), iptr(count), stream());
        }))
      return nullptr;
    return tuple_of({&cu_q, &nug_start, &nug_len, &loc_start, &loc_len, &count});
  });
}

PyObject* ste_score_grad(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 16, [](PyObject* const* a) -> PyObject* {
    const at::Tensor &Q = tensor(a[0]), &Kn = tensor(a[1]), &Vn = tensor(a[2]), &dO = tensor(a[3]), &O = tensor(a[4]), &lse = tensor(a[5]),
                     &cu_q = tensor(a[6]), &cu_n = tensor(a[7]);
    const int32_t max_q = int32(whole(a[8])), max_k = int32(whole(a[9]));
    const int64_t layout = whole(a[12]);
    at::Tensor grad = optional_tensor(a[13]), ws = optional_tensor(a[15]);
    const bool accumulate = truth(a[14]);
    require(Q.dim() == 3 && Kn.dim() >= 2 && cu_q.numel() >= 1 && Q.size(2) > 0);
    require(layout == DODO_LAYOUT_TOKEN_MAJOR || layout == DODO_LAYOUT_HEAD_MAJOR);
    const int64_t Sq = Q.size(0), rows[2] = {Sq, Q.size(1)};
    const int64_t Kt = Kn.size(layout == DODO_LAYOUT_TOKEN_MAJOR ? 0 : 1);
    const int32_t B = int32(cu_q.numel() - 1), H = int32(Q.size(1)), d_h = int32(Q.size(2));
    const int32_t H_kv = int32(Kn.size(layout == DODO_LAYOUT_TOKEN_MAJOR ? 1 : 0));
    const int code = dtype_code(Q);
    for (const at::Tensor* t : {&dO, &O}) require(t->sizes() == Q.sizes() && t->scalar_type() == Q.scalar_type());
    require(Kn.scalar_type() == Q.scalar_type() && Vn.scalar_type() == Q.scalar_type());
    require(lse.scalar_type() == at::kFloat && lse.sizes() == at::IntArrayRef(rows) && (grad.defined() || !accumulate));
    const double scale = a[10] == Py_None ? 1.0 / std::sqrt(static_cast<double>(d_h)) : real(a[10]);
    const double grad_scale = a[11] == Py_None ? scale : real(a[11]);
    if (!run("dodo_ste_score_grad", [&] {
          if (!grad.defined()) grad = at::empty({Kt}, lse.options());
          const size_t need = ws.defined() ? 0 : L.ste_ws(Sq, H, Kt);
          if (need > 0) ws = at::empty({static_cast<int64_t>(need)}, lse.options().dtype(at::kByte));
          return L.ste(ptr(Q), ptr(Kn), ptr(Vn), ptr(dO), ptr(O), fptr(lse), iptr(cu_q), iptr(cu_n), B, H, H_kv, d_h, max_q, max_k, Sq, Kt,
                       static_cast<float>(scale), static_cast<float>(grad_scale), accumulate ? 1 : 0, code, static_cast<int>(layout),
                       fptr(grad), ptr(ws), bytes_of(ws), stream());
        }))
      return nullptr;
    return same_or_new(a[13], grad);
  });
}

constexpr int kEntries = 18;

// bind(raise, address, ...): the function that raises the binding's error and the entry points, in the order of Entries
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* p[kEntries];
  if (n != kEntries + 1) {
    PyErr_SetString(PyExc_TypeError, "bind takes a function and the addresses of all entry points");
    return nullptr;
  }
  for (int i = 0; i < kEntries; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i + 1]);
    if (p[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
      return nullptr;
    }
  }
  L.score = reinterpret_cast<decltype(L.score)>(p[0]);
  L.select_topk = reinterpret_cast<decltype(L.select_topk)>(p[1]);
  L.gather = reinterpret_cast<decltype(L.gather)>(p[2]);
  L.attention_ws = reinterpret_cast<decltype(L.attention_ws)>(p[3]);
  L.attention_ws_grouped = reinterpret_cast<decltype(L.attention_ws_grouped)>(p[4]);
  L.attention = reinterpret_cast<decltype(L.attention)>(p[5]);
  L.attention_indexed = reinterpret_cast<decltype(L.attention_indexed)>(p[6]);
  L.attention_cached = reinterpret_cast<decltype(L.attention_cached)>(p[7]);
  L.stream_append = reinterpret_cast<decltype(L.stream_append)>(p[8]);
  L.score_mlp_ws = reinterpret_cast<decltype(L.score_mlp_ws)>(p[9]);
  L.score_mlp = reinterpret_cast<decltype(L.score_mlp)>(p[10]);
  L.threshold_ws = reinterpret_cast<decltype(L.threshold_ws)>(p[11]);
  L.threshold = reinterpret_cast<decltype(L.threshold)>(p[12]);
  L.select_threshold = reinterpret_cast<decltype(L.select_threshold)>(p[13]);
  L.segment_plan = reinterpret_cast<decltype(L.segment_plan)>(p[14]);
  L.attention_segments = reinterpret_cast<decltype(L.attention_segments)>(p[15]);
  L.ste_ws = reinterpret_cast<decltype(L.ste_ws)>(p[16]);
  L.ste = reinterpret_cast<decltype(L.ste)>(p[17]);
  Py_INCREF(a[0]);
  Py_XDECREF(raise_error);
  raise_error = a[0];
  Py_RETURN_NONE;
}

#define DODO_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DODO_METHOD(bind), DODO_METHOD(score), DODO_METHOD(select_topk), DODO_METHOD(gather_nuggets),
                         DODO_METHOD(nugget_attention), DODO_METHOD(nugget_attention_indexed), DODO_METHOD(nugget_attention_cached),
                         DODO_METHOD(nugget_attention_segments), DODO_METHOD(stream_append), DODO_METHOD(score_mlp), DODO_METHOD(threshold_from_sample),
                         DODO_METHOD(select_threshold), DODO_METHOD(segment_plan), DODO_METHOD(ste_score_grad), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_dodo_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dodo_torch() {
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddIntConstant(m, "ATTENTION_BLOCK_MIN_Q", DODO_ATTENTION_BLOCK_MIN_Q) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
