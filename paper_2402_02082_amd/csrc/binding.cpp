// The Python binding's fast path: argument checks and pointer marshalling in
// native code, for the calls of the decoding loop and of draft training named
// in Calls below.
//
// A decoding step makes tens of these calls of about ten microseconds of GPU
// work each, and one checked and marshalled in Python took longer than that
// (host time per call: tree attention of a 5-token chain 15.6 us, the commit
// of 40 layers' caches 92 us).  Every function here takes the same arguments
// as its namesake in _lib.py and makes the same checks.  It returns the
// status of the C call, or None when any argument is not of the plain form
// it handles (an exact torch.Tensor where one is expected, no explicit
// stream, every check passed); the caller then takes the Python path, which
// either makes the call or raises with the reason.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>

#include "glide.h"

namespace {

// Entry points of the loaded library (bind()).
struct Calls {
  decltype(&glide_tree_attn_workspace) tree_attn_workspace;
  decltype(&glide_tree_attn) tree_attn;
  decltype(&glide_verify_commit) verify_commit;
  decltype(&cape_expand_workspace) cape_workspace;
  decltype(&cape_expand) cape;
  decltype(&spec_sample_verify) spec_sample;
  decltype(&glide_rows_matmul) rows_matmul;
  decltype(&glide_block_attn) block_attn;
} calls;
PyObject* raw_stream;  // device index -> current stream handle
PyObject* workspaces;  // {(device index, stream handle): byte tensor}

// An exact torch.Tensor or nullptr.
const at::Tensor* tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

// ... on the GPU, contiguous and of the given type and rank (-1: any).
const at::Tensor* gpu(PyObject* o, at::ScalarType dtype, int rank) {
  const at::Tensor* t = tensor(o);
  if (!t || !t->is_cuda() || !t->is_contiguous() || t->scalar_type() != dtype) return nullptr;
  return rank < 0 || t->dim() == rank ? t : nullptr;
}

bool is_shape(const at::Tensor& t, at::IntArrayRef s) { return t.sizes() == s; }

// A Python int or bool that fits a C int.
bool as_int(PyObject* o, int* v) {
  if (!PyLong_Check(o)) return false;
  int overflow = 0;
  const long x = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int)x;
  return true;
}

bool as_float(PyObject* o, float* v) {
  if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
  const double d = PyFloat_AsDouble(o);
  if (d == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  *v = (float)d;
  return true;
}

bool fits(const at::Tensor& t) {  // every extent passes as a C int
  for (int64_t s : t.sizes())
    if (s > INT32_MAX) return false;
  return true;
}

bool stream_of(const at::Tensor& t, hipStream_t* s, PyObject** handle) {
  PyObject* index = PyLong_FromLong(t.get_device());
  PyObject* h = index ? PyObject_CallOneArg(raw_stream, index) : nullptr;
  Py_XDECREF(index);
  if (!h) {
    PyErr_Clear();
    return false;
  }
  *s = (hipStream_t)PyLong_AsVoidPtr(h);
  if (handle)
    *handle = h;
  else
    Py_DECREF(h);
  return true;
}

// The kept attention workspace of the device and stream, if it is large
// enough; `held` keeps it alive until the call has been enqueued (another
// thread may replace it meanwhile).  `handle` is consumed.
bool kept_workspace(const at::Tensor& on, PyObject* handle, size_t need, at::Tensor* held) {
  PyObject* key = Py_BuildValue("(lN)", (long)on.get_device(), handle);
  PyObject* ws = key ? PyDict_GetItemWithError(workspaces, key) : nullptr;
  Py_XDECREF(key);
  PyErr_Clear();
  const at::Tensor* t = ws ? tensor(ws) : nullptr;
  if (!t || (size_t)t->nbytes() < need) return false;
  *held = *t;
  return true;
}

// A reference that is given back with the scope.
struct Held {
  PyObject* o;
  explicit Held(PyObject* owned) : o(owned) {}
  Held(const Held&) = delete;
  ~Held() { Py_XDECREF(o); }
};

void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }

// Runs `f` without the GIL (the call may wait for the device when it
// validates device data) and returns its status.
template <class F>
PyObject* status_of(F f) {
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

constexpr auto kBf16 = at::kBFloat16;
constexpr auto kF32 = at::kFloat;
constexpr auto kI32 = at::kInt;

// (q, k_cache, v_cache, seq_lens, tree_parents, out, scale, max_splits, workspace, stream)
PyObject* tree_attn(PyObject* const* a, Py_ssize_t n) {
  if (n != 10 || a[9] != Py_None) return nullptr;
  const at::Tensor* q = tensor(a[0]);
  if (!q || (q->scalar_type() != kBf16 && q->scalar_type() != kF32)) return nullptr;
  const auto dtype = q->scalar_type();
  q = gpu(a[0], dtype, 4);
  const at::Tensor *k = gpu(a[1], dtype, 4), *v = gpu(a[2], dtype, 4), *lens = gpu(a[3], kI32, 1);
  const at::Tensor *parents = a[4] == Py_None ? nullptr : gpu(a[4], kI32, 2), *out = gpu(a[5], dtype, 4);
  if (!q || !k || !v || !lens || !out || (!parents && a[4] != Py_None) || !fits(*q) || !fits(*k)) return nullptr;
  const int64_t B = q->size(0), N = q->size(1), H = q->size(2), D = q->size(3), cap = k->size(2);
  if (!is_shape(*k, {B, H, cap, D}) || v->sizes() != k->sizes() || out->sizes() != q->sizes() ||
      !is_shape(*lens, {B}) || (parents && !is_shape(*parents, {B, N})))
    return nullptr;
  float scale;
  int splits;
  if (!as_float(a[6], &scale) || !as_int(a[7], &splits)) return nullptr;
  hipStream_t s;
  at::Tensor ws;
  if (a[8] == Py_None) {
    PyObject* handle;
    if (!stream_of(*q, &s, &handle)) return nullptr;
    const size_t need = calls.tree_attn_workspace(B, N, H, GLIDE_HEAD_DIM, cap, splits);
    if (need == 0)
      Py_DECREF(handle);
    else if (!kept_workspace(*q, handle, need, &ws))
      return nullptr;
  } else {
    const at::Tensor* w = tensor(a[8]);
    if (!w || !stream_of(*q, &s, nullptr)) return nullptr;
    ws = *w;
  }
  void* wp = ws.defined() ? ws.data_ptr() : nullptr;
  const size_t ws_bytes = ws.defined() ? ws.numel() * ws.element_size() : 0;
  void *qp = ptr(q), *kp = ptr(k), *vp = ptr(v), *op = ptr(out);
  const int32_t *lp = (const int32_t*)ptr(lens), *pp = (const int32_t*)ptr(parents);
  return status_of([&] {
    return calls.tree_attn(qp, kp, vp, lp, pp, op, B, N, H, D, cap, dtype == kBf16 ? GLIDE_BF16 : GLIDE_F32, scale,
                           splits, wp, ws_bytes, s);
  });
}

// (logits, cand_tokens, parents, k_caches, v_caches, seq_lens, seq_lens_out, target_argmax, accept_len, last_node,
//  bonus, path, stream); the caches as lists
PyObject* verify_commit(PyObject* const* a, Py_ssize_t n) {
  if (n != 13 || a[12] != Py_None || !PyList_CheckExact(a[3]) || !PyList_CheckExact(a[4])) return nullptr;
  const at::Tensor *logits = gpu(a[0], kF32, 3), *cand = gpu(a[1], kI32, 2), *parents = gpu(a[2], kI32, 2);
  if (!logits || !cand || !parents || !fits(*logits)) return nullptr;
  const int64_t B = cand->size(0), N = cand->size(1), V = logits->size(2);
  if (!is_shape(*logits, {B, N + 1, V}) || !is_shape(*parents, {B, N})) return nullptr;
  const at::Tensor* io[7];  // seq_lens, seq_lens_out, target_argmax, accept_len, last_node, bonus, path
  for (int i = 0; i < 7; ++i) {
    const bool optional = i >= 4;
    io[i] = optional && a[5 + i] == Py_None ? nullptr : gpu(a[5 + i], kI32, -1);
    if (!io[i]) {
      if (optional && a[5 + i] == Py_None) continue;
      return nullptr;
    }
    if (i == 2 ? !is_shape(*io[i], {B, N + 1}) : (i == 6 ? !is_shape(*io[i], {B, N}) : !is_shape(*io[i], {B})))
      return nullptr;
  }
  // the caches themselves are held, not the lists: another thread may change
  // those while the call runs without the GIL
  const Held caches[2] = {Held(PyList_AsTuple(a[3])), Held(PyList_AsTuple(a[4]))};
  if (!caches[0].o || !caches[1].o) return nullptr;
  const Py_ssize_t layers = PyTuple_GET_SIZE(caches[0].o);
  if (layers != PyTuple_GET_SIZE(caches[1].o) || layers > 128) return nullptr;
  int64_t H = 1, cap = N, D = GLIDE_HEAD_DIM;
  int dtype = GLIDE_BF16;
  void* p[2][128];
  const at::Tensor* ref = nullptr;
  for (int m = 0; m < 2; ++m)
    for (Py_ssize_t i = 0; i < layers; ++i) {
      PyObject* o = PyTuple_GET_ITEM(caches[m].o, i);
      if (!ref) {
        const at::Tensor* t = tensor(o);
        if (!t || (t->scalar_type() != kBf16 && t->scalar_type() != kF32)) return nullptr;
        ref = gpu(o, t->scalar_type(), 4);
        if (!ref || ref->size(0) != B || !fits(*ref)) return nullptr;
        H = ref->size(1), cap = ref->size(2), D = ref->size(3);
        dtype = ref->scalar_type() == kBf16 ? GLIDE_BF16 : GLIDE_F32;
      }
      const at::Tensor* t = gpu(o, ref->scalar_type(), 4);
      if (!t || t->sizes() != ref->sizes()) return nullptr;
      p[m][i] = t->data_ptr();
    }
  hipStream_t s;
  if (!stream_of(*logits, &s, nullptr)) return nullptr;
  const float* lp = (const float*)ptr(logits);
  int32_t *cp = (int32_t*)ptr(cand), *pp = (int32_t*)ptr(parents), *q[7];
  for (int i = 0; i < 7; ++i) q[i] = (int32_t*)ptr(io[i]);
  return status_of([&] {
    return calls.verify_commit(lp, V, cp, pp, B, N, p[0], p[1], layers, H, D, cap, dtype, q[0], q[1], q[2], q[3], q[4],
                               q[5], q[6], s);
  });
}

// (draft_probs, k, n_max, tokens_out, parents_out, n_nodes_out, fixed, workspace, stream)
PyObject* cape(PyObject* const* a, Py_ssize_t n) {
  if (n != 9 || a[8] != Py_None) return nullptr;
  const at::Tensor *probs = gpu(a[0], kF32, 3), *tok = gpu(a[3], kI32, 2), *par = gpu(a[4], kI32, 2);
  const at::Tensor* nodes = gpu(a[5], kI32, 1);
  int k, n_max;
  if (!probs || !tok || !par || !nodes || !fits(*probs) || !as_int(a[1], &k) || !as_int(a[2], &n_max) ||
      !PyBool_Check(a[6]))
    return nullptr;
  const int64_t B = probs->size(0), G = probs->size(1), V = probs->size(2);
  if (!is_shape(*tok, {B, n_max}) || !is_shape(*par, {B, n_max}) || !is_shape(*nodes, {B})) return nullptr;
  const bool fixed = a[6] == Py_True;
  hipStream_t s;
  if (!stream_of(*probs, &s, nullptr)) return nullptr;
  at::Tensor own;  // freed on return, to later work of the same stream
  const at::Tensor* ws = &own;
  if (a[7] == Py_None) {
    const int64_t need = calls.cape_workspace(B, G, V);
    own = at::empty({need > 0 ? need : 1}, probs->options().dtype(at::kByte));
  } else if (!(ws = tensor(a[7]))) {
    return nullptr;
  }
  void* wp = ws->data_ptr();
  const size_t ws_bytes = ws->numel() * ws->element_size();
  const float* pp = (const float*)ptr(probs);
  int32_t *o0 = (int32_t*)ptr(tok), *o1 = (int32_t*)ptr(par), *o2 = (int32_t*)ptr(nodes);
  return status_of([&] { return calls.cape(pp, B, G, V, k, fixed, n_max, o0, o1, o2, wp, ws_bytes, s); });
}

// (draft_tokens, draft_probs, target_probs, uniforms, accept_len, next_token, stream)
PyObject* spec_sample(PyObject* const* a, Py_ssize_t n) {
  if (n != 7 || a[6] != Py_None) return nullptr;
  const at::Tensor *tok = gpu(a[0], kI32, 2), *pd = gpu(a[1], kF32, 3), *pt = gpu(a[2], kF32, 3);
  const at::Tensor *u = gpu(a[3], kF32, 2), *acc = gpu(a[4], kI32, 1), *next = gpu(a[5], kI32, 1);
  if (!tok || !pd || !pt || !u || !acc || !next || !fits(*pd)) return nullptr;
  const int64_t B = tok->size(0), G = tok->size(1), V = pd->size(2);
  if (!is_shape(*pd, {B, G, V}) || !is_shape(*pt, {B, G + 1, V}) || !is_shape(*u, {B, G + 1}) ||
      !is_shape(*acc, {B}) || !is_shape(*next, {B}))
    return nullptr;
  hipStream_t s;
  if (!stream_of(*tok, &s, nullptr)) return nullptr;
  const int32_t* tp = (const int32_t*)ptr(tok);
  const float *dp = (const float*)ptr(pd), *gp = (const float*)ptr(pt), *up = (const float*)ptr(u);
  int32_t *ap = (int32_t*)ptr(acc), *np = (int32_t*)ptr(next);
  return status_of([&] { return calls.spec_sample(tp, dp, gp, up, B, G, V, ap, np, s); });
}

// (a, w_t, out, stream)
PyObject* rows_matmul(PyObject* const* a, Py_ssize_t n) {
  if (n != 4 || a[3] != Py_None) return nullptr;
  const at::Tensor *x = gpu(a[0], kBf16, 2), *w = gpu(a[1], kBf16, 2), *out = tensor(a[2]);
  if (!x || !w || !out || (out->scalar_type() != kBf16 && out->scalar_type() != kF32)) return nullptr;
  out = gpu(a[2], out->scalar_type(), 2);
  const int64_t M = x->size(0), K = x->size(1), N = w->size(0);
  if (!out || w->size(1) != K || !is_shape(*out, {M, N}) || !fits(*x) || !fits(*w)) return nullptr;
  hipStream_t s;
  if (!stream_of(*x, &s, nullptr)) return nullptr;
  const int dtype = out->scalar_type() == kBf16 ? GLIDE_BF16 : GLIDE_F32;
  void *xp = ptr(x), *wp = ptr(w), *op = ptr(out);
  return status_of([&] { return calls.rows_matmul(xp, wp, op, M, K, N, dtype, s); });
}

// (q, k_cache, v_cache, out, block, scale, stream)
PyObject* block_attn(PyObject* const* a, Py_ssize_t n) {
  if (n != 7 || a[6] != Py_None) return nullptr;
  const at::Tensor *q = gpu(a[0], kBf16, 4), *k = gpu(a[1], kBf16, 4), *v = gpu(a[2], kBf16, 4);
  const at::Tensor* out = gpu(a[3], kBf16, 4);
  int block;
  float scale;
  if (!q || !k || !v || !out || !as_int(a[4], &block) || !as_float(a[5], &scale) || !fits(*q) || !fits(*k))
    return nullptr;
  const int64_t B = q->size(0), T = q->size(1), H = q->size(2), D = q->size(3), cap = k->size(2);
  if (!is_shape(*k, {B, H, cap, D}) || v->sizes() != k->sizes() || out->sizes() != q->sizes()) return nullptr;
  hipStream_t s;
  if (!stream_of(*q, &s, nullptr)) return nullptr;
  void *qp = ptr(q), *kp = ptr(k), *vp = ptr(v), *op = ptr(out);
  return status_of([&] { return calls.block_attn(qp, kp, vp, op, B, T, H, D, cap, block, scale, s); });
}

// The Python entry of a function above: nullptr and C++ exceptions (a tensor
// without storage, an allocation that failed) become None.
template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  try {
    if (PyObject* r = F(args, n)) return r;
  } catch (...) {
  }
  PyErr_Clear();
  Py_RETURN_NONE;
}

// bind(addresses of the eight entry points in Calls' order, raw_stream, workspaces)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  constexpr int kCalls = sizeof(Calls) / sizeof(void*);
  if (n != 3 || !PyTuple_Check(args[0]) || PyTuple_GET_SIZE(args[0]) != kCalls || !PyDict_Check(args[2])) {
    PyErr_SetString(PyExc_TypeError, "bind(addresses, raw_stream, workspaces)");
    return nullptr;
  }
  void* p[kCalls];
  for (int i = 0; i < kCalls; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(args[0], i));
    if (PyErr_Occurred()) return nullptr;
  }
  memcpy(&calls, p, sizeof(calls));
  Py_INCREF(args[1]);
  Py_INCREF(args[2]);
  Py_XDECREF(raw_stream);
  Py_XDECREF(workspaces);
  raw_stream = args[1];
  workspaces = args[2];
  Py_RETURN_NONE;
}

#define FAST(f) ((PyCFunction)(void (*)(void))(f))
PyMethodDef methods[] = {{"bind", FAST(bind), METH_FASTCALL, nullptr},
                         {"tree_attn", FAST(entry<tree_attn>), METH_FASTCALL, nullptr},
                         {"verify_commit", FAST(entry<verify_commit>), METH_FASTCALL, nullptr},
                         {"cape", FAST(entry<cape>), METH_FASTCALL, nullptr},
                         {"spec_sample", FAST(entry<spec_sample>), METH_FASTCALL, nullptr},
                         {"rows_matmul", FAST(entry<rows_matmul>), METH_FASTCALL, nullptr},
                         {"block_attn", FAST(entry<block_attn>), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
