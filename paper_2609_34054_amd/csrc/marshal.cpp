// Argument marshalling of the Python binding in native code: the checks, sizes
// and strides that binding.py derives from torch tensors, then the C ABI call.
// In Python they cost 10 to 17 us a call, more than the smallest calls' kernels;
// here about 1 us.  Every function takes the address of its C ABI entry point
// (the release or the checked library's) and returns its status, a size the
// caller has to allocate first (as a tuple), or None whenever an argument is not
// what a plain valid call has: binding.py then runs its own checks, which raise
// the error or handle the case.  Nothing is kept from one call to the next.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "precache.h"

namespace {

using at::Tensor;

// A dense tensor of the exact torch class on a HIP device, or nullptr.
const Tensor* tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.unsafeGetTensorImpl()->has_storage()) return nullptr;
  return &t;
}

// Optional tensor argument: *t = nullptr for None; false if it is neither.
bool opt(PyObject* o, const Tensor** t) {
  *t = nullptr;
  return o == Py_None || (*t = tensor(o)) != nullptr;
}

bool bf16(const Tensor* t, int64_t dim) {
  return t->scalar_type() == at::kBFloat16 && t->dim() == dim && t->stride(dim - 1) == 1;
}
bool opt_bf16(const Tensor* t, int64_t dim) { return t == nullptr || bf16(t, dim); }
bool i32(const Tensor* t) { return t->scalar_type() == at::kInt; }

// Contiguous within its first dimension (t[0].is_contiguous()).
bool row_contiguous(const Tensor* t) {
  if (t->size(0) == 0) return false;  // t[0] does not exist
  int64_t want = 1;
  bool empty = false;
  for (int64_t i = 1; i < t->dim(); ++i) empty |= t->size(i) == 0;
  if (empty) return true;
  for (int64_t i = t->dim() - 1; i >= 1; --i) {
    if (t->size(i) != 1 && t->stride(i) != want) return false;
    want *= t->size(i);
  }
  return true;
}

bool alike(const Tensor* a, const Tensor* b) { return a->sizes() == b->sizes() && a->strides() == b->strides(); }
bool alike_opt(const Tensor* a, const Tensor* b) { return a == nullptr || b == nullptr || alike(a, b); }

// Elements between requests, 0 when one buffer serves all; false: neither.
bool req_stride(const Tensor* t, int64_t batch, int64_t* s) {
  *s = 0;
  if (t == nullptr || t->size(0) == 1) return true;
  if (t->size(0) != batch) return false;
  *s = t->stride(0);
  return true;
}

const uint16_t* u16(const Tensor* t) { return t == nullptr ? nullptr : static_cast<const uint16_t*>(t->data_ptr()); }
uint16_t* u16m(const Tensor* t) { return t == nullptr ? nullptr : static_cast<uint16_t*>(t->data_ptr()); }
const int32_t* i32p(const Tensor* t) { return t == nullptr ? nullptr : static_cast<const int32_t*>(t->data_ptr()); }
size_t nbytes(const Tensor* t) { return (size_t)t->numel() * t->element_size(); }

// Integers and doubles of plain Python type; anything else is left to Python.
bool as_int(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0 && !(*v == -1 && PyErr_Occurred());
}
bool as_i32(PyObject* o, int32_t* v) {
  int64_t x;
  if (!as_int(o, &x) || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}
bool as_double(PyObject* o, double* v) {
  if (PyFloat_CheckExact(o)) {
    *v = PyFloat_AS_DOUBLE(o);
    return true;
  }
  int64_t i;
  if (!as_int(o, &i)) return false;
  *v = (double)i;
  return true;
}
bool as_ptr(PyObject* o, void** p) {
  if (!PyLong_CheckExact(o)) return false;
  *p = PyLong_AsVoidPtr(o);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

PyObject* none() {
  PyErr_Clear();
  Py_RETURN_NONE;
}
PyObject* need_bytes(size_t n) { return Py_BuildValue("(n)", (Py_ssize_t)n); }

// Sizes that fit the C ABI's int32 fields.
bool fits(std::initializer_list<int64_t> v) {
  for (int64_t x : v)
    if (x < 0 || x > INT32_MAX) return false;
  return true;
}

// attention(fn, size_fn, noalloc, limit, Q, K, V, Lk, Lv, Bk, Bv, positions,
//           kv_len, theta, scale, O, lse, workspace, stream)
// limit: use at most the bytes size_fn asks for (a workspace of the paged size
// keeps the tile cache off).
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 19) return none();
  void *fn, *size_fn, *stream;
  const bool noalloc = a[2] == Py_True, limit = a[3] == Py_True;
  const Tensor *Q = tensor(a[4]), *K = tensor(a[5]), *V = tensor(a[6]), *pos = tensor(a[11]), *kvl = tensor(a[12]);
  const Tensor *O = tensor(a[15]), *Lk, *Lv, *Bk, *Bv, *lse, *ws;
  double theta, scale;
  if (!as_ptr(a[0], &fn) || !as_ptr(a[1], &size_fn) || !as_ptr(a[18], &stream) || !Q || !K || !V || !pos || !kvl || !O ||
      !opt(a[7], &Lk) || !opt(a[8], &Lv) || !opt(a[9], &Bk) || !opt(a[10], &Bv) || !opt(a[16], &lse) || !opt(a[17], &ws) ||
      !as_double(a[13], &theta) || !as_double(a[14], &scale))
    return none();
  if (!bf16(Q, 4) || !bf16(K, 4) || !bf16(V, 4) || !opt_bf16(Lk, 3) || !opt_bf16(Lv, 3) || !opt_bf16(Bk, 3) ||
      !opt_bf16(Bv, 3) || !alike(K, V))
    return none();
  if (noalloc) {
    if (!bf16(O, 4) || O->sizes() != Q->sizes() || !O->is_contiguous()) return none();
  } else if (!row_contiguous(Q) || !row_contiguous(K) || !row_contiguous(V) || !alike_opt(Lk, Lv) || !alike_opt(Bk, Bv)) {
    return none();
  }
  const Tensor *lr = Lk ? Lk : Lv, *bt = Bk ? Bk : Bv;
  const int64_t batch = Q->size(0), n_tok = Q->size(1), n_q = Q->size(2), d = Q->size(3);
  const int64_t s_cap = K->size(1), n_kv = K->size(2), rank = lr ? lr->size(2) : 0;
  if (K->size(3) != d || (lr && lr->size(1) != s_cap) || (bt && (bt->size(1) != rank || bt->size(2) != n_kv * d)) ||
      !fits({batch, n_tok, n_q, n_kv, d, rank}))
    return none();
  lrsa_dims dm{};
  dm.batch = (int32_t)batch;
  dm.n_tok = (int32_t)n_tok;
  dm.n_q_heads = (int32_t)n_q;
  dm.n_kv_heads = (int32_t)n_kv;
  dm.head_dim = (int32_t)d;
  dm.rank = (int32_t)rank;
  dm.s_cap = s_cap;
  dm.softmax_scale = (float)scale;
  dm.rope_theta = theta;
  if (!req_stride(K, batch, &dm.kv_req_stride) || !req_stride(lr, batch, &dm.l_req_stride) ||
      !req_stride(bt, batch, &dm.b_req_stride))
    return none();
  if (!i32(pos) || !i32(kvl)) return none();
  if (!noalloc && (pos->dim() != 2 || pos->size(0) != batch || pos->size(1) != n_tok || !pos->is_contiguous() ||
                   kvl->dim() != 1 || kvl->size(0) != batch))
    return none();
  void* wp = nullptr;
  size_t wb = 0;
  if (!noalloc) {
    const size_t need = reinterpret_cast<size_t (*)(const lrsa_dims*)>(size_fn)(&dm);
    if (need > 0 && (ws == nullptr || nbytes(ws) < need)) return need_bytes(need);
    if (ws != nullptr) {
      wp = ws->data_ptr();
      wb = nbytes(ws);
    }
    if (limit) {
      if (wb > need) wb = need;
      if (wb == 0) wp = nullptr;
    }
  }
  const uint16_t *q = u16(Q), *k = u16(K), *v = u16(V), *lk = u16(Lk), *lv = u16(Lv), *bk = u16(Bk), *bv = u16(Bv);
  const int32_t *pp = i32p(pos), *kp = i32p(kvl);
  uint16_t* o = u16m(O);
  float* lp = lse == nullptr ? nullptr : static_cast<float*>(lse->data_ptr());
  prc_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = noalloc ? reinterpret_cast<decltype(&lr_shared_attention_noalloc)>(fn)(&dm, q, k, v, lk, lv, bk, bv, pp, kp, o, lp, stream)
               : reinterpret_cast<decltype(&lr_shared_attention)>(fn)(&dm, q, k, v, lk, lv, bk, bv, pp, kp, o, lp, wp, wb, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong((long)st);
}

// Pool of `nd` dims shared by all requests, or one per request before them.
bool pool(const Tensor* t, int64_t batch, int64_t nd, int64_t* stride) {
  *stride = 0;
  if (t == nullptr) return true;
  if (t->scalar_type() != at::kBFloat16 || (t->dim() != nd && t->dim() != nd + 1) || t->stride(t->dim() - 1) != 1)
    return false;
  if (t->dim() == nd) return t->is_contiguous();
  if (t->size(0) != 1 && t->size(0) != batch) return false;
  if (!t->is_contiguous() && !row_contiguous(t)) return false;
  if (t->size(0) != 1) *stride = t->stride(0);
  return true;
}

// paged(fn, size_fn, Q, K, V, Lk, Lv, Bk, Bv, positions, kv_len, kv_table,
//       lr_table, theta, scale, O, lse, workspace, stream)
PyObject* paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 19) return none();
  void *fn, *size_fn, *stream;
  const Tensor *Q = tensor(a[2]), *K = tensor(a[3]), *V = tensor(a[4]), *pos = tensor(a[9]), *kvl = tensor(a[10]);
  const Tensor *kt = tensor(a[11]), *O = tensor(a[15]), *Lk, *Lv, *Bk, *Bv, *lt, *lse, *ws;
  double theta, scale;
  if (!as_ptr(a[0], &fn) || !as_ptr(a[1], &size_fn) || !as_ptr(a[18], &stream) || !Q || !K || !V || !pos || !kvl || !kt ||
      !O || !opt(a[5], &Lk) || !opt(a[6], &Lv) || !opt(a[7], &Bk) || !opt(a[8], &Bv) || !opt(a[12], &lt) ||
      !opt(a[16], &lse) || !opt(a[17], &ws) || !as_double(a[13], &theta) || !as_double(a[14], &scale))
    return none();
  if (!bf16(Q, 4) || !opt_bf16(Bk, 3) || !opt_bf16(Bv, 3) || !alike(K, V) || !alike_opt(Lk, Lv) || !alike_opt(Bk, Bv))
    return none();
  const int64_t batch = Q->size(0), n_tok = Q->size(1), n_q = Q->size(2), d = Q->size(3);
  lrsa_dims dm{};
  int64_t same;
  const Tensor *lr = Lk ? Lk : Lv, *bt = Bk ? Bk : Bv;
  if (!pool(K, batch, 4, &dm.kv_req_stride) || !pool(V, batch, 4, &same) || !pool(lr, batch, 3, &dm.l_req_stride) ||
      !pool(Lv, batch, 3, &same) || !req_stride(bt, batch, &dm.b_req_stride))
    return none();
  const int64_t kd = K->dim(), n_blk = K->size(kd - 4), blk = K->size(kd - 3), n_kv = K->size(kd - 2);
  const int64_t rank = lr ? lr->size(lr->dim() - 1) : 0, n_lr = lr ? lr->size(lr->dim() - 3) : 0;
  if (K->size(kd - 1) != d || (lr && lr->size(lr->dim() - 2) != blk) ||
      (bt && (bt->size(1) != rank || bt->size(2) != n_kv * d)))
    return none();
  auto table = [&](const Tensor* t) { return i32(t) && t->dim() == 2 && t->size(0) == batch && t->is_contiguous(); };
  if (!table(kt) || (lt && (!table(lt) || lt->size(1) != kt->size(1)))) return none();
  const int64_t mb = kt->size(1);
  if (!fits({batch, n_tok, n_q, n_kv, d, rank, n_blk, blk, n_lr, mb})) return none();
  if (!i32(pos) || !i32(kvl) || pos->dim() != 2 || pos->size(0) != batch || pos->size(1) != n_tok || !pos->is_contiguous() ||
      kvl->dim() != 1 || kvl->size(0) != batch)
    return none();
  dm.batch = (int32_t)batch;
  dm.n_tok = (int32_t)n_tok;
  dm.n_q_heads = (int32_t)n_q;
  dm.n_kv_heads = (int32_t)n_kv;
  dm.head_dim = (int32_t)d;
  dm.rank = (int32_t)rank;
  dm.s_cap = mb * blk;
  dm.softmax_scale = (float)scale;
  dm.rope_theta = theta;
  lrsa_paging pg{};
  pg.kv_block_table = i32p(kt);
  pg.lr_block_table = i32p(lt);
  pg.block_size = (int32_t)blk;
  pg.max_blocks = (int32_t)mb;
  pg.n_kv_blocks = (int32_t)n_blk;
  pg.n_lr_blocks = (int32_t)n_lr;
  const size_t need = reinterpret_cast<size_t (*)(const lrsa_dims*)>(size_fn)(&dm);
  if (need > 0 && (ws == nullptr || nbytes(ws) < need)) return need_bytes(need);
  void* wp = ws == nullptr ? nullptr : ws->data_ptr();
  const size_t wb = ws == nullptr ? 0 : nbytes(ws);
  const uint16_t *q = u16(Q), *k = u16(K), *v = u16(V), *lk = u16(Lk), *lv = u16(Lv), *bk = u16(Bk), *bv = u16(Bv);
  const int32_t *pp = i32p(pos), *kp = i32p(kvl);
  uint16_t* o = u16m(O);
  float* lp = lse == nullptr ? nullptr : static_cast<float*>(lse->data_ptr());
  prc_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = reinterpret_cast<decltype(&lr_shared_attention_paged)>(fn)(&dm, &pg, q, k, v, lk, lv, bk, bv, pp, kp, o, lp, wp, wb, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong((long)st);
}

// project(fn, X, W, A, n_kv, head_dim, n_proj, n_agents, rank, K, V, L, theta,
//         tok_offset, stream); W, K and V None: precompute_lr_cache.
PyObject* project(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 15) return none();
  void *fn, *stream;
  const Tensor *X = tensor(a[1]), *A = tensor(a[3]), *L = tensor(a[11]), *W, *K, *V;
  int32_t n_kv, d, n_proj, n_agents, rank;
  int64_t off;
  double theta;
  if (!as_ptr(a[0], &fn) || !as_ptr(a[14], &stream) || !X || !A || !L || !opt(a[2], &W) || !opt(a[9], &K) || !opt(a[10], &V) ||
      !as_i32(a[4], &n_kv) || !as_i32(a[5], &d) || !as_i32(a[6], &n_proj) || !as_i32(a[7], &n_agents) || !as_i32(a[8], &rank) ||
      !as_double(a[12], &theta) || !as_int(a[13], &off))
    return none();
  const bool lr_only = W == nullptr;
  if ((K == nullptr) != lr_only || (V == nullptr) != lr_only) return none();
  if (!bf16(X, 2) || !bf16(A, 2) || !bf16(L, 4) || !A->is_contiguous() || !L->is_contiguous()) return none();
  const int64_t T = X->size(0), d_in = X->size(1), cols = (int64_t)n_proj * n_agents * rank, s_cap = L->size(2);
  if (cols <= 0 || A->size(0) != d_in || A->size(1) != cols || L->size(0) != n_proj || L->size(1) != n_agents || L->size(3) != rank)
    return none();
  const uint16_t *x = u16(X), *w = u16(W), *ap = u16(A);
  uint16_t *k = u16m(K), *v = u16m(V), *l = u16m(L);
  const int64_t ldx = X->stride(0);
  prc_status st;
  if (lr_only) {
    Py_BEGIN_ALLOW_THREADS;
    st = reinterpret_cast<decltype(&precompute_lr_cache)>(fn)(x, T, d_in, ldx, ap, n_proj, n_agents, rank, l, s_cap, off, stream);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong((long)st);
  }
  if (!bf16(W, 2) || !bf16(K, 3) || !bf16(V, 3) || !W->is_contiguous() || !K->is_contiguous() || !V->is_contiguous() ||
      K->size(0) != s_cap || K->size(1) != n_kv || K->size(2) != d || V->sizes() != K->sizes() || W->size(0) != d_in ||
      W->size(1) != 2 * (int64_t)n_kv * d)
    return none();
  Py_BEGIN_ALLOW_THREADS;
  st = reinterpret_cast<decltype(&project_kv_and_lr_cache)>(fn)(x, T, d_in, ldx, w, n_kv, d, ap, n_proj, n_agents, rank, theta, k,
                                                               v, l, s_cap, off, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong((long)st);
}

// project_paged(fn, X, W, A, n_kv, head_dim, n_proj, n_agents, rank, K, V, L,
//               table, theta, tok_offset, stream), all pools given.
PyObject* project_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 16) return none();
  void *fn, *stream;
  const Tensor *X = tensor(a[1]), *W = tensor(a[2]), *A = tensor(a[3]), *K = tensor(a[9]), *V = tensor(a[10]);
  const Tensor *L = tensor(a[11]), *tb = tensor(a[12]);
  int32_t n_kv, d, n_proj, n_agents, rank;
  int64_t off;
  double theta;
  if (!as_ptr(a[0], &fn) || !as_ptr(a[15], &stream) || !X || !W || !A || !K || !V || !L || !tb || !as_i32(a[4], &n_kv) ||
      !as_i32(a[5], &d) || !as_i32(a[6], &n_proj) || !as_i32(a[7], &n_agents) || !as_i32(a[8], &rank) ||
      !as_double(a[13], &theta) || !as_int(a[14], &off))
    return none();
  if (!bf16(X, 2) || !bf16(W, 2) || !bf16(A, 2) || !bf16(K, 4) || !bf16(V, 4) || !bf16(L, 5) || !W->is_contiguous() ||
      !A->is_contiguous() || !K->is_contiguous() || !V->is_contiguous() || !L->is_contiguous() || !i32(tb) || tb->dim() != 1 ||
      !tb->is_contiguous())
    return none();
  const int64_t nb = K->size(0), blk = K->size(1), mb = tb->size(0), cols = (int64_t)n_proj * n_agents * rank;
  if (n_kv <= 0 || cols <= 0 || K->size(2) != n_kv || K->size(3) != d || V->sizes() != K->sizes() || L->size(0) != n_proj ||
      L->size(1) != n_agents || L->size(2) != nb || L->size(3) != blk || L->size(4) != rank || !fits({nb, blk, mb}) ||
      W->size(0) != X->size(1) || W->size(1) != 2 * (int64_t)n_kv * d || A->size(0) != X->size(1) || A->size(1) != cols)
    return none();
  const uint16_t *x = u16(X), *w = u16(W), *ap = u16(A);
  uint16_t *k = u16m(K), *v = u16m(V), *l = u16m(L);
  const int32_t* tp = i32p(tb);
  const int64_t T = X->size(0), d_in = X->size(1), ldx = X->stride(0);
  prc_status st;
  Py_BEGIN_ALLOW_THREADS;
  st = reinterpret_cast<decltype(&project_kv_and_lr_cache_paged)>(fn)(x, T, d_in, ldx, w, n_kv, d, ap, n_proj, n_agents, rank,
                                                                     theta, k, v, l, tp, (int32_t)blk, (int32_t)mb,
                                                                     (int32_t)nb, off, stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong((long)st);
}

// A tensor can refuse what is asked of it by throwing (a nested one has no
// sizes or strides), and nothing may throw through a C entry: such a call is
// left to Python like any other that is not plain.  (The ABI calls themselves
// throw nothing, so the interpreter lock is held here.)
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  try {
    return F(self, a, n);
  } catch (...) {
    return none();
  }
}
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<F>)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {
    method<attention>("attention"),
    method<paged>("paged"),
    method<project>("project"),
    method<project_paged>("project_paged"),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
