// Native half of the Python binding: the calls that a loop over chunks makes, from tensors to the C ABI.  A call of the
// library costs 10 to 25 us of host time in kernel launches; marshalled through ctypes it took another 6 us and more
// (every pointer an object, every shape and stride tuple built and compared in Python), which short calls felt.
// Every function returns the library's status, or -1 if a tensor does not fit the descriptor -- the Python wrapper
// then says which, or takes the call itself --, or -2 if the page lists have to be copied first.  So it does where torch throws (strides of a 0-dim or sparse tensor, the
// address of a tensor without storage): no exception leaves this file.  The interpreter lock is released during the
// call of the library.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/oomb.h"

namespace {

PyObject* g_raw_stream = nullptr;   // torch._C._cuda_getCurrentRawStream(device index)

struct Desc {
  Py_buffer view{};
  oomb_attn_desc* d = nullptr;
  explicit Desc(PyObject* o) {
    if (PyObject_GetBuffer(o, &view, PyBUF_WRITABLE) == 0) {
      if (view.len == (Py_ssize_t)sizeof(oomb_attn_desc)) d = (oomb_attn_desc*)view.buf;
    } else {
      PyErr_Clear();
    }
  }
  ~Desc() { if (view.obj) PyBuffer_Release(&view); }
};

// one argument: a tensor, None (nullptr), or neither (bad)
const at::Tensor* tensor(PyObject* o, bool& bad) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) { bad = true; return nullptr; }
  return &THPVariable_Unpack(o);
}
void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
size_t bytes(const at::Tensor* t) { return t ? t->numel() * t->element_size() : 0; }
at::ScalarType type_of(int32_t dt) { return dt == OOMB_BF16 ? at::kBFloat16 : at::kFloat; }

bool like(const at::Tensor* t, const at::Tensor& ref, at::ScalarType dt) {
  return !t || (t->scalar_type() == dt && t->sizes() == ref.sizes() && t->strides() == ref.strides());
}
// q and the pools against the descriptor, as the Python wrapper checks them
bool family(const oomb_attn_desc& d, const at::Tensor* q, const at::Tensor* k, const at::Tensor* lse) {
  if (!q || !k || q->dim() != 3 || k->dim() != 4) return false;
  if (lse && (lse->scalar_type() != at::kFloat || lse->dim() != 2 || lse->size(0) != d.n_q_heads || lse->size(1) != d.chunk_len || !lse->is_contiguous()))
    return false;
  return q->stride(0) == d.q_tok_stride && q->stride(1) == d.q_head_stride && q->scalar_type() == type_of(d.dtype) &&
         k->stride(0) == d.pool_page_stride && k->stride(1) == d.pool_head_stride && k->stride(2) == d.pool_tok_stride;
}
bool stream_of(const at::Tensor* t, void** st) {
  if (!t || !t->is_cuda()) return false;
  PyObject* idx = PyLong_FromLong(t->get_device());
  PyObject* r = idx ? PyObject_CallOneArg(g_raw_stream, idx) : nullptr;
  Py_XDECREF(idx);
  if (!r) { PyErr_Clear(); return false; }
  *st = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  return true;
}
PyObject* status(int s) { return PyLong_FromLong(s); }
struct Unlocked {   // (taken back on an exception too)
  PyThreadState* s = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(s); }
};
#define OOMB_CALL(expr) \
  oomb_status s_; \
  { Unlocked u_; s_ = (expr); } \
  return status((int)s_)

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)> PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  try {
    return F(self, a, nargs);
  } catch (const std::exception&) {
    PyErr_Clear();
    return status(-1);
  }
}

// 0, -1 (does not fit), or -2: lists that are a view whose last row ends with the memory before its stride does.  The kernels
// read whole rows of min(stride, n) entries before they know how many are valid.
int list_args(const oomb_attn_desc& d, const at::Tensor* sel, const at::Tensor* cnt, bool qp, int32_t* stride) {
  if (!qp) {
    *stride = sel ? (int32_t)sel->stride(0) : 0;
    if (!sel || sel->dim() != 2 || sel->size(0) != d.n_kv_heads || sel->size(1) >= sel->stride(0) || d.page_size <= 0) return 0;
    const int64_t n = d.ctx_len / d.page_size, row = sel->stride(0) < n ? sel->stride(0) : n;
    return (size_t)(sel->storage_offset() + (d.n_kv_heads - 1) * sel->stride(0) + row) * sel->element_size() > sel->storage().nbytes() ? -2 : 0;
  }
  const int64_t m = d.page_size > 0 ? d.chunk_len / d.page_size : 0;
  if (!sel || !cnt || sel->dim() != 3 || sel->size(0) != d.n_kv_heads || sel->size(1) != m || !sel->is_contiguous() || cnt->dim() != 2 ||
      cnt->size(0) != d.n_kv_heads || cnt->size(1) != m || !cnt->is_contiguous())
    return -1;
  *stride = (int32_t)sel->size(2);
  return 0;
}

#define OOMB_ARGS(n) if (nargs != (n)) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; } \
  bool bad = false; Desc desc(a[0]); void* st = nullptr; if (!desc.d) return status(-1); const oomb_attn_desc& d = *desc.d; (void)d; (void)bad; (void)st

// make_desc(desc, q, k_pool, ctx_len, sm_scale, grad_is_bf16)
PyObject* make_desc(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  OOMB_ARGS(6);
  const at::Tensor *q = tensor(a[1], bad), *k = tensor(a[2], bad);
  if (bad || !q || !k || q->dim() != 3 || k->dim() != 4 || q->stride(2) != 1 || k->stride(3) != 1 || q->size(2) != k->size(3)) return status(-1);
  if (q->scalar_type() != at::kFloat && q->scalar_type() != at::kBFloat16) return status(-1);
  const long long ctx = PyLong_AsLongLong(a[3]);
  const double scale = PyFloat_AsDouble(a[4]);
  if (PyErr_Occurred()) { PyErr_Clear(); return status(-1); }
  oomb_attn_desc& w = *desc.d;
  w.n_q_heads = (int32_t)q->size(1); w.n_kv_heads = (int32_t)k->size(1); w.head_dim = (int32_t)q->size(2); w.page_size = (int32_t)k->size(2);
  w.chunk_len = (int32_t)q->size(0); w.dtype = q->scalar_type() == at::kBFloat16 ? OOMB_BF16 : OOMB_F32;
  w.grad_dtype = a[5] == Py_True ? OOMB_BF16 : OOMB_F32; w.sm_scale = (float)scale; w.ctx_len = ctx;
  w.pool_page_stride = k->stride(0); w.pool_head_stride = k->stride(1); w.pool_tok_stride = k->stride(2);
  w.q_tok_stride = q->stride(0); w.q_head_stride = q->stride(1); w.num_phys_pages = k->size(0);
  return status(0);
}

// score_topk(desc, q, k_pool, page_table, top_k, sel_pages, sel_count, scores_out, workspace)
PyObject* score_topk(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  OOMB_ARGS(9);
  const at::Tensor *q = tensor(a[1], bad), *k = tensor(a[2], bad), *pt = tensor(a[3], bad), *sel = tensor(a[5], bad), *cnt = tensor(a[6], bad),
                   *sc = tensor(a[7], bad), *ws = tensor(a[8], bad);
  const long top_k = PyLong_AsLong(a[4]);
  if (PyErr_Occurred()) { PyErr_Clear(); return status(-1); }
  if (bad || !stream_of(q, &st)) return status(-1);
  OOMB_CALL(oomb_page_score_topk(&d, ptr(q), ptr(k), (const int32_t*)ptr(pt), (int32_t)top_k, (int32_t*)ptr(sel), (int32_t*)ptr(cnt), (float*)ptr(sc), ptr(ws),
                                 bytes(ws), st));
}

// score_topk_cached / vote_topk(desc, q, kbar_cache, top_k, sel_pages, sel_count, out, workspace)
template <oomb_status (*F)(const oomb_attn_desc*, const void*, const float*, int32_t, int32_t*, int32_t*, float*, void*, size_t, void*)>
PyObject* from_means(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  OOMB_ARGS(8);
  const at::Tensor *q = tensor(a[1], bad), *kb = tensor(a[2], bad), *sel = tensor(a[4], bad), *cnt = tensor(a[5], bad), *out = tensor(a[6], bad),
                   *ws = tensor(a[7], bad);
  const long top_k = PyLong_AsLong(a[3]);
  if (PyErr_Occurred()) { PyErr_Clear(); return status(-1); }
  if (bad || !stream_of(q, &st)) return status(-1);
  OOMB_CALL(F(&d, ptr(q), (const float*)ptr(kb), (int32_t)top_k, (int32_t*)ptr(sel), (int32_t*)ptr(cnt), (float*)ptr(out), ptr(ws), bytes(ws), st));
}

// attn_fwd / attn_fwd_qp(desc, q, k_pool, v_pool, page_table, sel_pages, sel_count, o, lse, workspace)
template <bool QP> PyObject* attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  OOMB_ARGS(10);
  const at::Tensor *q = tensor(a[1], bad), *k = tensor(a[2], bad), *v = tensor(a[3], bad), *pt = tensor(a[4], bad), *sel = tensor(a[5], bad),
                   *cnt = tensor(a[6], bad), *o = tensor(a[7], bad), *lse = tensor(a[8], bad), *ws = tensor(a[9], bad);
  int32_t stride = 0;
  if (bad || !family(d, q, k, lse) || !like(o, *q, q->scalar_type()) || !like(v, *k, k->scalar_type())) return status(-1);
  if (const int s = list_args(d, sel, cnt, QP, &stride); s != 0) return status(s);
  if (!stream_of(q, &st)) return status(-1);
  OOMB_CALL((QP ? oomb_paged_attn_fwd_qp : oomb_paged_attn_fwd)(&d, ptr(q), ptr(k), ptr(v), (const int32_t*)ptr(pt), (const int32_t*)ptr(sel),
                                                                (const int32_t*)ptr(cnt), stride, ptr(o), (float*)ptr(lse), ptr(ws), bytes(ws), st));
}

// attn_bwd / attn_bwd_qp(desc, q, k_pool, v_pool, page_table, sel_pages, sel_count, o, lse, d_o, d_q, dk_pool, dv_pool, workspace)
template <bool QP> PyObject* attn_bwd(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  OOMB_ARGS(14);
  const at::Tensor *q = tensor(a[1], bad), *k = tensor(a[2], bad), *v = tensor(a[3], bad), *pt = tensor(a[4], bad), *sel = tensor(a[5], bad),
                   *cnt = tensor(a[6], bad), *o = tensor(a[7], bad), *lse = tensor(a[8], bad), *d_o = tensor(a[9], bad), *d_q = tensor(a[10], bad),
                   *dk = tensor(a[11], bad), *dv = tensor(a[12], bad), *ws = tensor(a[13], bad);
  int32_t stride = 0;
  if (bad || !family(d, q, k, lse)) return status(-1);
  const at::ScalarType t = q->scalar_type(), gt = type_of(d.grad_dtype);
  if (!like(o, *q, t) || !like(d_o, *q, t) || !like(d_q, *q, t) || !like(v, *k, k->scalar_type()) || !like(dk, *k, gt) || !like(dv, *k, gt)) return status(-1);
  if (const int s = list_args(d, sel, cnt, QP, &stride); s != 0) return status(s);
  if (!stream_of(q, &st)) return status(-1);
  OOMB_CALL((QP ? oomb_paged_attn_bwd_qp : oomb_paged_attn_bwd)(&d, ptr(q), ptr(k), ptr(v), (const int32_t*)ptr(pt), (const int32_t*)ptr(sel),
                                                                (const int32_t*)ptr(cnt), stride, ptr(o), (const float*)ptr(lse), ptr(d_o), ptr(d_q), ptr(dk),
                                                                ptr(dv), ptr(ws), bytes(ws), st));
}

// kv_append(desc, k_chunk, v_chunk, page_table, k_pool, v_pool, kbar_cache)
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  OOMB_ARGS(7);
  const at::Tensor *kc = tensor(a[1], bad), *vc = tensor(a[2], bad), *pt = tensor(a[3], bad), *k = tensor(a[4], bad), *v = tensor(a[5], bad),
                   *kb = tensor(a[6], bad);
  if (bad || !kc || !vc || !k || !kc->is_contiguous() || !vc->is_contiguous() || kc->sizes() != vc->sizes() || kc->scalar_type() != k->scalar_type() ||
      vc->scalar_type() != k->scalar_type() || !like(v, *k, k->scalar_type()) || !stream_of(k, &st))
    return status(-1);
  OOMB_CALL(oomb_kv_append(&d, ptr(kc), ptr(vc), (const int32_t*)ptr(pt), ptr(k), ptr(v), (float*)ptr(kb), st));
}

// local_page_list(desc, window_pages, sel_pages, sel_count)
PyObject* local_page_list(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  OOMB_ARGS(4);
  const long window = PyLong_AsLong(a[1]);
  if (PyErr_Occurred()) { PyErr_Clear(); return status(-1); }
  const at::Tensor *sel = tensor(a[2], bad), *cnt = tensor(a[3], bad);
  if (bad || !stream_of(sel, &st)) return status(-1);
  OOMB_CALL(oomb_local_page_list(&d, (int32_t)window, (int32_t*)ptr(sel), (int32_t*)ptr(cnt), st));
}

#define OOMB_METHOD(name, fn) {name, (PyCFunction)(void (*)(void))(guarded<fn>), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    OOMB_METHOD("make_desc", make_desc),
    OOMB_METHOD("score_topk", score_topk),
    OOMB_METHOD("score_topk_cached", from_means<oomb_page_score_topk_cached>),
    OOMB_METHOD("vote_topk", from_means<oomb_page_vote_topk>),
    OOMB_METHOD("attn_fwd", attn_fwd<false>),
    OOMB_METHOD("attn_fwd_qp", attn_fwd<true>),
    OOMB_METHOD("attn_bwd", attn_bwd<false>),
    OOMB_METHOD("attn_bwd_qp", attn_bwd<true>),
    OOMB_METHOD("kv_append", kv_append),
    OOMB_METHOD("local_page_list", local_page_list),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  PyObject* c = PyImport_ImportModule("torch._C");
  if (!c) return nullptr;
  g_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
  Py_DECREF(c);
  return g_raw_stream ? PyModule_Create(&module) : nullptr;
}
