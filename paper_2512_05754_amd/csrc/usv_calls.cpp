// Marshalling of the calls that a small step is made of, as a CPython extension: the three stages and the work order on tensors that
// are all there already.  A call of a few microseconds of kernels is bound by its host side, and reading a tensor's shape, type and
// address costs Python about 0.4 us a tensor and the foreign-function call another 1.5 us (three stages on 1024 tokens, fp32: 21.5 -> 17.2 us with the kernels of 17 us that they launch; the first pass on new inputs 57 -> 41).
//
// Every function takes what the binding's function of that name was given, checks what it checks, calls the library and returns its
// status; or it returns None, having done nothing, for whatever it does not know: the binding then goes its own way, which also says
// what is wrong with an argument.  No tensor is kept, allocated or changed, and no exception of torch's leaves a function.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "usv.h"

namespace {

struct Table {
  decltype(&usv_block_scores) block_scores;
  decltype(&usv_select_topk_ex) select_topk_ex;
  decltype(&usv_attn_work_order) attn_work_order;
  decltype(&usv_block_sparse_attn) block_sparse_attn;
  decltype(&usv_block_sparse_attn_ordered) block_sparse_attn_ordered;
} table;  // of the library the binding has loaded

// A plain tensor in GPU memory (no subclass, which may stand for something else; no wrapper without storage of its own).
bool plain(PyObject* o, const at::Tensor** t) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& x = THPVariable_Unpack(o);
  if (!x.defined() || !x.is_cuda() || x.layout() != at::kStrided || !x.has_storage() || !x.is_contiguous()) return false;
  *t = &x;
  return true;
}
bool plain(PyObject* o, const at::Tensor** t, at::ScalarType type) { return plain(o, t) && (*t)->scalar_type() == type; }

bool whole(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long x = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}

bool fits(int64_t x) { return x >= 0 && x <= INT32_MAX; }

// Shape of Q, K or V [B, Hh, N, d]
bool shape_of(const at::Tensor& x, PyObject* seq_valid, usv_shape* s) {
  if (x.dim() != 4) return false;
  const auto n = x.sizes();
  for (int64_t e : n)
    if (!fits(e)) return false;
  if (x.scalar_type() == at::kBFloat16) s->dtype = USV_BF16;
  else if (x.scalar_type() == at::kFloat) s->dtype = USV_F32;
  else return false;
  s->batch = (int32_t)n[0], s->heads = (int32_t)n[1], s->seq_len = (int32_t)n[2], s->head_dim = (int32_t)n[3];
  s->block = 64;
  s->seq_valid = s->seq_len;
  return seq_valid == Py_None || whole(seq_valid, &s->seq_valid);
}
// ... of tensors that know the blocks only
bool shape_of_blocks(int64_t B, int64_t Hh, int64_t nb, PyObject* seq_valid, usv_shape* s) {
  if (!fits(B) || !fits(Hh) || !fits(nb * 64)) return false;
  *s = usv_shape{(int32_t)B, (int32_t)Hh, (int32_t)(nb * 64), (int32_t)(nb * 64), 0, 64, USV_F32};
  return seq_valid == Py_None || whole(seq_valid, &s->seq_valid);
}

bool alike(const at::Tensor& a, const at::Tensor& b) { return a.sizes() == b.sizes() && a.scalar_type() == b.scalar_type(); }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

template <typename F>
PyObject* call(F f) {  // the launch itself without the interpreter lock, as the foreign-function call does it
  int32_t status;
  Py_BEGIN_ALLOW_THREADS
  status = (int32_t)f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    if (PyObject* r = F(a, n)) return r;
  } catch (...) {  // (nothing has been called by then: the library throws nothing)
  }
  PyErr_Clear();
  Py_RETURN_NONE;
}

// (q, k, seq_valid, out, workspace)
PyObject* block_scores(PyObject* const* a, Py_ssize_t n) {
  const at::Tensor *q, *k, *out, *ws;
  usv_shape s;
  if (n != 5 || !table.block_scores || !plain(a[0], &q) || !plain(a[1], &k) || !plain(a[3], &out, at::kFloat) || !plain(a[4], &ws)) return nullptr;
  if (!shape_of(*q, a[2], &s) || !alike(*q, *k)) return nullptr;
  const void *qp = q->data_ptr(), *kp = k->data_ptr();
  float* op = static_cast<float*>(out->data_ptr());
  void *wp = ws->data_ptr(), *st = stream();
  const size_t bytes = ws->nbytes();
  return call([&] { return table.block_scores(qp, kp, &s, op, wp, bytes, st); });
}

// (scores, k, seq_valid, budgets, kmax, idx, cnt, force_local)
PyObject* select_topk(PyObject* const* a, Py_ssize_t n) {
  const at::Tensor *scores, *budgets = nullptr, *idx, *cnt;
  usv_shape s;
  int32_t k, kmax;
  if (n != 8 || !table.select_topk_ex || !plain(a[0], &scores, at::kFloat) || !whole(a[1], &k) || !plain(a[5], &idx, at::kInt) ||
      !plain(a[6], &cnt, at::kInt))
    return nullptr;
  if (a[3] != Py_None && !plain(a[3], &budgets, at::kInt)) return nullptr;
  if (a[4] == Py_None) kmax = k;
  else if (!whole(a[4], &kmax)) return nullptr;
  if (a[7] != Py_False && a[7] != Py_True) return nullptr;
  if (scores->dim() != 4 || scores->size(2) != scores->size(3)) return nullptr;
  if (!shape_of_blocks(scores->size(0), scores->size(1), scores->size(2), a[2], &s)) return nullptr;
  const uint32_t flags = a[7] == Py_True ? USV_TOPK_FORCE_LOCAL : 0u;
  const float* sp = static_cast<const float*>(scores->data_ptr());
  const int32_t* bp = budgets ? static_cast<const int32_t*>(budgets->data_ptr()) : nullptr;
  int32_t *ip = static_cast<int32_t*>(idx->data_ptr()), *cp = static_cast<int32_t*>(cnt->data_ptr());
  void* st = stream();
  return call([&] { return table.select_topk_ex(sp, &s, k, bp, kmax, flags, ip, cp, st); });
}

// (cnt, kmax, idx, out)
PyObject* attn_work_order(PyObject* const* a, Py_ssize_t n) {
  const at::Tensor *cnt, *idx = nullptr, *out;
  usv_shape s;
  int32_t kmax;
  if (n != 4 || !table.attn_work_order || !plain(a[0], &cnt, at::kInt) || !whole(a[1], &kmax) || !plain(a[3], &out, at::kInt)) return nullptr;
  if (cnt->dim() != 3 || !shape_of_blocks(cnt->size(0), cnt->size(1), cnt->size(2), Py_None, &s)) return nullptr;
  if (a[2] != Py_None) {
    if (!plain(a[2], &idx, at::kInt) || idx->dim() != 4 || idx->sizes().slice(0, 3) != cnt->sizes() || idx->size(3) != kmax) return nullptr;
  }
  const int32_t *ip = idx ? static_cast<const int32_t*>(idx->data_ptr()) : nullptr, *cp = static_cast<const int32_t*>(cnt->data_ptr());
  int32_t* op = static_cast<int32_t*>(out->data_ptr());
  void* st = stream();
  return call([&] { return table.attn_work_order(ip, cp, &s, kmax, op, st); });
}

// (q, k, v, idx, cnt, seq_valid, scale, out, lse, work_order)
PyObject* block_sparse_attn(PyObject* const* a, Py_ssize_t n) {
  const at::Tensor *q, *k, *v, *idx, *cnt, *out, *lse = nullptr, *wo = nullptr;
  usv_shape s;
  if (n != 10 || !table.block_sparse_attn || !plain(a[0], &q) || !plain(a[1], &k) || !plain(a[2], &v) || !plain(a[3], &idx, at::kInt) ||
      !plain(a[4], &cnt, at::kInt) || !PyFloat_CheckExact(a[6]) || !plain(a[7], &out))
    return nullptr;
  if (!shape_of(*q, a[5], &s) || !alike(*q, *k) || !alike(*q, *v)) return nullptr;
  const int64_t rows[3] = {s.batch, s.heads, s.seq_len / 64};
  const at::IntArrayRef want(rows, 3);
  if (idx->dim() != 4 || idx->sizes().slice(0, 3) != want || cnt->sizes() != want || !fits(idx->size(3))) return nullptr;
  if (out->sizes() != q->sizes()) return nullptr;
  int32_t odt;
  if (out->scalar_type() == at::kFloat) odt = USV_F32;
  else if (out->scalar_type() == at::kBFloat16) odt = USV_BF16;
  else return nullptr;
  if (a[8] != Py_None && !plain(a[8], &lse, at::kFloat)) return nullptr;
  if (a[9] != Py_None && (!plain(a[9], &wo, at::kInt) || wo->sizes() != want)) return nullptr;
  const int32_t kmax = (int32_t)idx->size(3);
  const float scale = (float)PyFloat_AS_DOUBLE(a[6]);
  const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
  const int32_t *ip = static_cast<const int32_t*>(idx->data_ptr()), *cp = static_cast<const int32_t*>(cnt->data_ptr());
  void *op = out->data_ptr(), *st = stream();
  float* lp = lse ? static_cast<float*>(lse->data_ptr()) : nullptr;
  if (!wo) return call([&] { return table.block_sparse_attn(qp, kp, vp, &s, ip, cp, kmax, scale, odt, op, lp, st); });
  const int32_t* wp = static_cast<const int32_t*>(wo->data_ptr());
  return call([&] { return table.block_sparse_attn_ordered(qp, kp, vp, &s, ip, cp, kmax, wp, scale, odt, op, lp, st); });
}

// (the addresses of the five functions above, in the table's order)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* p[5];
  if (n != 5) return PyErr_Format(PyExc_TypeError, "five addresses");
  for (int i = 0; i < 5; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  table = Table{reinterpret_cast<decltype(table.block_scores)>(p[0]), reinterpret_cast<decltype(table.select_topk_ex)>(p[1]),
                reinterpret_cast<decltype(table.attn_work_order)>(p[2]), reinterpret_cast<decltype(table.block_sparse_attn)>(p[3]),
                reinterpret_cast<decltype(table.block_sparse_attn_ordered)>(p[4])};
  Py_RETURN_NONE;
}

#define USV_METHOD(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {USV_METHOD("block_scores", guarded<block_scores>), USV_METHOD("select_topk", guarded<select_topk>),
                         USV_METHOD("attn_work_order", guarded<attn_work_order>),
                         USV_METHOD("block_sparse_attn", guarded<block_sparse_attn>), USV_METHOD("bind", bind),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
