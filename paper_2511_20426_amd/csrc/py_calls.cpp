// The calls that a program makes at every layer and step, from Python objects straight to the C ABI: what runner.py's methods check
// and pass on, without a Python object for every look at a tensor.  Small calls are bound by the host (a launch alone takes 2.6
// us).  Host time of a call, through ctypes and here: a linear map 5.2 and 3.3 us, a cache write 7.1 and 3.9, a rotation 5.1 and
// 3.8, attention on rotated queries 5.1 and 3.5, on raw ones 8.6 and 7.2 (its launches take most of that); the smallest
// rollout step in fp32 18 to 20 -> 15.1 us, a linear map of 257 x 768 x 1024 5.76 -> 5.53.
//
// A function here takes a call only if everything is as it should be (plain tensors, exact integers, lists or tuples, shapes and
// strides that fit); otherwise it returns None and has done nothing, and the Python code does what it does: checks one by one and
// raises.  It returns the result, or the library's code where that is not CA_OK.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include "cascade_attn.h"

namespace {

// the library's entry points, as the module that loaded it hands them over
decltype(&kv_cache_append_batch) append_batch_fn = nullptr;
decltype(&rope3d_apply_strided) rope_fn = nullptr;
decltype(&cascade_attn_forward) forward_fn = nullptr;
decltype(&cascade_attn_forward_share) share_fn = nullptr;
decltype(&cascade_attn_forward_rope) forward_rope_fn = nullptr;
decltype(&layer_qkv_publish) publish_fn = nullptr;
decltype(&layer_linear_bf16) linear_fn = nullptr;

constexpr int kMaxBlocks = 64;                    // of a call taken here

PyObject* not_taken() { Py_RETURN_NONE; }

// a tensor that is nothing but one: no subclass, no wrapper without memory of its own
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckTypeExact(Py_TYPE(o))) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.defined() && t.has_storage() && t.layout() == at::kStrided ? &t : nullptr;
}

bool whole(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0;
}
bool whole32(PyObject* o, int32_t* v) {
  int64_t x;
  if (!whole(o, &x) || x != int32_t(x)) return false;
  *v = int32_t(x);
  return true;
}

// items of a list or tuple, or -1
Py_ssize_t items(PyObject* o, PyObject*** first) {
  if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return -1;
  *first = PySequence_Fast_ITEMS(o);
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
  return n <= kMaxBlocks ? n : -1;
}

template <typename T, bool (*read)(PyObject*, T*)>
int all(PyObject* o, T* out) {
  PyObject** at;
  const Py_ssize_t n = items(o, &at);
  for (Py_ssize_t i = 0; i < n; ++i)
    if (!read(at[i], out + i)) return -1;
  return int(n);
}

struct Pool {                                     // a CascadePool: its context, and what its tensors have to look like
  ca_ctx* ctx;
  int64_t heads, head_dim, block_tokens, f32, device;
  at::ScalarType dtype() const { return f32 ? at::kFloat : at::kBFloat16; }
  void* stream() const {
    return c10::hip::getCurrentHIPStream(device < 0 ? c10::hip::current_device() : c10::DeviceIndex(device)).stream();
  }
};

bool pool_of(PyObject* handle, PyObject* shape, Pool* p) {
  int64_t h;
  if (!whole(handle, &h) || h == 0 || !PyTuple_CheckExact(shape) || PyTuple_GET_SIZE(shape) != 5) return false;
  p->ctx = reinterpret_cast<ca_ctx*>(h);
  int64_t* const to[] = {&p->heads, &p->head_dim, &p->block_tokens, &p->f32, &p->device};
  for (int i = 0; i < 5; ++i)
    if (!whole(PyTuple_GET_ITEM(shape, i), to[i])) return false;
  return true;
}

// [n, heads, head_dim] with any token and head strides
bool fits(const Pool& p, const at::Tensor* t) {
  return t && t->is_cuda() && t->scalar_type() == p.dtype() && t->dim() == 3 && t->stride(2) == 1 && t->size(1) == p.heads && t->size(2) == p.head_dim;
}

// memory of the device that `like` is on (pinned host memory, which kernels reach too, is left to the Python code)
bool beside(const at::Tensor& t, const at::Tensor& like) { return t.is_cuda() && t.device() == like.device(); }

template <typename F>
int32_t released(const F& call) {
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return rc;
}

// None, or a result given by the caller, or a new tensor
struct Result {
  at::Tensor made;
  const at::Tensor* t = nullptr;
  PyObject* given = nullptr;
  bool take(PyObject* o) {
    if (o == Py_None) return true;
    given = o;
    t = plain(o);
    return t != nullptr;
  }
  const at::Tensor& or_empty(at::IntArrayRef sizes, const at::Tensor& like) {
    if (!t) {
      made = at::empty(sizes, like.options());
      t = &made;
    }
    return *t;
  }
  PyObject* give(int32_t rc) {
    if (rc != CA_OK) return PyLong_FromLong(rc);
    if (given) {
      Py_INCREF(given);
      return given;
    }
    return THPVariable_Wrap(made);
  }
};

// Anything that throws (a tensor whose memory cannot be looked at, no memory for a result) is left to the Python code, but for
// what Python code raised in here (a dispatch mode around the allocation), which is the caller's to see.
template <PyObject* (*call)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    return call(a, n);
  } catch (python_error& e) {
    e.restore();
  } catch (...) {
  }
  return PyErr_Occurred() ? nullptr : not_taken();
}

// linear(x, w, out)
PyObject* linear(PyObject* const* a, Py_ssize_t n) {
  if (n != 3) return not_taken();
  const at::Tensor *x = plain(a[0]), *w = plain(a[1]);
  Result r;
  if (!x || !w || !r.take(a[2]) || !x->is_cuda() || !w->is_cuda() || x->scalar_type() != at::kBFloat16 || w->scalar_type() != at::kBFloat16 ||
      x->dim() != 2 || w->dim() != 2 || x->size(1) != w->size(1) || x->stride(1) != 1 || w->stride(1) != 1)
    return not_taken();
  const int64_t m = x->size(0), cols = w->size(0), k = x->size(1);
  if (cols != int32_t(cols) || k != int32_t(k)) return not_taken();
  const at::Tensor& y = r.or_empty({m, cols}, *x);
  if (y.dim() != 2 || y.size(0) != m || y.size(1) != cols || y.stride(1) != 1 || y.scalar_type() != at::kBFloat16 || !beside(y, *x)) return not_taken();
  void* const stream = c10::hip::getCurrentHIPStream(x->device().index()).stream();
  const void *xp = x->data_ptr(), *wp = w->data_ptr();
  void* const yp = y.data_ptr();
  const int64_t ldx = x->stride(0), ldw = w->stride(0), ldy = y.stride(0);
  return r.give(released([&] { return linear_fn(xp, wp, yp, m, int32_t(cols), int32_t(k), ldx, ldw, ldy, stream); }));
}

// append_batch(handle, shape, block_ids, timesteps, epoch, ks, vs) -> slots
PyObject* append_batch(PyObject* const* a, Py_ssize_t n) {
  Pool p;
  int64_t ids[kMaxBlocks];
  int32_t ts[kMaxBlocks], slots[kMaxBlocks], epoch;
  const void *ks[kMaxBlocks], *vs[kMaxBlocks];
  if (n != 7 || !pool_of(a[0], a[1], &p) || !whole32(a[4], &epoch)) return not_taken();
  const int blocks = all<int64_t, whole>(a[2], ids);
  PyObject **k, **v;
  if (blocks < 1 || all<int32_t, whole32>(a[3], ts) != blocks || items(a[5], &k) != blocks || items(a[6], &v) != blocks) return not_taken();
  int64_t tok = 0, head = 0;
  for (int i = 0; i < blocks; ++i) {
    const at::Tensor *kt = plain(k[i]), *vt = plain(v[i]);
    if (!fits(p, kt) || !fits(p, vt) || kt->size(0) != p.block_tokens || vt->size(0) != p.block_tokens) return not_taken();
    if (i == 0) tok = kt->stride(0), head = kt->stride(1);
    if (kt->stride(0) != tok || kt->stride(1) != head || vt->stride(0) != tok || vt->stride(1) != head) return not_taken();
    ks[i] = kt->data_ptr();
    vs[i] = vt->data_ptr();
  }
  void* const stream = p.stream();
  const int32_t rc = released([&] { return append_batch_fn(p.ctx, blocks, ids, ts, epoch, ks, vs, tok, head, stream, slots); });
  if (rc != CA_OK) return PyLong_FromLong(rc);
  PyObject* const out = PyList_New(blocks);
  for (int i = 0; out && i < blocks; ++i) PyList_SET_ITEM(out, i, PyLong_FromLong(slots[i]));
  return out;
}

// rope(handle, shape, x, first_frame, out)
PyObject* rope(PyObject* const* a, Py_ssize_t n) {
  Pool p;
  Result r;
  int64_t first;
  if (n != 5 || !pool_of(a[0], a[1], &p) || !whole(a[3], &first) || !r.take(a[4])) return not_taken();
  const at::Tensor* x = plain(a[2]);
  if (!fits(p, x)) return not_taken();
  const at::Tensor& y = r.or_empty(x->sizes(), *x);
  if (!fits(p, &y) || y.size(0) != x->size(0)) return not_taken();
  void *const stream = p.stream(), *const yp = y.data_ptr();
  const void* const xp = x->data_ptr();
  const int64_t s[] = {x->stride(0), x->stride(1), y.stride(0), y.stride(1)}, rows = x->size(0);
  return r.give(released([&] { return rope_fn(p.ctx, xp, s[0], s[1], yp, s[2], s[3], rows, first, stream); }));
}

// forward(handle, shape, q_rot, inflight, mode, out, share) with share None or (first, count)
PyObject* forward(PyObject* const* a, Py_ssize_t n) {
  Pool p;
  Result r;
  int64_t ids[kMaxBlocks];
  int32_t mode, share[2];
  if (n != 7 || !pool_of(a[0], a[1], &p) || !whole32(a[4], &mode) || !r.take(a[5])) return not_taken();
  const int blocks = all<int64_t, whole>(a[3], ids);
  const bool part = a[6] != Py_None;
  PyObject** of_share;
  if (blocks < 1 || (part && (items(a[6], &of_share) != 2 || !whole32(of_share[0], share) || !whole32(of_share[1], share + 1)))) return not_taken();
  const at::Tensor* q = plain(a[2]);
  if (!fits(p, q) || !q->is_contiguous() || q->size(0) != (part ? share[1] : blocks) * p.block_tokens) return not_taken();
  const at::Tensor& o = r.or_empty(q->sizes(), *q);
  if (!o.is_contiguous() || o.sizes() != q->sizes() || !fits(p, &o) || !beside(o, *q)) return not_taken();
  void *const stream = p.stream(), *const op = o.data_ptr();
  const void* const qp = q->data_ptr();
  return r.give(released([&] {
    return part ? share_fn(p.ctx, qp, ids, blocks, share[0], share[1], mode, op, stream) : forward_fn(p.ctx, qp, ids, blocks, mode, op, stream);
  }));
}

// forward_rope(handle, shape, q, inflight, mode, out)
PyObject* forward_rope(PyObject* const* a, Py_ssize_t n) {
  Pool p;
  Result r;
  int64_t ids[kMaxBlocks];
  int32_t mode;
  if (n != 6 || !pool_of(a[0], a[1], &p) || !whole32(a[4], &mode) || !r.take(a[5])) return not_taken();
  const int blocks = all<int64_t, whole>(a[3], ids);
  const at::Tensor* q = plain(a[2]);
  if (blocks < 1 || !fits(p, q) || q->size(0) != blocks * p.block_tokens) return not_taken();
  const at::Tensor& o = r.or_empty(q->sizes(), *q);
  if (!o.is_contiguous() || o.sizes() != q->sizes() || !fits(p, &o) || !beside(o, *q)) return not_taken();
  void *const stream = p.stream(), *const op = o.data_ptr();
  const void* const qp = q->data_ptr();
  const int64_t tok = q->stride(0), head = q->stride(1);
  return r.give(released([&] { return forward_rope_fn(p.ctx, qp, tok, head, ids, blocks, mode, op, stream); }));
}

// qkv_publish(handle, shape, x, w_qkv, block_ids, timesteps, epoch, q_out)
PyObject* qkv_publish(PyObject* const* a, Py_ssize_t n) {
  Pool p;
  Result r;
  int64_t ids[kMaxBlocks];
  int32_t ts[kMaxBlocks], slots[kMaxBlocks], epoch;
  if (n != 8 || !pool_of(a[0], a[1], &p) || !whole32(a[6], &epoch) || !r.take(a[7])) return not_taken();
  const int blocks = all<int64_t, whole>(a[4], ids);
  const at::Tensor *x = plain(a[2]), *w = plain(a[3]);
  const int64_t rows = blocks * p.block_tokens, width = p.heads * p.head_dim;
  if (blocks < 1 || all<int32_t, whole32>(a[5], ts) != blocks || !x || !w || !x->is_cuda() || x->scalar_type() != at::kBFloat16 || x->dim() != 2 ||
      x->size(0) != rows || x->stride(1) != 1 || x->size(1) != int32_t(x->size(1)) || w->dim() != 2 || w->size(0) != 3 * width ||
      w->size(1) != x->size(1) || w->stride(1) != 1 || w->scalar_type() != at::kBFloat16 || !beside(*w, *x))
    return not_taken();
  const at::Tensor& q = r.or_empty({rows, p.heads, p.head_dim}, *x);
  if (q.dim() != 3 || !q.is_contiguous() || q.size(0) != rows || q.size(1) != p.heads || q.size(2) != p.head_dim || q.scalar_type() != at::kBFloat16 ||
      !beside(q, *x))
    return not_taken();
  void *const stream = p.stream(), *const qp = q.data_ptr();
  const void *const xp = x->data_ptr(), *const wp = w->data_ptr();
  const int64_t ldx = x->stride(0), ldw = w->stride(0);
  const int32_t k = int32_t(x->size(1));
  return r.give(released([&] { return publish_fn(p.ctx, blocks, ids, ts, epoch, xp, ldx, wp, ldw, k, qp, stream, slots); }));
}

// bind(addresses of the seven entry points in the order above)
PyObject* bind(PyObject* const* a, Py_ssize_t n) {
  int64_t f[7];
  if (n != 7) {
    PyErr_SetString(PyExc_TypeError, "seven addresses");
    return nullptr;
  }
  for (int i = 0; i < 7; ++i)
    if (!whole(a[i], f + i) || f[i] == 0) {
      PyErr_SetString(PyExc_TypeError, "an address is an int");
      return nullptr;
    }
  append_batch_fn = reinterpret_cast<decltype(append_batch_fn)>(f[0]);
  rope_fn = reinterpret_cast<decltype(rope_fn)>(f[1]);
  forward_fn = reinterpret_cast<decltype(forward_fn)>(f[2]);
  share_fn = reinterpret_cast<decltype(share_fn)>(f[3]);
  forward_rope_fn = reinterpret_cast<decltype(forward_rope_fn)>(f[4]);
  publish_fn = reinterpret_cast<decltype(publish_fn)>(f[5]);
  linear_fn = reinterpret_cast<decltype(linear_fn)>(f[6]);
  Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(linear), METHOD(append_batch), METHOD(rope), METHOD(forward), METHOD(forward_rope), METHOD(qkv_publish),
                         METHOD(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
