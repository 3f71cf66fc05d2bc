// Native argument marshalling of the calls a training step makes many times: torch tensors, lists and numbers straight into
// the structs of the C ABI (include/startrail.h).  Bounded by nothing but instructions; through ctypes a ring call with 8
// chunks took 15 us (forward) and 30 us (backward) of Python beside the 4 to 13 us its launches take, more with more chunks,
// and small shares were that much host time: 128 rows of one fp32 head 68 us a pass for 43 us of kernels.
//
// Every function returns the status of the call, or None without having called anything when an argument is not what the
// short way takes (another sequence type, a tensor subclass, a shape or dtype that does not fit ...): the Python wrapper
// then goes the general way, which accepts what is acceptable and raises the error that belongs to the rest.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/startrail.h"

namespace {

// ---- arguments; false: not for the short way
using Tensor = const at::Tensor*;

bool tensor(PyObject* o, Tensor* t) {
  if (!THPVariable_CheckExact(o)) return false;
  *t = &THPVariable_Unpack(o);
  const at::Tensor& x = **t;
  if (!x.defined() || x.layout() != at::kStrided || !x.is_cuda() || !x.has_storage()) return false;
  // wrappers of transforms, fake and lazy tensors and views with a pending operation have other keys
  const auto plain = c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                                          c10::DispatchKey::AutocastCUDA});
  return ((x.key_set() - plain).raw_repr() & ~c10::full_backend_mask) == 0;
}
void* address(Tensor t) { return t->numel() ? t->data_ptr() : nullptr; }
bool pointer(PyObject* o, void** p) {          // None: null
  *p = nullptr;
  Tensor t;
  if (o == Py_None) return true;
  if (!tensor(o, &t)) return false;
  *p = address(t);
  return true;
}
bool dtype_code(Tensor t, int32_t* code) {
  *code = t->scalar_type() == at::kFloat ? ST_F32 : ST_BF16;
  return t->scalar_type() == at::kFloat || t->scalar_type() == at::kBFloat16;
}
bool dense_f32(PyObject* o, at::IntArrayRef shape, float** p) {
  Tensor t;
  if (!tensor(o, &t) || t->scalar_type() != at::kFloat || t->sizes() != shape || !t->is_contiguous()) return false;
  *p = (float*)address(t);
  return true;
}
bool strides_fit(Tensor t) { return t->dim() == 4 && (t->stride(3) == 1 || t->size(3) <= 1); }
bool view(PyObject* o, Tensor* t, st_tensor* v) {
  if (!tensor(o, t) || !strides_fit(*t)) return false;
  *v = st_tensor{address(*t), (*t)->stride(0), (*t)->stride(1), (*t)->stride(2)};
  return true;
}
bool integer(PyObject* o, int64_t* x) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  *x = PyLong_AsLongLongAndOverflow(o, &overflow);
  return overflow == 0;
}
bool integer(PyObject* o, int32_t* x) {
  int64_t y;
  if (!integer(o, &y) || y < INT32_MIN || y > INT32_MAX) return false;
  *x = (int32_t)y;
  return true;
}
bool real(PyObject* o, float* x) {
  if (!PyFloat_CheckExact(o)) return false;
  *x = (float)PyFloat_AS_DOUBLE(o);
  return true;
}
bool truth(PyObject* o, int32_t* x) {
  *x = o == Py_True;
  return o == Py_True || o == Py_False;
}
bool handle(PyObject* o, void** p) {
  int64_t x;
  if (!integer(o, &x)) return false;
  *p = (void*)x;
  return true;
}
struct Items {
  Py_ssize_t n = 0;
  PyObject** at = nullptr;
};
bool items(PyObject* o, Items* s) {
  if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
  s->n = PySequence_Fast_GET_SIZE(o);
  s->at = PySequence_Fast_ITEMS(o);
  return true;
}
bool integers(PyObject* o, int32_t* to, Py_ssize_t most, Py_ssize_t* n) {
  Items s;
  if (!items(o, &s) || s.n > most) return false;
  for (Py_ssize_t i = 0; i < s.n; ++i)
    if (!integer(s.at[i], to + i)) return false;
  *n = s.n;
  return true;
}
template <typename Desc>
bool where(PyObject* o, Desc* d) {             // position of row 0, or (position, rows of the first run, position of the second)
  d->q_seg = 0;
  d->q_offset2 = 0;
  if (!PyTuple_CheckExact(o)) return integer(o, &d->q_offset);
  return PyTuple_GET_SIZE(o) == 3 && integer(PyTuple_GET_ITEM(o, 0), &d->q_offset) && integer(PyTuple_GET_ITEM(o, 1), &d->q_seg) &&
         integer(PyTuple_GET_ITEM(o, 2), &d->q_offset2);
}
template <typename Desc>
bool shape(Tensor q, Desc* d) {
  if (q->dim() != 4 || !dtype_code(q, &d->dtype)) return false;
  for (int i = 0; i < 4; ++i)
    if (q->size(i) > INT32_MAX) return false;
  d->B = (int32_t)q->size(0);
  d->Sq = (int32_t)q->size(1);
  d->Hq = (int32_t)q->size(2);
  d->D = (int32_t)q->size(3);
  return true;
}
bool bytes_of(PyObject* o, void** p, size_t* n) {   // first 256-byte boundary of a buffer and what is left from there
  Tensor t;
  if (!tensor(o, &t)) return false;
  const uintptr_t at = (uintptr_t)t->data_ptr(), up = (at + 255) / 256 * 256;
  const size_t have = (size_t)t->numel() * t->element_size();
  if (have < up - at) return false;
  *p = (void*)up;
  *n = have - (up - at);
  return true;
}

// the tables of a ring call
struct Ring {
  st_ring_desc d;
  Tensor q, k0;
  st_tensor tq;
  const void *k[ST_MAX_CHUNKS], *v[ST_MAX_CHUNKS];
  int64_t k_offset[ST_MAX_CHUNKS];
  int32_t order[ST_MAX_CHUNKS];
  Py_ssize_t n_visit;
  int32_t mode;

  bool chunks(PyObject* o, const void** to, Tensor first, int64_t* strides) {
    Items s;
    if (!items(o, &s) || s.n != d.n_chunks) return false;
    Tensor t0 = nullptr;
    for (Py_ssize_t i = 0; i < s.n; ++i) {
      Tensor t;
      if (!tensor(s.at[i], &t)) return false;
      if (i == 0) {
        t0 = t;
        if (!strides_fit(t)) return false;
        if (first == nullptr) first = k0 = t;
      }
      if (t->sizes() != first->sizes() || t->strides() != t0->strides() || t->scalar_type() != q->scalar_type()) return false;
      to[i] = t->data_ptr();
    }
    for (int i = 0; i < 3; ++i) strides[i] = t0->stride(i);
    return true;
  }
  bool read(PyObject* oq, PyObject* ks, PyObject* vs, PyObject* q_where, PyObject* k_offsets, PyObject* causal, PyObject* scale,
            PyObject* visit, PyObject* mode_) {
    Items off;
    if (!items(k_offsets, &off) || off.n < 1 || off.n > ST_MAX_CHUNKS) return false;
    d.n_chunks = (int32_t)off.n;
    for (Py_ssize_t i = 0; i < off.n; ++i)
      if (!integer(off.at[i], k_offset + i)) return false;
    if (!view(oq, &q, &tq) || !shape(q, &d) || !where(q_where, &d) || !truth(causal, &d.causal) || !real(scale, &d.scale)) return false;
    if (!chunks(ks, k, nullptr, &d.k_stride_b) || !chunks(vs, v, k0, &d.v_stride_b)) return false;
    if (k0->size(1) > INT32_MAX || k0->size(2) > INT32_MAX) return false;
    d.Sk = (int32_t)k0->size(1);
    d.Hkv = (int32_t)k0->size(2);
    d.k_ptr = k;
    d.v_ptr = v;
    d.k_offset = k_offset;
    return integers(visit, order, ST_MAX_CHUNKS, &n_visit) && integer(mode_, &mode);
  }
  at::IntArrayRef q_shape() const { return q->sizes(); }
  std::array<int64_t, 3> stat_shape() const { return {d.B, d.Hq, d.Sq}; }
};
static_assert(offsetof(st_ring_desc, k_stride_h) == offsetof(st_ring_desc, k_stride_b) + 16 &&
              offsetof(st_ring_desc, v_stride_h) == offsetof(st_ring_desc, v_stride_b) + 16, "strides lie side by side");

// gradient accumulators (fp32) or their copies (low: the dtype of q) per chunk, None where there is none
bool tables(PyObject* o, const Ring& r, bool low, void** to) {
  Items s;
  if (!items(o, &s) || s.n != r.d.n_chunks) return false;
  for (Py_ssize_t i = 0; i < s.n; ++i) {
    to[i] = nullptr;
    if (s.at[i] == Py_None) continue;
    Tensor t;
    if (!tensor(s.at[i], &t) || t->scalar_type() != (low ? r.q->scalar_type() : at::kFloat) || t->sizes() != r.k0->sizes() || !t->is_contiguous()) return false;
    to[i] = t->data_ptr();
  }
  return true;
}

struct Unlocked {                              // other Python threads run meanwhile
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename F>
PyObject* call(F f) {
  st_status s;
  {
    Unlocked u;
    s = f();
  }
  return PyLong_FromLong(s);
}
// Python calls in through C: an exception of a tensor's accessors (memory that may not be touched, a copy on write that does not
// fit) must not leave here.  Nothing has been called yet then; the general way meets the same exception and raises it.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  try {
    return F(self, a, n);
  } catch (...) {
    Py_RETURN_NONE;
  }
}
#define ST_SHORT(cond) \
  if (!(cond)) Py_RETURN_NONE

// ring_fwd(q, ks, vs, where, k_offsets, causal, scale, order, members, mode, o, lse, o_low, workspace, stream)
PyObject* ring_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 15);
  Ring r;
  int32_t members[ST_MAX_CHUNKS];
  Py_ssize_t n_members = 0;
  float *o, *lse;
  void *low, *ws, *stream;
  size_t ws_bytes;
  ST_SHORT(r.read(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[9]));
  const bool has_members = a[8] != Py_None;
  ST_SHORT(!has_members || (integers(a[8], members, ST_MAX_CHUNKS, &n_members) && n_members == r.n_visit));
  ST_SHORT(dense_f32(a[10], r.q_shape(), &o) && dense_f32(a[11], r.stat_shape(), &lse) && pointer(a[12], &low) &&
           bytes_of(a[13], &ws, &ws_bytes) && handle(a[14], &stream));
  return call([&] {
    return st_ring_fwd(&r.d, &r.tq, r.order, has_members ? members : nullptr, (int32_t)r.n_visit, r.mode, o, lse, low, ws, ws_bytes, stream);
  });
}

// ring_bwd(q, ks, vs, d_o, o, lse, where, k_offsets, causal, scale, order, dq, dk, dv, assign, dk_low, dv_low, mode, workspace,
// stream): st_ring_bwd_last, or st_ring_bwd_noalloc where the workspace is None (then without assign and copies)
PyObject* ring_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 20);
  Ring r;
  Tensor t_do, t_o;
  st_tensor tdo, to;
  int32_t o_dtype, assign;
  float *lse, *dq;
  void *dk[ST_MAX_CHUNKS], *dv[ST_MAX_CHUNKS], *lk[ST_MAX_CHUNKS], *lv[ST_MAX_CHUNKS], *ws = nullptr, *stream;
  size_t ws_bytes = 0;
  ST_SHORT(r.read(a[0], a[1], a[2], a[6], a[7], a[8], a[9], a[10], a[17]));
  ST_SHORT(view(a[3], &t_do, &tdo) && view(a[4], &t_o, &to) && dtype_code(t_o, &o_dtype) && dense_f32(a[5], r.stat_shape(), &lse) &&
           dense_f32(a[11], r.q_shape(), &dq) && tables(a[12], r, false, dk) && tables(a[13], r, false, dv) && truth(a[14], &assign));
  const bool low_k = a[15] != Py_None, low_v = a[16] != Py_None, own = a[18] == Py_None;
  ST_SHORT((!low_k || tables(a[15], r, true, lk)) && (!low_v || tables(a[16], r, true, lv)) && handle(a[19], &stream));
  ST_SHORT(own ? !assign && !low_k && !low_v : bytes_of(a[18], &ws, &ws_bytes));
  return call([&] {
    if (own)
      return st_ring_bwd_noalloc(&r.d, &r.tq, &tdo, &to, o_dtype, lse, r.order, (int32_t)r.n_visit, r.mode, dq, (float* const*)dk, (float* const*)dv, stream);
    return st_ring_bwd_last(&r.d, &r.tq, &tdo, &to, o_dtype, lse, r.order, (int32_t)r.n_visit, r.mode, dq, (float* const*)dk, (float* const*)dv,
                            assign ? ST_KV_ASSIGN : 0, low_k ? lk : nullptr, low_v ? lv : nullptr, ws, ws_bytes, stream);
  });
}

bool block(PyObject* oq, PyObject* ok, PyObject* ov, PyObject* q_where, PyObject* k_offset, PyObject* causal, PyObject* scale, st_block_desc* d,
           Tensor* q, Tensor* k, st_tensor* tq, st_tensor* tk, st_tensor* tv) {
  Tensor v;
  if (!view(oq, q, tq) || !view(ok, k, tk) || !view(ov, &v, tv) || !shape(*q, d) || !where(q_where, d) || !integer(k_offset, &d->k_offset) ||
      !truth(causal, &d->causal) || !real(scale, &d->scale))
    return false;
  if ((*k)->size(1) > INT32_MAX || (*k)->size(2) > INT32_MAX) return false;
  d->Sk = (int32_t)(*k)->size(1);
  d->Hkv = (int32_t)(*k)->size(2);
  return true;
}

// block_fwd(q, k, v, where, k_offset, causal, scale, o, lse, stream)
PyObject* block_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 10);
  st_block_desc d;
  Tensor q, k;
  st_tensor tq, tk, tv;
  float *o, *lse;
  void* stream;
  ST_SHORT(block(a[0], a[1], a[2], a[3], a[4], a[5], a[6], &d, &q, &k, &tq, &tk, &tv));
  ST_SHORT(dense_f32(a[7], q->sizes(), &o) && dense_f32(a[8], {d.B, d.Hq, d.Sq}, &lse) && handle(a[9], &stream));
  return call([&] { return st_attn_block_fwd(&d, &tq, &tk, &tv, o, lse, stream); });
}

// block_bwd(q, k, v, d_o, lse, delta, where, k_offset, causal, scale, dq, dk, dv, workspace, stream)
PyObject* block_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 15);
  st_block_desc d;
  Tensor q, k, t_do;
  st_tensor tq, tk, tv, tdo;
  float *lse, *delta, *dq, *dk, *dv;
  void *ws, *stream;
  size_t ws_bytes;
  ST_SHORT(block(a[0], a[1], a[2], a[6], a[7], a[8], a[9], &d, &q, &k, &tq, &tk, &tv));
  ST_SHORT(view(a[3], &t_do, &tdo) && dense_f32(a[4], {d.B, d.Hq, d.Sq}, &lse) && dense_f32(a[5], {d.B, d.Hq, d.Sq}, &delta) &&
           dense_f32(a[10], q->sizes(), &dq) && dense_f32(a[11], {d.B, d.Sk, d.Hkv, d.D}, &dk) && dense_f32(a[12], {d.B, d.Sk, d.Hkv, d.D}, &dv) &&
           bytes_of(a[13], &ws, &ws_bytes) && handle(a[14], &stream));
  return call([&] { return st_attn_block_bwd(&d, &tq, &tk, &tv, &tdo, lse, delta, dq, dk, dv, ws, ws_bytes, stream); });
}

// a dense copy of shape `s` in out_dtype, or None
bool low_copy(PyObject* o, at::IntArrayRef s, int32_t out_dtype, void** p) {
  *p = nullptr;
  if (o == Py_None) return true;
  Tensor t;
  int32_t code;
  if (!tensor(o, &t) || t->sizes() != s || !t->is_contiguous() || !dtype_code(t, &code) || code != out_dtype) return false;
  *p = address(t);
  return true;
}

// merge(o, lse, o_part, lse_part, out_dtype, o_low, stream)
PyObject* merge(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 7);
  Tensor t;
  float *o, *lse, *op, *lp;
  void *low, *stream;
  int32_t out;
  ST_SHORT(tensor(a[0], &t) && t->dim() == 4 && dense_f32(a[0], t->sizes(), &o) && dense_f32(a[2], t->sizes(), &op));
  const int64_t B = t->size(0), S = t->size(1), H = t->size(2), D = t->size(3);
  ST_SHORT(B <= INT32_MAX && S <= INT32_MAX && H <= INT32_MAX && D <= INT32_MAX);
  ST_SHORT(dense_f32(a[1], {B, H, S}, &lse) && dense_f32(a[3], {B, H, S}, &lp) && integer(a[4], &out) && low_copy(a[5], t->sizes(), out, &low) &&
           handle(a[6], &stream));
  return call([&] { return st_attn_merge(o, lse, op, lp, (int32_t)B, (int32_t)S, (int32_t)H, (int32_t)D, out, low, stream); });
}

// combine(o_parts, lse_parts, row0, rows, out_dtype, o, lse, o_low, stream)
PyObject* combine(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 9);
  Items so, sl;
  const float *op[ST_MAX_CHUNKS], *lp[ST_MAX_CHUNKS];
  int32_t row0, rows, out;
  ST_SHORT(items(a[0], &so) && items(a[1], &sl) && so.n == sl.n && so.n > 0 && so.n <= ST_MAX_CHUNKS && integer(a[2], &row0) && integer(a[3], &rows) &&
           integer(a[4], &out));
  Tensor t;
  ST_SHORT(tensor(so.at[0], &t) && t->dim() == 4);
  const int64_t B = t->size(0), S = t->size(1), H = t->size(2), D = t->size(3);
  ST_SHORT(B <= INT32_MAX && S <= INT32_MAX && H <= INT32_MAX && D <= INT32_MAX && rows >= 0);
  for (Py_ssize_t i = 0; i < so.n; ++i)
    ST_SHORT(dense_f32(so.at[i], t->sizes(), (float**)&op[i]) && dense_f32(sl.at[i], {B, H, S}, (float**)&lp[i]));
  float *o, *lse;
  void *low, *stream;
  ST_SHORT(dense_f32(a[5], {B, rows, H, D}, &o) && dense_f32(a[6], {B, H, rows}, &lse) && low_copy(a[7], {B, rows, H, D}, out, &low) &&
           handle(a[8], &stream));
  return call([&] {
    return st_attn_combine(op, lp, (int32_t)so.n, (int32_t)B, (int32_t)S, (int32_t)H, (int32_t)D, row0, rows, o, lse, out, low, stream);
  });
}

// delta(d_o, o, delta, stream)
PyObject* delta(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 4);
  st_block_desc d;
  memset(&d, 0, sizeof(d));
  Tensor t_do, t_o;
  st_tensor tdo, to;
  int32_t o_dtype;
  float* out;
  void* stream;
  ST_SHORT(view(a[0], &t_do, &tdo) && view(a[1], &t_o, &to) && shape(t_do, &d) && dtype_code(t_o, &o_dtype) &&
           dense_f32(a[2], {d.B, d.Hq, d.Sq}, &out) && handle(a[3], &stream));
  d.Hkv = d.Hq;
  d.scale = 1.f;
  return call([&] { return st_attn_delta(&d, &tdo, &to, o_dtype, out, stream); });
}

// cast(src, dst, dst_dtype, stream)
PyObject* cast(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ST_SHORT(n == 4);
  Tensor src, dst;
  int32_t out, code;
  void* stream;
  ST_SHORT(tensor(a[0], &src) && tensor(a[1], &dst) && integer(a[2], &out) && handle(a[3], &stream));
  ST_SHORT(src->scalar_type() == at::kFloat && src->is_contiguous() && dst->is_contiguous() && dst->numel() == src->numel() &&
           dtype_code(dst, &code) && code == out);
  float* from = (float*)address(src);
  void* to = address(dst);
  const int64_t count = src->numel();
  return call([&] { return st_cast_from_f32(from, to, count, out, stream); });
}

#define ST_METHOD(f) {#f, (PyCFunction)(void*)guarded<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ST_METHOD(ring_fwd), ST_METHOD(ring_bwd), ST_METHOD(block_fwd), ST_METHOD(block_bwd), ST_METHOD(merge),
                         ST_METHOD(combine),  ST_METHOD(delta),    ST_METHOD(cast),      {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", ST_BUILT_FOR) < 0) Py_CLEAR(m);
  return m;
}
