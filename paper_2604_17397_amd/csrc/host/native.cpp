// Argument marshalling of the calls a denoising loop makes most often (attention, rotary embedding, the routing
// decision, commit, rollback, snapshot), in C++: the same checks and the same call into libsdvg as
// binding.py makes. Every function either finds all checks of its Python counterpart satisfied and
// makes the call, or returns None without having done anything; the Python counterpart then takes
// over, raises what it always raised, or handles the rarer form (fp32, tensor subclasses, ...).
//
// Why: on a small layer the GPU is done in 4 to 16 us, while checking and converting six tensors
// through ctypes took 15 us per attention call and 12 per rotary pass. A batch of 1, 2 or 3 items took 21, 32 and 43 us,
// commit, rollback and snapshot 7 to 10, which the GPU waits for behind a routing decision.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>

#include <string.h>

#include "sdvg.h"

namespace {

constexpr int kMaxItems = 8;  // of a batch; larger ones are Python's, which raises

using attn_fn = int (*)(const sdvg_attn_desc *, const void *, const void *, const void *, const void *, const void *,
                        int64_t, void *, void *);
using attn_commit_fn = int (*)(const sdvg_attn_desc *, const void *, void *, void *, const void *, const void *, int64_t,
                               void *, void *);
using rope_fn = int (*)(const void *, const float *, const float *, void *, int64_t, int32_t, int32_t, int64_t, int64_t,
                        int64_t, int64_t, void *);
using route_fn = int (*)(const float *, int32_t, float, int32_t, float *, void *);
using batch_fn = int (*)(const sdvg_attn_desc *, int32_t, const void *const *, const void *const *, const void *const *,
                         const void *const *, const void *const *, int64_t, void *const *, void *, int64_t, int32_t, void *);
using batch_static_fn = int (*)(const sdvg_attn_desc *, int32_t, const void *const *, const void *const *,
                                const void *const *, const void *const *, const void *const *, int64_t, void *const *,
                                int32_t, void *);
using commit_fn = int (*)(sdvg_kv_cache *, const void *, const void *, int32_t, void *);
using commit_rope_fn = int (*)(sdvg_kv_cache *, const void *, const void *, int32_t, const float *, const float *, void *);
using rollback_fn = int (*)(sdvg_kv_cache *, int64_t, void *);
using snapshot_fn = int (*)(void *, const void *, int64_t, void *);

// Entry points of the libsdvg that binding.py has loaded, and torch's current-stream functions.
struct Api {
  attn_fn attn = nullptr;
  attn_commit_fn attn_commit = nullptr;
  rope_fn rope = nullptr;
  route_fn route_min = nullptr, route_mean = nullptr;
  batch_fn batch = nullptr;
  batch_static_fn batch_static = nullptr;
  commit_fn commit = nullptr;
  commit_rope_fn commit_rope = nullptr;
  rollback_fn rollback = nullptr;
  snapshot_fn snapshot = nullptr;
  PyObject *get_device = nullptr, *get_raw_stream = nullptr, *float32 = nullptr, *cache_type = nullptr;
} api;

// A plain strided GPU tensor, or null (subclasses, wrappers and CPU tensors are Python's).
const at::Tensor *gpu_tensor(PyObject *o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.unsafeGetTensorImpl()->is_python_dispatch())
    return nullptr;
  return &t;
}

bool integer(PyObject *o, int64_t &v) {
  if (!PyLong_CheckExact(o)) return false;
  v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

// The stream to launch on: torch's current one for None, else the raw pointer binding.py passes.
bool stream_ptr(PyObject *o, void *&s) {
  if (o != Py_None) {
    int64_t v;
    if (!integer(o, v)) return false;
    s = reinterpret_cast<void *>(v);
    return true;
  }
  PyObject *dev = PyObject_CallNoArgs(api.get_device);
  PyObject *raw = dev ? PyObject_CallOneArg(api.get_raw_stream, dev) : nullptr;
  Py_XDECREF(dev);
  int64_t v;
  const bool ok = raw && integer(raw, v);
  Py_XDECREF(raw);
  if (!ok) {
    PyErr_Clear();
    return false;
  }
  s = reinterpret_cast<void *>(v);
  return true;
}

// The output tensor: the one given if it matches `like`, a new one for None; undefined if neither.
at::Tensor output(PyObject *o, const at::Tensor &like) {
  if (o == Py_None) {
    at::Tensor out = at::empty(like.sizes(), at::TensorOptions().dtype(like.scalar_type()).device(like.device()));
    return out.unsafeGetTensorImpl()->is_python_dispatch() ? at::Tensor() : out;
  }
  const at::Tensor *out = gpu_tensor(o);
  if (!out || out->sizes() != like.sizes() || out->scalar_type() != like.scalar_type() || out->stride(2) != 1 ||
      out->device() != like.device())
    return at::Tensor();
  return *out;
}

// What a call returns to binding.py: the output for status 0, the status otherwise.
PyObject *result(int status, PyObject *given, const at::Tensor &out) {
  if (status != 0) return PyLong_FromLong(status);
  if (given == Py_None) return THPVariable_Wrap(out);
  Py_INCREF(given);
  return given;
}

#define PYTHON_TAKES_OVER \
  do {                    \
    Py_RETURN_NONE;       \
  } while (0)

// One (q, k_cache, v_cache, k_blk, v_blk) set that passes every check but the output's.
struct Item {
  const at::Tensor *q, *kc, *vc, *kb, *vb;  // kc, vc null without a cache
};
bool attn_item(PyObject *const *a, int64_t cache_len, Item &it) {
  const bool cached = a[1] != Py_None;
  it = Item{gpu_tensor(a[0]), cached ? gpu_tensor(a[1]) : nullptr, cached ? gpu_tensor(a[2]) : nullptr, gpu_tensor(a[3]),
            gpu_tensor(a[4])};
  if (!it.q || !it.kb || !it.vb || cache_len < 0) return false;
  if (cached ? (!it.kc || !it.vc) : (a[2] != Py_None || cache_len > 0)) return false;
  const at::Tensor &q = *it.q;
  if (q.scalar_type() != at::kBFloat16 || q.dim() != 3 || q.stride(2) != 1) return false;
  for (const at::Tensor *t : {it.kc, it.vc, it.kb, it.vb})
    if (t && (t->scalar_type() != at::kBFloat16 || t->dim() != 3 || t->stride(2) != 1 || t->size(1) != q.size(1) ||
              t->size(2) != q.size(2) || t->device() != q.device()))
      return false;
  if (it.kb->sizes() != it.vb->sizes() || it.kb->strides() != it.vb->strides()) return false;
  return !cached || (it.kc->sizes() == it.vc->sizes() && it.kc->strides() == it.vc->strides() && cache_len <= it.kc->size(0));
}
sdvg_attn_desc attn_desc(const Item &it, const at::Tensor &out, double scale) {
  return sdvg_attn_desc{static_cast<int32_t>(it.q->size(0)), static_cast<int32_t>(it.kb->size(0)),
                        static_cast<int32_t>(it.q->size(1)), static_cast<int32_t>(it.q->size(2)),
                        it.q->stride(0), it.q->stride(1), out.stride(0), out.stride(1),
                        it.kc ? it.kc->stride(0) : 128, it.kc ? it.kc->stride(1) : 128, it.kb->stride(0), it.kb->stride(1),
                        static_cast<float>(scale), SDVG_BF16};
}
bool scale_of(PyObject *o, double &scale) {
  scale = 0.0;
  if (o == Py_None) return true;
  if (!PyFloat_CheckExact(o)) return false;
  scale = PyFloat_AS_DOUBLE(o);
  return true;
}

// (q, k_cache, v_cache, k_blk, v_blk, cache_len, out, scale, stream, commit)
PyObject *block_attn_impl(PyObject *const *a, Py_ssize_t n) {
  if (n != 10) PYTHON_TAKES_OVER;
  const bool commit = a[9] == Py_True;
  Item it;
  int64_t cache_len;
  double scale;
  if (!integer(a[5], cache_len) || !attn_item(a, cache_len, it) || !scale_of(a[7], scale)) PYTHON_TAKES_OVER;
  if (commit && (!it.kc || cache_len + it.kb->size(0) > it.kc->size(0))) PYTHON_TAKES_OVER;
  void *stream;
  if (!stream_ptr(a[8], stream)) PYTHON_TAKES_OVER;
  const at::Tensor out = output(a[6], *it.q);
  if (!out.defined()) PYTHON_TAKES_OVER;
  const sdvg_attn_desc d = attn_desc(it, out, scale);
  void *const qp = it.q->data_ptr(), *const kcp = it.kc ? it.kc->data_ptr() : nullptr,
             *const vcp = it.vc ? it.vc->data_ptr() : nullptr, *const kbp = it.kb->data_ptr(),
             *const vbp = it.vb->data_ptr(), *const op = out.data_ptr();
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = commit ? api.attn_commit(&d, qp, kcp, vcp, kbp, vbp, cache_len, op, stream)
                  : api.attn(&d, qp, kcp, vcp, kbp, vbp, cache_len, op, stream);
  Py_END_ALLOW_THREADS
  return result(status, a[6], out);
}

// Item i of a list or tuple (borrowed), or null.
PyObject *entry(PyObject *seq, Py_ssize_t i) {
  if (PyList_CheckExact(seq)) return i < PyList_GET_SIZE(seq) ? PyList_GET_ITEM(seq, i) : nullptr;
  return PyTuple_CheckExact(seq) && i < PyTuple_GET_SIZE(seq) ? PyTuple_GET_ITEM(seq, i) : nullptr;
}
bool has_length(PyObject *seq, Py_ssize_t n) {
  return PyList_CheckExact(seq) ? PyList_GET_SIZE(seq) == n : PyTuple_CheckExact(seq) && PyTuple_GET_SIZE(seq) == n;
}

// (qs, k_caches, v_caches, k_blks, v_blks, cache_len, outs, workspace, split, scale, stream, static)
PyObject *batch_impl(PyObject *const *a, Py_ssize_t n_args) {
  if (n_args != 12) PYTHON_TAKES_OVER;
  const Py_ssize_t n = PyList_CheckExact(a[0]) ? PyList_GET_SIZE(a[0]) : PyTuple_CheckExact(a[0]) ? PyTuple_GET_SIZE(a[0]) : 0;
  if (n < 1 || n > kMaxItems || !has_length(a[3], n) || !has_length(a[4], n)) PYTHON_TAKES_OVER;
  const bool no_caches = a[1] == Py_None, own_outs = a[6] == Py_None, is_static = a[11] == Py_True;
  if (!no_caches && (!has_length(a[1], n) || !has_length(a[2], n))) PYTHON_TAKES_OVER;
  int64_t cache_len, split;
  double scale;
  if (!integer(a[5], cache_len) || !integer(a[8], split) || !scale_of(a[9], scale)) PYTHON_TAKES_OVER;
  Item items[kMaxItems];
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject *const set[5] = {entry(a[0], i), no_caches ? Py_None : entry(a[1], i), no_caches ? Py_None : entry(a[2], i),
                              entry(a[3], i), entry(a[4], i)};
    if (!attn_item(set, cache_len, items[i]) || items[i].q->device() != items[0].q->device()) PYTHON_TAKES_OVER;
  }
  const at::Tensor *ws = a[7] == Py_None ? nullptr : gpu_tensor(a[7]);
  if (a[7] != Py_None && (!ws || !ws->is_contiguous() || ws->device() != items[0].q->device())) PYTHON_TAKES_OVER;
  void *stream;
  if (!stream_ptr(a[10], stream)) PYTHON_TAKES_OVER;
  at::Tensor outs[kMaxItems];
  sdvg_attn_desc d{};
  const void *qp[kMaxItems], *kcp[kMaxItems], *vcp[kMaxItems], *kbp[kMaxItems], *vbp[kMaxItems];
  void *op[kMaxItems];
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject *given = own_outs ? Py_None : entry(a[6], i);
    if (!given || (given == Py_None && !own_outs)) PYTHON_TAKES_OVER;
    outs[i] = output(given, *items[i].q);
    if (!outs[i].defined()) PYTHON_TAKES_OVER;
    const sdvg_attn_desc di = attn_desc(items[i], outs[i], scale);
    if (i == 0)
      d = di;
    else if (memcmp(&di, &d, sizeof d) != 0)
      PYTHON_TAKES_OVER;
    qp[i] = items[i].q->data_ptr();
    kcp[i] = items[i].kc ? items[i].kc->data_ptr() : nullptr;
    vcp[i] = items[i].vc ? items[i].vc->data_ptr() : nullptr;
    kbp[i] = items[i].kb->data_ptr();
    vbp[i] = items[i].vb->data_ptr();
    op[i] = outs[i].data_ptr();
  }
  PyObject *ret = a[6];
  if (own_outs) {
    ret = PyList_New(n);
    if (!ret) return nullptr;
    for (Py_ssize_t i = 0; i < n; ++i) PyList_SET_ITEM(ret, i, THPVariable_Wrap(outs[i]));
  } else {
    Py_INCREF(ret);
  }
  void *const wp = ws ? ws->data_ptr() : nullptr;
  const int64_t w_bytes = ws ? static_cast<int64_t>(ws->nbytes()) : 0;
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = is_static ? api.batch_static(&d, static_cast<int32_t>(n), qp, kcp, vcp, kbp, vbp, cache_len, op,
                                        static_cast<int32_t>(split), stream)
                     : api.batch(&d, static_cast<int32_t>(n), qp, kcp, vcp, kbp, vbp, cache_len, op, wp, w_bytes,
                                 static_cast<int32_t>(split), stream);
  Py_END_ALLOW_THREADS
  if (status == 0) return ret;
  Py_DECREF(ret);
  return PyLong_FromLong(status);
}

// The sdvg_kv_cache inside a ctypes structure of binding.py, for as long as this lives.
struct CacheRef {
  Py_buffer view{};
  sdvg_kv_cache *c = nullptr;
  explicit CacheRef(PyObject *o) {
    if (reinterpret_cast<PyObject *>(Py_TYPE(o)) != api.cache_type) return;
    if (PyObject_GetBuffer(o, &view, PyBUF_WRITABLE) != 0) {
      PyErr_Clear();
      return;
    }
    if (view.len == static_cast<Py_ssize_t>(sizeof(sdvg_kv_cache))) c = static_cast<sdvg_kv_cache *>(view.buf);
  }
  ~CacheRef() {
    if (view.obj) PyBuffer_Release(&view);
  }
  CacheRef(const CacheRef &) = delete;
  CacheRef &operator=(const CacheRef &) = delete;
};

// A dense bf16 [layers][T][heads][dim] block of the cache's shape.
const at::Tensor *block_tensor(PyObject *o, const sdvg_kv_cache &c) {
  const at::Tensor *t = gpu_tensor(o);
  if (!t || t->scalar_type() != at::kBFloat16 || t->dim() != 4 || !t->is_contiguous() || t->size(0) != c.n_layers ||
      t->size(1) != c.block_tokens || t->size(2) != c.n_heads || t->size(3) != c.head_dim)
    return nullptr;
  return t;
}

// (cache.c, k_blk, v_blk, slot, stream), and cos, sin with the rotation of K
PyObject *commit_impl(PyObject *const *a, Py_ssize_t n) {
  if (n != 5 && n != 7) PYTHON_TAKES_OVER;
  const CacheRef cache(a[0]);
  int64_t slot;
  if (!cache.c || !integer(a[3], slot) || slot != static_cast<int32_t>(slot)) PYTHON_TAKES_OVER;
  const at::Tensor *kb = block_tensor(a[1], *cache.c), *vb = block_tensor(a[2], *cache.c);
  if (!kb || !vb) PYTHON_TAKES_OVER;
  const float *tables[2] = {nullptr, nullptr};
  for (int i = 0; n == 7 && i < 2; ++i) {
    const at::Tensor *t = gpu_tensor(a[5 + i]);
    if (!t || t->scalar_type() != at::kFloat || t->dim() != 2 || t->size(0) != cache.c->block_tokens || t->size(1) != 64 ||
        !t->is_contiguous() || t->device() != kb->device())
      PYTHON_TAKES_OVER;
    tables[i] = static_cast<const float *>(t->data_ptr());
  }
  void *stream;
  if (!stream_ptr(a[4], stream)) PYTHON_TAKES_OVER;
  const void *const kp = kb->data_ptr(), *const vp = vb->data_ptr();
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = n == 5 ? api.commit(cache.c, kp, vp, static_cast<int32_t>(slot), stream)
                  : api.commit_rope(cache.c, kp, vp, static_cast<int32_t>(slot), tables[0], tables[1], stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// (cache.c, new_len, stream)
PyObject *rollback_impl(PyObject *const *a, Py_ssize_t n) {
  if (n != 3) PYTHON_TAKES_OVER;
  const CacheRef cache(a[0]);
  int64_t new_len;
  void *stream;
  if (!cache.c || !integer(a[1], new_len) || !stream_ptr(a[2], stream)) PYTHON_TAKES_OVER;
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = api.rollback(cache.c, new_len, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// (dst, src, n_bytes, stream)
PyObject *snapshot_impl(PyObject *const *a, Py_ssize_t n) {
  if (n != 4) PYTHON_TAKES_OVER;
  const at::Tensor *dst = gpu_tensor(a[0]), *src = gpu_tensor(a[1]);
  if (!dst || !src || !dst->is_contiguous() || !src->is_contiguous()) PYTHON_TAKES_OVER;
  const int64_t dst_bytes = static_cast<int64_t>(dst->nbytes()), src_bytes = static_cast<int64_t>(src->nbytes());
  int64_t n_bytes = src_bytes;
  if (a[2] != Py_None && !integer(a[2], n_bytes)) PYTHON_TAKES_OVER;
  void *stream;
  if (n_bytes > dst_bytes || n_bytes > src_bytes || !stream_ptr(a[3], stream)) PYTHON_TAKES_OVER;
  void *const dp = dst->data_ptr(), *const sp = src->data_ptr();
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = api.snapshot(dp, sp, n_bytes, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// (x, cos, sin, out, stream)
PyObject *rope_impl(PyObject *const *a, Py_ssize_t n) {
  if (n != 5) PYTHON_TAKES_OVER;
  const at::Tensor *x = gpu_tensor(a[0]), *cos = gpu_tensor(a[1]), *sin = gpu_tensor(a[2]);
  if (!x || !cos || !sin) PYTHON_TAKES_OVER;
  if (x->scalar_type() != at::kBFloat16 || x->dim() != 3 || x->size(2) != 128 || x->stride(2) != 1) PYTHON_TAKES_OVER;
  for (const at::Tensor *t : {cos, sin})
    if (t->scalar_type() != at::kFloat || t->dim() != 2 || t->size(0) != x->size(0) || t->size(1) != 64 ||
        !t->is_contiguous() || t->device() != x->device())
      PYTHON_TAKES_OVER;
  void *stream;
  if (!stream_ptr(a[4], stream)) PYTHON_TAKES_OVER;
  const at::Tensor out = output(a[3], *x);
  if (!out.defined()) PYTHON_TAKES_OVER;
  void *const xp = x->data_ptr(), *const op = out.data_ptr();
  const float *const cp = static_cast<const float *>(cos->data_ptr()), *const sp = static_cast<const float *>(sin->data_ptr());
  const int64_t n_tokens = x->size(0), xs0 = x->stride(0), xs1 = x->stride(1), os0 = out.stride(0), os1 = out.stride(1);
  const int32_t heads = static_cast<int32_t>(x->size(1));
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = api.rope(xp, cp, sp, op, n_tokens, heads, 128, xs0, xs1, os0, os1, stream);
  Py_END_ALLOW_THREADS
  return result(status, a[3], out);
}

// (frame_scores, tau, block_idx, mean, stream) -> (decision, numpy float32), a negative status, or None
PyObject *route_impl(PyObject *const *a, Py_ssize_t n) {
  if (n != 5) PYTHON_TAKES_OVER;
  const at::Tensor *s = gpu_tensor(a[0]);
  int64_t block_idx;
  if (!s || s->scalar_type() != at::kFloat || s->dim() != 1 || !s->is_contiguous()) PYTHON_TAKES_OVER;
  if (!PyFloat_CheckExact(a[1]) || !integer(a[2], block_idx) || block_idx != static_cast<int32_t>(block_idx) ||
      s->size(0) > INT32_MAX)
    PYTHON_TAKES_OVER;
  void *stream;
  if (!stream_ptr(a[4], stream)) PYTHON_TAKES_OVER;
  const float *const sp = static_cast<const float *>(s->data_ptr());
  const int32_t frames = static_cast<int32_t>(s->size(0));
  const float tau = static_cast<float>(PyFloat_AS_DOUBLE(a[1]));
  const route_fn fn = a[3] == Py_True ? api.route_mean : api.route_min;
  float q_b = 0.f;
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = fn(sp, frames, tau, static_cast<int32_t>(block_idx), &q_b, stream);
  Py_END_ALLOW_THREADS
  if (status < 0) return PyLong_FromLong(status);
  PyObject *value = PyFloat_FromDouble(static_cast<double>(q_b));
  PyObject *scalar = value ? PyObject_CallOneArg(api.float32, value) : nullptr;
  Py_XDECREF(value);
  return scalar ? Py_BuildValue("(iN)", status, scalar) : nullptr;
}

// Anything torch throws (a tensor without storage, ...) happens before the launch: Python repeats
// the call and reports it its own way.
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n) {
  try {
    return F(args, n);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// (addresses of attn, attn_commit, rope, route_min, route_mean, batch, batch_static, commit, commit_rope, rollback,
// snapshot; torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, numpy.float32, the ctypes class of the cache)
PyObject *init(PyObject *, PyObject *const *a, Py_ssize_t n) {
  constexpr int kEntries = 11;
  int64_t p[kEntries];
  if (n != kEntries + 4) {
    PyErr_SetString(PyExc_TypeError, "init takes 15 arguments");
    return nullptr;
  }
  for (int i = 0; i < kEntries; ++i)
    if (!integer(a[i], p[i]) || !p[i]) {
      PyErr_SetString(PyExc_TypeError, "init: not an address");
      return nullptr;
    }
  for (int i = kEntries; i < n; ++i) Py_INCREF(a[i]);
  api = Api{reinterpret_cast<attn_fn>(p[0]),    reinterpret_cast<attn_commit_fn>(p[1]),  reinterpret_cast<rope_fn>(p[2]),
            reinterpret_cast<route_fn>(p[3]),   reinterpret_cast<route_fn>(p[4]),        reinterpret_cast<batch_fn>(p[5]),
            reinterpret_cast<batch_static_fn>(p[6]), reinterpret_cast<commit_fn>(p[7]),  reinterpret_cast<commit_rope_fn>(p[8]),
            reinterpret_cast<rollback_fn>(p[9]), reinterpret_cast<snapshot_fn>(p[10]),   a[11], a[12], a[13], a[14]};
  Py_RETURN_NONE;
}

#define METHOD(name, fn) \
  { name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr }
PyMethodDef methods[] = {METHOD("init", init), METHOD("block_attn", guarded<block_attn_impl>),
                         METHOD("rope", guarded<rope_impl>), METHOD("route", guarded<route_impl>),
                         METHOD("batch", guarded<batch_impl>), METHOD("commit", guarded<commit_impl>),
                         METHOD("rollback", guarded<rollback_impl>), METHOD("snapshot", guarded<snapshot_impl>),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "Argument marshalling of libsdvg's most frequent calls.",
                          -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__native() { return PyModule_Create(&module_def); }
