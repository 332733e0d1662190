// Argument marshalling of the calls a denoising loop makes most often (attention of one layer,
// rotary embedding, the routing decision), in C++: the same checks and the same call into libsdvg as
// binding.py makes. Every function either finds all checks of its Python counterpart satisfied and
// makes the call, or returns None without having done anything; the Python counterpart then takes
// over, raises what it always raised, or handles the rarer form (fp32, tensor subclasses, ...).
//
// Why: on a small layer the GPU is done in 4 to 16 us, while checking and converting six tensors
// through ctypes took 15 us per attention call and 12 per rotary pass.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>

#include "sdvg.h"

namespace {

using attn_fn = int (*)(const sdvg_attn_desc *, const void *, const void *, const void *, const void *, const void *,
                        int64_t, void *, void *);
using attn_commit_fn = int (*)(const sdvg_attn_desc *, const void *, void *, void *, const void *, const void *, int64_t,
                               void *, void *);
using rope_fn = int (*)(const void *, const float *, const float *, void *, int64_t, int32_t, int32_t, int64_t, int64_t,
                        int64_t, int64_t, void *);
using route_fn = int (*)(const float *, int32_t, float, int32_t, float *, void *);

// Entry points of the libsdvg that binding.py has loaded, and torch's current-stream functions.
struct Api {
  attn_fn attn = nullptr;
  attn_commit_fn attn_commit = nullptr;
  rope_fn rope = nullptr;
  route_fn route_min = nullptr, route_mean = nullptr;
  PyObject *get_device = nullptr, *get_raw_stream = nullptr, *float32 = nullptr;
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

// (q, k_cache, v_cache, k_blk, v_blk, cache_len, out, scale, stream, commit)
PyObject *block_attn_impl(PyObject *const *a, Py_ssize_t n) {
  if (n != 10) PYTHON_TAKES_OVER;
  const at::Tensor *q = gpu_tensor(a[0]), *kb = gpu_tensor(a[3]), *vb = gpu_tensor(a[4]);
  const bool cached = a[1] != Py_None, commit = a[9] == Py_True;
  const at::Tensor *kc = cached ? gpu_tensor(a[1]) : nullptr, *vc = cached ? gpu_tensor(a[2]) : nullptr;
  int64_t cache_len;
  if (!q || !kb || !vb || !integer(a[5], cache_len) || cache_len < 0) PYTHON_TAKES_OVER;
  if (cached ? (!kc || !vc) : (a[2] != Py_None || cache_len > 0 || commit)) PYTHON_TAKES_OVER;
  if (q->scalar_type() != at::kBFloat16 || q->dim() != 3 || q->stride(2) != 1) PYTHON_TAKES_OVER;
  for (const at::Tensor *t : {kc, vc, kb, vb})
    if (t && (t->scalar_type() != at::kBFloat16 || t->dim() != 3 || t->stride(2) != 1 || t->size(1) != q->size(1) ||
              t->size(2) != q->size(2) || t->device() != q->device()))
      PYTHON_TAKES_OVER;
  if (kb->sizes() != vb->sizes() || kb->strides() != vb->strides()) PYTHON_TAKES_OVER;
  if (cached && (kc->sizes() != vc->sizes() || kc->strides() != vc->strides() || cache_len > kc->size(0))) PYTHON_TAKES_OVER;
  if (commit && cache_len + kb->size(0) > kc->size(0)) PYTHON_TAKES_OVER;
  double scale = 0.0;
  if (a[7] != Py_None) {
    if (!PyFloat_CheckExact(a[7])) PYTHON_TAKES_OVER;
    scale = PyFloat_AS_DOUBLE(a[7]);
  }
  void *stream;
  if (!stream_ptr(a[8], stream)) PYTHON_TAKES_OVER;
  const at::Tensor out = output(a[6], *q);
  if (!out.defined()) PYTHON_TAKES_OVER;
  const sdvg_attn_desc d{static_cast<int32_t>(q->size(0)), static_cast<int32_t>(kb->size(0)),
                         static_cast<int32_t>(q->size(1)), static_cast<int32_t>(q->size(2)),
                         q->stride(0), q->stride(1), out.stride(0), out.stride(1),
                         cached ? kc->stride(0) : 128, cached ? kc->stride(1) : 128, kb->stride(0), kb->stride(1),
                         static_cast<float>(scale), SDVG_BF16};
  void *const qp = q->data_ptr(), *const kcp = cached ? kc->data_ptr() : nullptr,
             *const vcp = cached ? vc->data_ptr() : nullptr, *const kbp = kb->data_ptr(), *const vbp = vb->data_ptr(),
             *const op = out.data_ptr();
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = commit ? api.attn_commit(&d, qp, kcp, vcp, kbp, vbp, cache_len, op, stream)
                  : api.attn(&d, qp, kcp, vcp, kbp, vbp, cache_len, op, stream);
  Py_END_ALLOW_THREADS
  return result(status, a[6], out);
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

// (addresses of attn, attn_commit, rope, route_min, route_mean; torch._C._cuda_getDevice,
// torch._C._cuda_getCurrentRawStream, numpy.float32)
PyObject *init(PyObject *, PyObject *const *a, Py_ssize_t n) {
  int64_t p[5];
  if (n != 8) {
    PyErr_SetString(PyExc_TypeError, "init takes 8 arguments");
    return nullptr;
  }
  for (int i = 0; i < 5; ++i)
    if (!integer(a[i], p[i]) || !p[i]) {
      PyErr_SetString(PyExc_TypeError, "init: not an address");
      return nullptr;
    }
  for (int i = 5; i < 8; ++i) Py_INCREF(a[i]);
  api = Api{reinterpret_cast<attn_fn>(p[0]),  reinterpret_cast<attn_commit_fn>(p[1]), reinterpret_cast<rope_fn>(p[2]),
            reinterpret_cast<route_fn>(p[3]), reinterpret_cast<route_fn>(p[4]),       a[5], a[6], a[7]};
  Py_RETURN_NONE;
}

#define METHOD(name, fn) \
  { name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr }
PyMethodDef methods[] = {METHOD("init", init), METHOD("block_attn", guarded<block_attn_impl>),
                         METHOD("rope", guarded<rope_impl>), METHOD("route", guarded<route_impl>),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "Argument marshalling of libsdvg's most frequent calls.",
                          -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__native() { return PyModule_Create(&module_def); }
