// The tensor calls of binding.py without the interpreter: checks the arguments as the Python functions do, fills the descriptor and
// calls the C ABI.  A function returns the call's status, or -1 for whatever is not the plain case (a tensor subclass, a mode
// that intercepts tensor functions, a tensor of another device, any argument the Python code would refuse): the
// caller then takes the Python path, which raises what it always raised.
// Why: a call of the Python path costs 8 to 12 us of host time in attribute look-ups and conversions, more than its launches;
// steps of small segments were bound by it (2 x 1357
// tokens in 4 segments, bf16, head_dim 64, with the cache calls: 18 calls, 218 us a step; now 159, bound by the kernels).
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <torch/version.h>

#include "s1f.h"

namespace {

// Entry points of the library that binding.py has loaded, and torch's current device and stream.
struct Api {
  decltype(&s1f_seg_attn_fwd) fwd;
  decltype(&s1f_seg_attn_fwd_ws) fwd_ws;
  decltype(&s1f_seg_attn_bwd) bwd;
  decltype(&s1f_seg_attn_bwd_noalloc) bwd_noalloc;
  decltype(&s1f_kv_append) append;
  decltype(&s1f_kv_grad_emit) emit;
};
Api api = {};
PyObject *get_device = nullptr, *get_stream = nullptr;

constexpr int kPython = -1;

// A plain tensor of the current kind of device, or null.
const at::Tensor *plain(PyObject *x) {
  if (!THPVariable_CheckExact(x)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(x);
  return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}

struct Args {
  const at::Tensor *t[10];
  int64_t off = 0;
  void *stream = nullptr;
  // n arguments; number `off_at` is the offset, number `optional` may be None (then a null pointer)
  bool read(PyObject *const *args, Py_ssize_t n, Py_ssize_t want, Py_ssize_t off_at, Py_ssize_t optional) {
    if (n != want || get_device == nullptr || at::impl::PythonTorchFunctionTLS::stack_len() > 0) return false;
    for (Py_ssize_t i = 0, k = 0; i < n; ++i) {
      if (i == off_at) {
        int overflow = 0;
        if (!PyLong_CheckExact(args[i])) return false;
        off = PyLong_AsLongLongAndOverflow(args[i], &overflow);
        if (overflow != 0) return false;
        continue;
      }
      t[k] = i == optional && args[i] == Py_None ? nullptr : plain(args[i]);
      if (t[k] == nullptr && !(i == optional && args[i] == Py_None)) return false;
      ++k;
    }
    return true;
  }
  bool read_stream() {
    PyObject *dev = PyObject_CallNoArgs(get_device);
    PyObject *st = dev ? PyObject_CallOneArg(get_stream, dev) : nullptr;
    Py_XDECREF(dev);
    if (st == nullptr) return PyErr_Clear(), false;
    stream = PyLong_AsVoidPtr(st);
    Py_DECREF(st);
    return PyErr_Occurred() == nullptr || (PyErr_Clear(), false);
  }
};

bool same_layout(const at::Tensor &a, const at::Tensor &b) {
  return a.sizes() == b.sizes() && a.strides() == b.strides() && a.scalar_type() == b.scalar_type();
}
bool rows_of(const at::Tensor &t) { return t.dim() == 4 && t.stride(3) == 1; }
bool dtype_of(const at::Tensor &t, int32_t *code) {
  *code = t.scalar_type() == at::kBFloat16 ? S1F_BF16 : S1F_F32;
  return t.scalar_type() == at::kBFloat16 || t.scalar_type() == at::kFloat;
}
bool fits(int64_t x) { return x >= 0 && x <= 0x7fffffff; }

// Batch entries and head_dim of `small` are what the kernels address `big` with.
bool covers(const at::Tensor &big, const at::Tensor &small) { return big.size(0) >= small.size(0) && big.size(3) >= small.size(3); }

bool desc_of(const at::Tensor &q, const at::Tensor &kv, s1f_desc *d) {
  *d = {};
  if (!rows_of(q) || !rows_of(kv) || !dtype_of(q, &d->dtype) || kv.scalar_type() != q.scalar_type() || !covers(kv, q)) return false;
  if (!fits(q.size(0)) || !fits(q.size(1)) || !fits(kv.size(1)) || !fits(q.size(3))) return false;
  d->batch = (int32_t)q.size(0); d->n_q_heads = (int32_t)q.size(1); d->n_kv_heads = (int32_t)kv.size(1); d->head_dim = (int32_t)q.size(3);
  d->q_stride_b = q.stride(0); d->q_stride_h = q.stride(1); d->q_stride_s = q.stride(2);
  d->kv_stride_b = kv.stride(0); d->kv_stride_h = kv.stride(1); d->kv_stride_s = kv.stride(2);
  d->kv_capacity = kv.size(2);
  return true;
}
bool cache_desc_of(const at::Tensor &cache, const at::Tensor &typed, s1f_desc *d) {
  *d = {};
  if (!rows_of(cache) || !dtype_of(typed, &d->dtype) || !fits(cache.size(0)) || !fits(cache.size(1)) || !fits(cache.size(3))) return false;
  d->batch = (int32_t)cache.size(0); d->n_q_heads = d->n_kv_heads = (int32_t)cache.size(1); d->head_dim = (int32_t)cache.size(3);
  d->q_stride_s = cache.size(3);
  d->kv_stride_b = cache.stride(0); d->kv_stride_h = cache.stride(1); d->kv_stride_s = cache.stride(2);
  d->kv_capacity = cache.size(2);
  return true;
}
bool segment_ok(const at::Tensor &seg, const at::Tensor &cache) {
  return rows_of(seg) && covers(seg, cache) && seg.size(1) >= cache.size(1);
}
bool lse_ok(const at::Tensor &lse, const at::Tensor &q) {
  return lse.scalar_type() == at::kFloat && lse.is_contiguous() && lse.sizes() == q.sizes().slice(0, 3);
}
bool acc_ok(const at::Tensor &k, const at::Tensor &dk, const at::Tensor &dv) {
  return same_layout(dk, dv) && dk.sizes() == k.sizes() && dk.strides() == k.strides() && dk.scalar_type() == at::kFloat;
}
template <typename T = void> T *ptr(const at::Tensor *t) { return static_cast<T *>(t->data_ptr()); }
size_t bytes(const at::Tensor *t) { return t ? (size_t)t->numel() * t->element_size() : 0; }

// The call itself without the interpreter lock; a C++ exception out of a tensor (one without memory) is the Python path's to report.
template <typename F> PyObject *call(F f) {
  int rc = kPython;
  try {
    rc = f();
  } catch (...) {
    rc = kPython;
  }
  return PyLong_FromLong(rc);
}
struct Unlocked {
  PyThreadState *state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// (q, k, v, off, out, lse)
PyObject *fwd(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return call([&]() -> int {
    Args x;
    s1f_desc d;
    if (!x.read(args, n, 6, 3, -1)) return kPython;
    auto &[q, k, v, out, lse] = reinterpret_cast<const at::Tensor *(&)[5]>(x.t);
    if (!same_layout(*q, *out) || !same_layout(*k, *v) || !desc_of(*q, *k, &d) || !lse_ok(*lse, *q) || !x.read_stream()) return kPython;
    void *const p[] = {ptr(q), ptr(k), ptr(v), ptr(out), ptr(lse)};
    Unlocked u;
    return api.fwd(&d, p[0], p[1], p[2], x.off, q->size(2), p[3], static_cast<float *>(p[4]), x.stream);
  });
}
// (q, k, v, off, out, lse, workspace or None)
PyObject *fwd_ws(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return call([&]() -> int {
    Args x;
    s1f_desc d;
    if (!x.read(args, n, 7, 3, 6)) return kPython;
    auto &[q, k, v, out, lse, ws] = reinterpret_cast<const at::Tensor *(&)[6]>(x.t);
    if (!same_layout(*q, *out) || !same_layout(*k, *v) || !desc_of(*q, *k, &d) || !lse_ok(*lse, *q) || !x.read_stream()) return kPython;
    void *const p[] = {ptr(q), ptr(k), ptr(v), ptr(out), ptr(lse), ws ? ptr(ws) : nullptr};
    Unlocked u;
    return api.fwd_ws(&d, p[0], p[1], p[2], x.off, q->size(2), p[3], static_cast<float *>(p[4]), p[5], bytes(ws), x.stream);
  });
}
// (dout, q, k, v, out, lse, off, dq, dk, dv[, workspace])
PyObject *bwd_any(PyObject *const *args, Py_ssize_t n, bool has_ws) {
  return call([&]() -> int {
    Args x;
    s1f_desc d;
    if (!x.read(args, n, has_ws ? 11 : 10, 6, -1)) return kPython;
    auto &[dout, q, k, v, out, lse, dq, dk, dv, ws] = x.t;
    if (!same_layout(*q, *dout) || !same_layout(*q, *out) || !same_layout(*q, *dq) || !same_layout(*k, *v) || !acc_ok(*k, *dk, *dv) ||
        !lse_ok(*lse, *q) || !desc_of(*q, *k, &d) || !x.read_stream())
      return kPython;
    void *const p[] = {ptr(dout), ptr(q), ptr(k), ptr(v), ptr(out), ptr(lse), ptr(dq), ptr(dk), ptr(dv), has_ws ? ptr(ws) : nullptr};
    const float *l = static_cast<const float *>(p[5]);
    float *dkp = static_cast<float *>(p[7]), *dvp = static_cast<float *>(p[8]);
    const size_t ws_bytes = has_ws ? bytes(ws) : 0;
    Unlocked u;
    return has_ws ? api.bwd(&d, p[0], p[1], p[2], p[3], p[4], l, x.off, q->size(2), p[6], dkp, dvp, p[9], ws_bytes, x.stream)
                  : api.bwd_noalloc(&d, p[0], p[1], p[2], p[3], p[4], l, x.off, q->size(2), p[6], dkp, dvp, x.stream);
  });
}
PyObject *bwd(PyObject *, PyObject *const *args, Py_ssize_t n) { return bwd_any(args, n, true); }
PyObject *bwd_noalloc(PyObject *, PyObject *const *args, Py_ssize_t n) { return bwd_any(args, n, false); }
// (k_seg, v_seg, off, k_cache, v_cache)
PyObject *append(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return call([&]() -> int {
    Args x;
    s1f_desc d;
    if (!x.read(args, n, 5, 2, -1)) return kPython;
    auto &[ks, vs, kc, vc] = reinterpret_cast<const at::Tensor *(&)[4]>(x.t);
    if (!same_layout(*ks, *vs) || !same_layout(*kc, *vc) || !cache_desc_of(*kc, *kc, &d) || !segment_ok(*ks, *kc) ||
        ks->scalar_type() != kc->scalar_type() || !x.read_stream())
      return kPython;
    void *const p[] = {ptr(ks), ptr(vs), ptr(kc), ptr(vc)};
    Unlocked u;
    return api.append(&d, p[0], p[1], ks->stride(0), ks->stride(1), ks->stride(2), x.off, ks->size(2), p[2], p[3], x.stream);
  });
}
// (dk, dv, off, dk_seg, dv_seg)
PyObject *emit(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return call([&]() -> int {
    Args x;
    s1f_desc d;
    if (!x.read(args, n, 5, 2, -1)) return kPython;
    auto &[dk, dv, ks, vs] = reinterpret_cast<const at::Tensor *(&)[4]>(x.t);
    if (!same_layout(*dk, *dv) || !same_layout(*ks, *vs) || dk->scalar_type() != at::kFloat || !cache_desc_of(*dk, *ks, &d) ||
        !segment_ok(*ks, *dk) || !x.read_stream())
      return kPython;
    void *const p[] = {ptr(dk), ptr(dv), ptr(ks), ptr(vs)};
    Unlocked u;
    return api.emit(&d, static_cast<const float *>(p[0]), static_cast<const float *>(p[1]), x.off, ks->size(2), p[2], p[3], ks->stride(0),
                    ks->stride(1), ks->stride(2), x.stream);
  });
}
// (addresses of the six entry points, torch's functions for the current device and for a device's stream)
PyObject *bind(PyObject *, PyObject *args) {
  unsigned long long a[6];
  PyObject *dev, *st;
  if (!PyArg_ParseTuple(args, "KKKKKKOO", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &dev, &st)) return nullptr;
  api = Api{reinterpret_cast<decltype(api.fwd)>(a[0]),         reinterpret_cast<decltype(api.fwd_ws)>(a[1]),
            reinterpret_cast<decltype(api.bwd)>(a[2]),         reinterpret_cast<decltype(api.bwd_noalloc)>(a[3]),
            reinterpret_cast<decltype(api.append)>(a[4]),      reinterpret_cast<decltype(api.emit)>(a[5])};
  Py_INCREF(dev);
  Py_INCREF(st);
  Py_XDECREF(get_device);
  Py_XDECREF(get_stream);
  get_device = dev;
  get_stream = st;
  Py_RETURN_NONE;
}

#define S1F_METHOD(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f))
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"fwd", S1F_METHOD(fwd), METH_FASTCALL, nullptr},
                         {"fwd_ws", S1F_METHOD(fwd_ws), METH_FASTCALL, nullptr},
                         {"bwd", S1F_METHOD(bwd), METH_FASTCALL, nullptr},
                         {"bwd_noalloc", S1F_METHOD(bwd_noalloc), METH_FASTCALL, nullptr},
                         {"append", S1F_METHOD(append), METH_FASTCALL, nullptr},
                         {"emit", S1F_METHOD(emit), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_calls() {
  PyObject *m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) != 0) Py_CLEAR(m);
  return m;
}
