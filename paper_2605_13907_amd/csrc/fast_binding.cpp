// The binding's calls without the interpreter: argument checks, output tensors and the call of the C ABI.
//
// A step of the smallest batches was bound by the host: of the 40 us of a step over 512 rows, whose kernels then took 24 (22
// since the gradient sweep forms the coefficients of such batches itself), most went into some twenty argument checks, eight
// output tensors and three calls through ctypes.  Every function here does what the method of the same name in binding.py
// does when nothing is wrong with its arguments, and returns None otherwise: the caller then takes the method's own way,
// which raises what it always raised.  A failing call of the library returns its error code.  us a call, method and here:
// token_logprob 9.0 and 5.4, diagnostics 11.1 and 7.7 (its kernel's), grpo_loss_grad 17.3 and 10.7, grpo_row_scale 11.9 and
// 7.1; the step 40 and 24.  Only plain tensors with storage are taken (no subclasses, no wrappers of transforms).
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>

#include <algorithm>

#include "ais.h"

namespace {

// The library's entry points, as binding.py has loaded them.
struct Library {
  decltype(&ais_set_stream) set_stream;
  decltype(&ais_token_logprob) token_logprob;
  decltype(&ais_diagnostics) diagnostics;
  decltype(&ais_grpo_loss_grad) grpo_loss_grad;
  decltype(&ais_grpo_row_scale) grpo_row_scale;
  decltype(&ais_token_logprob_softmax_grad) token_logprob_softmax_grad;
  decltype(&ais_fp8_quantize_rows) fp8_quantize_rows;
  decltype(&ais_fp8_dequantize_rows) fp8_dequantize_rows;
  decltype(&ais_fp8_rollout_logprob) fp8_rollout_logprob;
  decltype(&ais_lm_head_logprob) lm_head_logprob;
  decltype(&ais_lm_head_grad) lm_head_grad;
} lib;

// Reads positional arguments; `ok` turns false at the first one that is not what the call takes.
struct Args {
  PyObject* const* a;
  Py_ssize_t n;
  bool ok = true;
  int device = -1;
  Py_ssize_t at = 0;

  PyObject* next() {
    if (at >= n) {
      ok = false;
      return nullptr;
    }
    return a[at++];
  }
  long long integer() {
    PyObject* o = next();
    if (o == nullptr || !PyLong_CheckExact(o)) return ok = false, 0;
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return v;
  }
  double real() {
    PyObject* o = next();
    if (o == nullptr || !PyFloat_CheckExact(o)) return ok = false, 0.0;
    return PyFloat_AS_DOUBLE(o);
  }
  void* pointer() {
    PyObject* o = next();
    if (o == nullptr || !PyLong_CheckExact(o)) return ok = false, nullptr;
    void* p = PyLong_AsVoidPtr(o);
    if (p == nullptr && PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return p;
  }
  // A tensor on the context's GPU, or null.
  const at::Tensor* tensor() {
    PyObject* o = next();
    if (o == nullptr || !THPVariable_CheckExact(o)) return ok = false, nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || t.layout() != at::kStrided || !t.is_cuda() || t.get_device() != device ||
        t.is_conj() || t.is_neg())
      return ok = false, nullptr;
    return &t;
  }
  // The address of a contiguous array of n elements, null for None where that is allowed.
  template <typename T>
  T* array(at::ScalarType type, long long count, bool none_allowed = false) {
    if (at < n && a[at] == Py_None && none_allowed) {
      ++at;
      return nullptr;
    }
    const at::Tensor* t = tensor();
    if (t == nullptr || t->scalar_type() != type || !t->is_contiguous() || t->numel() != count) return ok = false, nullptr;
    return static_cast<T*>(t->data_ptr());
  }
};

// A [rows, width] matrix with unit stride along its rows.
struct Matrix {
  const at::Tensor* t = nullptr;
  long long rows = 0, width = 0, stride = 0;
  ais_dtype dtype = AIS_BF16;
  explicit Matrix(Args& args) {
    t = args.tensor();
    if (t == nullptr) return;
    if (t->dim() != 2 || (t->stride(1) != 1 && t->size(1) > 1) ||
        (t->scalar_type() != at::kBFloat16 && t->scalar_type() != at::kFloat)) {
      args.ok = false;
      return;
    }
    dtype = t->scalar_type() == at::kBFloat16 ? AIS_BF16 : AIS_F32;
    rows = t->size(0);
    width = t->size(1);
    stride = rows > 1 ? t->stride(0) : std::max<long long>(width, t->stride(0));
  }
  void* data() const { return t->data_ptr(); }
  // a matrix laid out like this one: the caller's, or a new one for None
  at::Tensor like(Args& args) const {
    if (args.at < args.n && args.a[args.at] == Py_None) {
      ++args.at;
      return args.ok ? at::empty_strided(t->sizes(), t->strides(), t->options()) : at::Tensor();
    }
    const at::Tensor* o = args.tensor();
    if (o == nullptr || !args.ok) return at::Tensor();
    if (o->scalar_type() != t->scalar_type() || o->sizes() != t->sizes() || o->strides() != t->strides())
      return args.ok = false, at::Tensor();
    return *o;
  }
};

at::Tensor empty(int device, at::IntArrayRef sizes, at::ScalarType type = at::kFloat) {
  return at::empty(sizes, at::TensorOptions().dtype(type).device(at::Device(at::kCUDA, (at::DeviceIndex)device)));
}

template <typename... T>
PyObject* result(const T&... t) {
  PyObject* out = PyTuple_New(sizeof...(T));
  if (out == nullptr) return nullptr;
  Py_ssize_t i = 0;
  (PyTuple_SET_ITEM(out, i++, t.defined() ? THPVariable_Wrap(t) : (Py_INCREF(Py_None), Py_None)), ...);
  return out;
}

// What every call begins with: context handle, device index, stream.
struct Call : Args {
  ais_ctx* ctx;
  void* stream;
  Call(PyObject* const* a, Py_ssize_t n) : Args{a, n} {
    ctx = static_cast<ais_ctx*>(pointer());
    device = (int)integer();
    stream = pointer();
    ok = ok && ctx != nullptr;
  }
  // Runs `call` on the stream, without the interpreter's lock, which is taken again however that ends: the address of a
  // tensor's storage may be refused (a copy-on-write one has to be allocated first) with a C++ exception.
  template <typename F>
  int run(F call) {
    struct Unlocked {
      PyThreadState* state = PyEval_SaveThread();
      ~Unlocked() { PyEval_RestoreThread(state); }
    } unlocked;
    const int rc = lib.set_stream(ctx, stream);
    return rc == 0 ? call() : rc;
  }
};

#define AIS_REFUSE Py_RETURN_NONE
// C++ exceptions (an allocation that fails) become None too: the slow way then raises its own.
#define AIS_CALL(NAME)                                                          \
  PyObject* NAME##_body(Call& c);                                               \
  PyObject* NAME(PyObject*, PyObject* const* args, Py_ssize_t n) {              \
    try {                                                                       \
      Call c(args, n);                                                          \
      if (!c.ok) AIS_REFUSE;                                                    \
      return NAME##_body(c);                                                    \
    } catch (...) {                                                             \
      if (PyErr_Occurred()) PyErr_Clear();                                      \
      AIS_REFUSE;                                                               \
    }                                                                           \
  }                                                                             \
  PyObject* NAME##_body(Call& c)

AIS_CALL(token_logprob) {
  const Matrix z(c);
  if (!c.ok) AIS_REFUSE;
  const int* ids = c.array<int>(at::kInt, z.rows);
  const unsigned char* valid = c.array<unsigned char>(at::kByte, z.rows, true);
  const float inv_t = (float)c.real();
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor logp = empty(c.device, {z.rows}), lse = empty(c.device, {z.rows});
  float *lp = logp.data_ptr<float>(), *ls = lse.data_ptr<float>();
  const int rc = c.run([&] {
    return lib.token_logprob(c.ctx, z.data(), z.dtype, z.rows, z.width, z.stride, ids, valid, inv_t, lp, ls);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(logp, lse);
}

AIS_CALL(token_logprob_softmax_grad) {
  const Matrix z(c);
  if (!c.ok) AIS_REFUSE;
  const int* ids = c.array<int>(at::kInt, z.rows);
  const unsigned char* valid = c.array<unsigned char>(at::kByte, z.rows, true);
  const float inv_t = (float)c.real();
  if (!c.ok) AIS_REFUSE;
  const at::Tensor s = z.like(c);
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor logp = empty(c.device, {z.rows}), lse = empty(c.device, {z.rows});
  float *lp = logp.data_ptr<float>(), *ls = lse.data_ptr<float>();
  void* sp = s.data_ptr();
  const int rc = c.run([&] {
    return lib.token_logprob_softmax_grad(c.ctx, z.data(), z.dtype, z.rows, z.width, z.stride, ids, valid, inv_t, lp, ls,
                                          sp);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(logp, lse, s);
}

// The sizes of a batch of scalars: rows of `logp_train`, responses of `per_response`.
AIS_CALL(diagnostics) {
  const at::Tensor *train = c.tensor(), *rewards = nullptr;
  if (!c.ok) AIS_REFUSE;
  const long long rows = train->numel();
  --c.at;
  const float* lt = c.array<float>(at::kFloat, rows);
  const float* roll = c.array<float>(at::kFloat, rows);
  const unsigned char* valid = c.array<unsigned char>(at::kByte, rows, true);
  const Py_ssize_t cu_at = c.at++;
  rewards = c.tensor();
  if (!c.ok) AIS_REFUSE;
  const long long resp = rewards->numel();
  --c.at;
  const float* rw = c.array<float>(at::kFloat, resp);
  const Py_ssize_t after = c.at;
  c.at = cu_at;
  const long long* cu = reinterpret_cast<const long long*>(c.array<int64_t>(at::kLong, resp + 1));
  c.at = after;
  const long long group = c.integer();
  const ais_params* p = static_cast<const ais_params*>(c.pointer());
  if (!c.ok || c.at != c.n || p == nullptr || resp > 0x7fffffff || group != (int)group) AIS_REFUSE;
  const at::Tensor adv = empty(c.device, {resp}), count = empty(c.device, {resp}, at::kInt),
                   diag = empty(c.device, {(long long)sizeof(ais_diag)}, at::kByte);
  float* ap = adv.data_ptr<float>();
  int* cp = count.data_ptr<int>();
  ais_diag* dp = static_cast<ais_diag*>(diag.data_ptr());
  const int rc = c.run([&] {
    return lib.diagnostics(c.ctx, lt, roll, valid, rows, cu, (int)resp, (int)group, rw, p, ap, cp, dp);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(adv, count, diag);
}

// The arguments that the loss's two calls share, in their order.
struct LossArgs {
  const float *lt, *roll, *old, *ref, *adv;
  const int* count;
  const ais_diag* diag;
  const ais_params* p;
  const unsigned char* valid;
  const long long* cu;
  long long resp = 0;
  LossArgs(Call& c, long long rows) {
    lt = c.array<float>(at::kFloat, rows);
    roll = c.array<float>(at::kFloat, rows);
    valid = c.array<unsigned char>(at::kByte, rows, true);
    const Py_ssize_t cu_at = c.at++;
    const at::Tensor* a = c.tensor();
    if (!c.ok) return;
    resp = a->numel();
    if (resp > 0x7fffffff) c.ok = false;
    --c.at;
    adv = c.array<float>(at::kFloat, resp);
    const Py_ssize_t after = c.at;
    c.at = cu_at;
    cu = reinterpret_cast<const long long*>(c.array<int64_t>(at::kLong, resp + 1));
    c.at = after;
    count = c.array<int>(at::kInt, resp);
    diag = reinterpret_cast<const ais_diag*>(c.array<unsigned char>(at::kByte, sizeof(ais_diag)));
    p = static_cast<const ais_params*>(c.pointer());
    old = c.array<float>(at::kFloat, rows, true);
    ref = c.array<float>(at::kFloat, rows, true);
    if (p == nullptr) c.ok = false;
  }
};

AIS_CALL(grpo_loss_grad) {
  const Matrix z(c);
  if (!c.ok) AIS_REFUSE;
  const int* ids = c.array<int>(at::kInt, z.rows);
  const float* lse = c.array<float>(at::kFloat, z.rows);
  const bool want_wtilde = c.integer() != 0;
  if (!c.ok) AIS_REFUSE;
  const LossArgs l(c, z.rows);
  if (!c.ok) AIS_REFUSE;
  const at::Tensor dz = z.like(c);
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor wt = want_wtilde ? empty(c.device, {z.rows}) : at::Tensor(), loss = empty(c.device, {1}, at::kDouble);
  float* wp = want_wtilde ? wt.data_ptr<float>() : nullptr;
  double* lp = loss.data_ptr<double>();
  void* dp = dz.data_ptr();
  const int rc = c.run([&] {
    return lib.grpo_loss_grad(c.ctx, z.data(), z.dtype, z.rows, z.width, z.stride, ids, l.valid, l.cu, (int)l.resp, l.lt,
                              lse, l.roll, l.old, l.ref, l.adv, l.count, l.diag, l.p, wp, lp, dp);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(loss, wt, dz);
}

AIS_CALL(grpo_row_scale) {
  const at::Tensor* train = c.tensor();
  if (!c.ok) AIS_REFUSE;
  const long long rows = train->numel();
  --c.at;
  const LossArgs l(c, rows);
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor wt = empty(c.device, {rows}), g = empty(c.device, {rows}), loss = empty(c.device, {1}, at::kDouble);
  float *wp = wt.data_ptr<float>(), *gp = g.data_ptr<float>();
  double* lp = loss.data_ptr<double>();
  const int rc = c.run([&] {
    return lib.grpo_row_scale(c.ctx, l.lt, l.roll, l.old, l.ref, l.valid, rows, l.cu, (int)l.resp, l.adv, l.count, l.diag,
                              l.p, wp, lp, gp);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(loss, wt, g);
}

AIS_CALL(fp8_quantize_rows) {
  const Matrix z(c);
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor codes = empty(c.device, {z.rows, z.width}, at::kByte), scale = empty(c.device, {z.rows});
  unsigned char* cp = codes.data_ptr<unsigned char>();
  float* sp = scale.data_ptr<float>();
  const int rc = c.run([&] {
    return lib.fp8_quantize_rows(c.ctx, z.data(), z.dtype, z.rows, z.width, z.stride, cp, z.width, sp);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(codes, scale);
}

// codes, scale, 1 for a bf16 result or 0 for fp32
AIS_CALL(fp8_dequantize_rows) {
  const at::Tensor* codes = c.tensor();
  if (!c.ok || codes->dim() != 2 || (codes->stride(1) != 1 && codes->size(1) > 1) || codes->scalar_type() != at::kByte)
    AIS_REFUSE;
  const long long rows = codes->size(0), width = codes->size(1);
  const float* scale = c.array<float>(at::kFloat, rows);
  const bool bf16 = c.integer() != 0;
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor out = empty(c.device, {rows, width}, bf16 ? at::kBFloat16 : at::kFloat);
  const unsigned char* cp = static_cast<const unsigned char*>(codes->data_ptr());
  const long long stride = rows > 1 ? codes->stride(0) : width;
  void* op = out.data_ptr();
  const int rc = c.run([&] {
    return lib.fp8_dequantize_rows(c.ctx, cp, stride, scale, rows, width, op, bf16 ? AIS_BF16 : AIS_F32, width);
  });
  return rc != 0 ? PyLong_FromLong(rc) : THPVariable_Wrap(out);
}

AIS_CALL(fp8_rollout_logprob) {
  const Matrix z(c);
  if (!c.ok) AIS_REFUSE;
  const int* ids = c.array<int>(at::kInt, z.rows);
  const unsigned char* valid = c.array<unsigned char>(at::kByte, z.rows, true);
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor logp = empty(c.device, {z.rows});
  float* lp = logp.data_ptr<float>();
  const int rc = c.run([&] {
    return lib.fp8_rollout_logprob(c.ctx, z.data(), z.dtype, z.rows, z.width, z.stride, ids, valid, lp);
  });
  return rc != 0 ? PyLong_FromLong(rc) : THPVariable_Wrap(logp);
}

AIS_CALL(lm_head_logprob) {
  const Matrix h(c), w(c);
  if (!c.ok || h.dtype != AIS_BF16 || w.dtype != AIS_BF16 || h.width != w.width || h.t->stride(1) != 1 ||
      w.t->stride(1) != 1)
    AIS_REFUSE;
  const int* ids = c.array<int>(at::kInt, h.rows);
  const unsigned char* valid = c.array<unsigned char>(at::kByte, h.rows, true);
  const float inv_t = (float)c.real();
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor logp = empty(c.device, {h.rows}), lse = empty(c.device, {h.rows});
  float *lp = logp.data_ptr<float>(), *ls = lse.data_ptr<float>();
  const int rc = c.run([&] {
    return lib.lm_head_logprob(c.ctx, h.data(), h.stride, w.data(), w.stride, AIS_BF16, h.rows, h.width, w.rows, ids, valid,
                               inv_t, lp, ls);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(logp, lse);
}

AIS_CALL(lm_head_grad) {
  const Matrix h(c), w(c);
  if (!c.ok || h.dtype != AIS_BF16 || w.dtype != AIS_BF16 || h.width != w.width || h.t->stride(1) != 1 ||
      w.t->stride(1) != 1)
    AIS_REFUSE;
  const int* ids = c.array<int>(at::kInt, h.rows);
  const float* lse = c.array<float>(at::kFloat, h.rows);
  const float* logp = c.array<float>(at::kFloat, h.rows);
  const float* coeff = c.array<float>(at::kFloat, h.rows);
  const float inv_t = (float)c.real();
  const long long chunk = c.integer(), live = c.integer();
  if (!c.ok || c.at != c.n) AIS_REFUSE;
  const at::Tensor dh = empty(c.device, {h.rows, h.width}), dw = empty(c.device, {w.rows, w.width});
  float *hp = dh.data_ptr<float>(), *wp = dw.data_ptr<float>();
  const int rc = c.run([&] {
    return lib.lm_head_grad(c.ctx, h.data(), h.stride, w.data(), w.stride, AIS_BF16, h.rows, h.width, w.rows, ids, lse, logp,
                            coeff, inv_t, chunk, live, hp, wp);
  });
  return rc != 0 ? PyLong_FromLong(rc) : result(dh, dw);
}

// init(addresses): the entry points, in the order of Library.
PyObject* init(PyObject*, PyObject* const* args, Py_ssize_t n) {
  constexpr Py_ssize_t kEntries = sizeof(Library) / sizeof(void*);
  static_assert(sizeof(void (*)()) == sizeof(void*), "");
  if (n != kEntries) {
    PyErr_SetString(PyExc_TypeError, "init: one address for every entry point");
    return nullptr;
  }
  void* at[kEntries];
  for (Py_ssize_t i = 0; i < n; ++i) {
    at[i] = PyLong_AsVoidPtr(args[i]);
    if (at[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "init: a null address");
      return nullptr;
    }
  }
  std::copy(at, at + kEntries, reinterpret_cast<void**>(&lib));
  Py_RETURN_NONE;
}

#define AIS_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {AIS_METHOD(init),
                         AIS_METHOD(token_logprob),
                         AIS_METHOD(token_logprob_softmax_grad),
                         AIS_METHOD(diagnostics),
                         AIS_METHOD(grpo_loss_grad),
                         AIS_METHOD(grpo_row_scale),
                         AIS_METHOD(fp8_quantize_rows),
                         AIS_METHOD(fp8_dequantize_rows),
                         AIS_METHOD(fp8_rollout_logprob),
                         AIS_METHOD(lm_head_logprob),
                         AIS_METHOD(lm_head_grad),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ais_fast", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// `stamp`: of the sources and the torch that this was compiled from, which the binding compares before it calls anything.
PyMODINIT_FUNC PyInit__ais_fast(void) {
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "stamp", AIS_FAST_STAMP) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
