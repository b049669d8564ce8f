// binding.cpp - the common case of cmsd.py's calls, marshalled natively (CPython API and
// ATen, no HIP).  Each function takes the tensors and numbers of one call, checks them as
// cmsd.py does, and calls the C entry point (include/cmsd.h) whose address bind() was
// given.  It returns the status, or None when a check does not hold or an argument is not
// of the plain type: the caller then takes its Python path, which converts, allocates or
// raises.  Nothing is kept between calls.
//
// A call's Python marshalling (about 30 attribute reads and conversions through ctypes)
// took as long as the kernels of a small call; figures at cmsd.py's _native.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>

#include "cmsd.h"

namespace {

decltype(&cmsd_confidence) f_confidence;
decltype(&cmsd_confidence_var) f_confidence_var;
decltype(&cmsd_draft_len) f_draft_len;
decltype(&cmsd_draft_sample) f_draft_sample;
decltype(&cmsd_verify) f_verify;
decltype(&cmsd_logit_pass) f_logit_pass;
decltype(&cmsd_logit_pass_fused) f_logit_pass_fused;

// Arguments in order; ok turns false at the first that does not fit.
struct Args {
  PyObject* const* a;
  Py_ssize_t n, i = 0;
  bool ok = true;

  PyObject* next() {
    if (i >= n) {
      ok = false;
      return Py_None;
    }
    return a[i++];
  }
  const at::Tensor* tensor() {
    PyObject* o = next();
    if (!ok || !THPVariable_CheckExact(o)) {
      ok = false;
      return nullptr;
    }
    return &THPVariable_Unpack(o);
  }
  int64_t integer() {
    PyObject* o = next();
    if (!ok || !PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    if (over) ok = false;
    return v;
  }
  int32_t int32() {
    const int64_t v = integer();
    if (v < INT32_MIN || v > INT32_MAX) ok = false;
    return (int32_t)v;
  }
  float number() { return as_float(next()); }
  float as_float(PyObject* o) {
    if (!ok || !PyFloat_CheckExact(o)) {
      ok = false;
      return 0.f;
    }
    return (float)PyFloat_AS_DOUBLE(o);
  }
  void* stream() { return reinterpret_cast<void*>(integer()); }
  cmsd_conf_params conf() {  // lambdas, beta_margin
    cmsd_conf_params p{};
    PyObject* l = next();
    if (!ok || !PyTuple_CheckExact(l) || PyTuple_GET_SIZE(l) < 3) {
      ok = false;
      return p;
    }
    p.lambda_ent = as_float(PyTuple_GET_ITEM(l, 0));
    p.lambda_margin = as_float(PyTuple_GET_ITEM(l, 1));
    p.lambda_soft = as_float(PyTuple_GET_ITEM(l, 2));
    p.beta_margin = number();
    return p;
  }
};

// A [rows, vocab] logit matrix on the GPU with unit inner stride.
struct Rows {
  void* p = nullptr;
  int32_t dtype = 0;
  int64_t n = 0, vocab = 0, stride = 0;
  c10::Device dev = c10::Device(c10::kCPU);

  Rows(Args& a) {
    const at::Tensor* t = a.tensor();
    if (!a.ok) return;
    const auto st = t->scalar_type();
    if (!t->is_cuda() || t->dim() != 2 || t->stride(1) != 1 || (st != at::kFloat && st != at::kBFloat16)) {
      a.ok = false;
      return;
    }
    dtype = st == at::kFloat ? CMSD_F32 : CMSD_BF16;
    n = t->size(0);
    vocab = t->size(1);
    stride = t->stride(0);
    dev = t->device();
    p = t->data_ptr();
  }
};

// A contiguous buffer of at least `least` elements on `dev`.
void* buffer(Args& a, at::ScalarType type, int64_t least, const c10::Device& dev) {
  const at::Tensor* t = a.tensor();
  if (!a.ok) return nullptr;
  if (t->scalar_type() != type || !t->is_contiguous() || t->numel() < least || t->device() != dev) {
    a.ok = false;
    return nullptr;
  }
  return t->data_ptr();
}
template <typename T>
T* buffer_of(Args& a, int64_t least, const c10::Device& dev);
template <>
float* buffer_of<float>(Args& a, int64_t least, const c10::Device& dev) {
  return static_cast<float*>(buffer(a, at::kFloat, least, dev));
}
template <>
int32_t* buffer_of<int32_t>(Args& a, int64_t least, const c10::Device& dev) {
  return static_cast<int32_t*>(buffer(a, at::kInt, least, dev));
}
float* floats_or_none(Args& a, int64_t least, const c10::Device& dev) {
  if (a.ok && a.i < a.n && a.a[a.i] == Py_None) {
    ++a.i;
    return nullptr;
  }
  return buffer_of<float>(a, least, dev);
}
void* workspace(Args& a, size_t& bytes, const c10::Device& dev) {
  const Py_ssize_t at = a.i;
  void* p = buffer(a, at::kDouble, 0, dev);
  if (a.ok) bytes = 8 * (size_t)THPVariable_Unpack(a.a[at]).numel();
  return p;
}
cmsd_row_stats* stats_of(Args& a, int64_t rows, const c10::Device& dev) {
  return reinterpret_cast<cmsd_row_stats*>(buffer_of<float>(a, 8 * rows, dev));
}

// The call itself without the interpreter lock (a full stream queue can block it).
template <typename F>
PyObject* answer(const Args& a, F&& call) {
  if (!a.ok || a.i != a.n) Py_RETURN_NONE;
  cmsd_status s;
  Py_BEGIN_ALLOW_THREADS
  s = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(s);
}
// ATen throws where a tensor has no plain storage: the Python path reports it.
template <typename F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyObject* confidence(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&] {
    Args a{args, n};
    const Rows x(a);
    cmsd_row_stats* stats = stats_of(a, x.n, x.dev);
    const cmsd_conf_params p = a.conf();
    void* st = a.stream();
    return answer(a, [&] { return f_confidence(x.p, x.dtype, x.n, x.vocab, x.stride, &p, stats, st); });
  });
}

PyObject* confidence_var(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&] {
    Args a{args, n};
    const Rows x(a);
    cmsd_row_stats* stats = stats_of(a, x.n, x.dev);
    float* var = buffer_of<float>(a, x.n, x.dev);
    const cmsd_conf_params p = a.conf();
    void* st = a.stream();
    return answer(a, [&] { return f_confidence_var(x.p, x.dtype, x.n, x.vocab, x.stride, &p, stats, var, st); });
  });
}

PyObject* draft_len(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args a{args, n};
    const int32_t batch = a.int32();
    cmsd_draft_params p{};
    p.k_min = a.int32();
    p.k_max = a.int32();
    p.alpha = a.number();
    if (!a.ok || a.i >= n || !THPVariable_CheckExact(args[a.i])) Py_RETURN_NONE;
    const at::Tensor& s = THPVariable_Unpack(args[a.i]);
    if (!s.is_cuda()) Py_RETURN_NONE;
    const c10::Device dev = s.device();
    cmsd_row_stats* stats = stats_of(a, (int64_t)batch * p.k_max, dev);
    int32_t* k = buffer_of<int32_t>(a, batch, dev);
    int32_t* off = buffer_of<int32_t>(a, (int64_t)batch + 1, dev);
    void* st = a.stream();
    return answer(a, [&] { return f_draft_len(stats, batch, &p, k, off, st); });
  });
}

PyObject* draft_sample(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&] {
    Args a{args, n};
    const Rows x(a);
    cmsd_row_stats* stats = stats_of(a, x.n, x.dev);
    float* u = buffer_of<float>(a, x.n, x.dev);
    int32_t* y = buffer_of<int32_t>(a, x.n, x.dev);
    size_t bytes = 0;
    void* ws = workspace(a, bytes, x.dev);
    void* st = a.stream();
    return answer(a, [&] { return f_draft_sample(x.p, x.dtype, x.n, x.vocab, x.stride, stats, u, y, ws, bytes, st); });
  });
}

PyObject* verify(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&] {
    Args a{args, n};
    const int32_t batch = a.int32(), k_max = a.int32();
    const int64_t drows = (int64_t)batch * k_max;
    cmsd_verify_params p{};
    p.mode = a.int32();
    p.top_beta = a.int32();
    p.tau_base = a.number();
    p.gamma = a.number();
    const Rows d(a), t(a);
    a.ok = a.ok && d.vocab == t.vocab && d.dtype == t.dtype && d.dev == t.dev && d.n >= drows;
    cmsd_row_stats* stats = stats_of(a, drows, t.dev);
    int32_t* off = buffer_of<int32_t>(a, (int64_t)batch + 1, t.dev);
    int32_t* k = buffer_of<int32_t>(a, batch, t.dev);
    int32_t* drafted = buffer_of<int32_t>(a, drows, t.dev);
    float* u = floats_or_none(a, t.n, t.dev);
    cmsd_target_stats* ts = reinterpret_cast<cmsd_target_stats*>(buffer_of<float>(a, 8 * t.n, t.dev));
    int32_t* n_acc = buffer_of<int32_t>(a, batch, t.dev);
    int32_t* next = buffer_of<int32_t>(a, batch, t.dev);
    size_t bytes = 0;
    void* ws = workspace(a, bytes, t.dev);
    void* st = a.stream();
    return answer(a, [&] {
      return f_verify(d.p, d.stride, stats, t.p, t.stride, t.n, off, k, drafted, u, t.dtype, batch, k_max, t.vocab, &p,
                      ts, n_acc, next, ws, bytes, st);
    });
  });
}

// cmsd_logit_pass and cmsd_logit_pass_fused take the same arguments.
PyObject* pass(decltype(f_logit_pass) f, PyObject* const* args, Py_ssize_t n) {
  return guarded([&] {
    Args a{args, n};
    const int32_t batch = a.int32(), k_max = a.int32(), adaptive = a.int32();
    const int64_t drows = (int64_t)batch * k_max, trows = (int64_t)batch * ((int64_t)k_max + 1);
    const cmsd_conf_params cp = a.conf();
    cmsd_draft_params dp{};
    dp.k_min = a.int32();
    dp.k_max = k_max;
    dp.alpha = a.number();
    cmsd_verify_params vp{};
    vp.mode = a.int32();
    vp.top_beta = a.int32();
    vp.tau_base = a.number();
    vp.gamma = a.number();
    const Rows d(a), t(a);
    a.ok = a.ok && d.vocab == t.vocab && d.dtype == t.dtype && d.dev == t.dev && d.n >= drows && t.n >= trows;
    int32_t* drafted = buffer_of<int32_t>(a, drows, t.dev);
    float* u = floats_or_none(a, trows, t.dev);
    cmsd_row_stats* stats = stats_of(a, drows, t.dev);
    int32_t* k = buffer_of<int32_t>(a, batch, t.dev);
    cmsd_target_stats* ts = reinterpret_cast<cmsd_target_stats*>(buffer_of<float>(a, 8 * trows, t.dev));
    int32_t* n_acc = buffer_of<int32_t>(a, batch, t.dev);
    int32_t* next = buffer_of<int32_t>(a, batch, t.dev);
    size_t bytes = 0;
    void* ws = workspace(a, bytes, t.dev);
    void* st = a.stream();
    return answer(a, [&] {
      return f(d.p, d.stride, t.p, t.stride, drafted, u, t.dtype, batch, k_max, t.vocab, &cp, &dp, &vp, adaptive, stats,
               k, ts, n_acc, next, ws, bytes, st);
    });
  });
}
PyObject* logit_pass(PyObject*, PyObject* const* args, Py_ssize_t n) { return pass(f_logit_pass, args, n); }
PyObject* logit_pass_fused(PyObject*, PyObject* const* args, Py_ssize_t n) { return pass(f_logit_pass_fused, args, n); }

// bind(addresses): the entry points' addresses in the library that cmsd.py loaded, in the
// order below.
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 7) {
    PyErr_SetString(PyExc_TypeError, "bind takes 7 addresses");
    return nullptr;
  }
  void* p[7];
  for (int i = 0; i < 7; ++i) {
    p[i] = PyLong_AsVoidPtr(args[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  f_confidence = reinterpret_cast<decltype(f_confidence)>(p[0]);
  f_confidence_var = reinterpret_cast<decltype(f_confidence_var)>(p[1]);
  f_draft_len = reinterpret_cast<decltype(f_draft_len)>(p[2]);
  f_draft_sample = reinterpret_cast<decltype(f_draft_sample)>(p[3]);
  f_verify = reinterpret_cast<decltype(f_verify)>(p[4]);
  f_logit_pass = reinterpret_cast<decltype(f_logit_pass)>(p[5]);
  f_logit_pass_fused = reinterpret_cast<decltype(f_logit_pass_fused)>(p[6]);
  Py_RETURN_NONE;
}

#define CMSD_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CMSD_METHOD(bind),         CMSD_METHOD(confidence), CMSD_METHOD(confidence_var),
                         CMSD_METHOD(draft_len),    CMSD_METHOD(draft_sample), CMSD_METHOD(verify),
                         CMSD_METHOD(logit_pass),   CMSD_METHOD(logit_pass_fused), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
