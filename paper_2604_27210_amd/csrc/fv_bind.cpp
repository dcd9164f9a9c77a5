// fv_bind.cpp -- marshalling of torch tensors to the C ABI of fastvol.h.
//
// A call on few quotes costs what the host spends around one launch of 4 us:
// field checks, two output tensors and the argument block.  Through
// interpreted checks and ctypes structures that was 9.7 of 13.3 us for 4,096
// quotes (checks 3.4, structure 1.7, outputs 2.6, ctypes 0.8); here they are
// direct reads of the tensors' own fields: 5.4 us, of which the launch is 2.8.
// Only marshalling lives here: the addresses of the library's functions come
// from the loader, which owns the choice of the library.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/fastvol.h"

namespace {

// The library's functions, in the order in which init() receives them.
enum Fn : int {
  kIv, kPrice, kGreeks, kIvBackward, kPriceBackward, kLbrTrace, kHalleyTrace, kIvF32, kChains,
  kLastError, kFnCount
};
const char* const kFnName[kFnCount] = {
    "fv_implied_vol", "fv_price",       "fv_greeks",       "fv_implied_vol_backward",
    "fv_price_backward", "fv_lbr_trace", "fv_halley_trace", "fv_implied_vol_f32",
    "fv_implied_vol_chains", "fv_last_error"};
void* g_fn[kFnCount];
PyObject* g_error = nullptr;   // the package's exception class
PyObject* g_stream = nullptr;  // device ordinal -> raw handle of its current stream

template <class F>
F fn(int which) {
  return reinterpret_cast<F>(g_fn[which]);
}

// A Python exception is set.
struct Raised {};

[[noreturn]] void raise(PyObject* type, const char* fmt, const char* name) {
  PyErr_Format(type, fmt, name);
  throw Raised{};
}

[[noreturn]] void raise_got(PyObject* type, const char* fmt, const char* name, PyObject* v,
                            const char* attr) {
  PyObject* got = PyObject_GetAttrString(v, attr);
  if (got) PyErr_Format(type, fmt, name, got);
  Py_XDECREF(got);
  throw Raised{};
}

const at::Tensor* as_tensor(PyObject* v) {
  return THPVariable_Check(v) ? &THPVariable_Unpack(v) : nullptr;
}

// On the GPU, of the given type, contiguous.
const at::Tensor& dev_tensor(PyObject* v, const char* name, at::ScalarType type) {
  const at::Tensor* t = as_tensor(v);
  if (!t) raise(PyExc_TypeError, "%s must be a tensor", name);
  if (!t->is_cuda())
    raise_got(PyExc_ValueError, "%s must be on the GPU (got %S)", name, v, "device");
  if (t->scalar_type() != type) {
    const char* want = type == at::kDouble  ? "%s must be torch.float64 (got %S)"
                       : type == at::kFloat ? "%s must be torch.float32 (got %S)"
                       : type == at::kLong  ? "%s must be torch.int64 (got %S)"
                                            : "%s must be torch.int8 (got %S)";
    raise_got(PyExc_TypeError, want, name, v, "dtype");
  }
  if (!t->is_contiguous()) raise(PyExc_ValueError, "%s must be contiguous", name);
  return *t;
}

// The same with an entry for each of n quotes at least (a 0-dim tensor, which a
// field reads as a number, has one).
const at::Tensor& whole_tensor(PyObject* v, const char* name, at::ScalarType type, int64_t n) {
  const at::Tensor& t = dev_tensor(v, name, type);
  if (t.numel() < n) {
    PyErr_Format(PyExc_ValueError, "length mismatch: %s has %lld, expected %lld", name,
                 (long long)t.numel(), (long long)n);
    throw Raised{};
  }
  return t;
}

void* ptr(const at::Tensor& t) { return t.data_ptr(); }

double number(PyObject* v) {
  PyObject* f = PyNumber_Float(v);
  if (!f) throw Raised{};
  const double x = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return x;
}

int integer(PyObject* v) {
  const long x = PyLong_AsLong(v);
  if (x == -1 && PyErr_Occurred()) throw Raised{};
  return (int)x;
}

// The length and device that a call's per-quote tensors share.
struct Batch {
  int64_t n = -1;
  int device = -1;

  // A per-quote field: None (absent), a number for all quotes, or a 1-D
  // tensor.
  template <class ARG>
  ARG field(PyObject* v, const char* name) {
    constexpr at::ScalarType type =
        std::is_same<ARG, fv_arg_f32>::value ? at::kFloat : at::kDouble;
    ARG a{};
    if (v == Py_None) return a;
    const at::Tensor* t = as_tensor(v);
    if (!t || t->dim() == 0) {
      a.value = (decltype(a.value))number(v);
      return a;
    }
    if (t->dim() != 1) raise(PyExc_ValueError, "%s must be 1-D", name);
    dev_tensor(v, name, type);
    const int64_t m = t->numel();
    if (n < 0) {
      n = m;
      device = t->get_device();
    } else if (m != n) {
      PyErr_Format(PyExc_ValueError, "length mismatch: %s has %lld, expected %lld", name,
                   (long long)m, (long long)n);
      throw Raised{};
    }
    a.ptr = (decltype(a.ptr))ptr(*t);
    return a;
  }

  void some() const {
    if (n < 0)
      raise(PyExc_ValueError, "at least one per-quote field must be a 1-D GPU %s", "tensor");
  }

  // 'c'/'p', +1/-1, or an int8 tensor.
  void flag(PyObject* v, const int8_t*& p, int8_t& value) const {
    p = nullptr;
    value = 1;
    if (PyUnicode_Check(v)) {
      const char* s = PyUnicode_AsUTF8(v);
      if (!s) throw Raised{};
      value = s[0] == 'c' || s[0] == 'C' ? 1 : -1;
      return;
    }
    if (PyLong_Check(v) || PyFloat_Check(v)) {
      PyObject* i = PyNumber_Long(v);
      if (!i) throw Raised{};
      value = (int8_t)PyLong_AsUnsignedLongLongMask(i);
      Py_DECREF(i);
      return;
    }
    const at::Tensor* t = as_tensor(v);
    if (!t || t->dim() == 0)
      raise(PyExc_TypeError, "flag must be 'c'/'p', +1/-1 or an int8 GPU %s", "tensor");
    if (t->scalar_type() != at::kChar)
      raise(PyExc_TypeError, "flag tensor must be int8 (+1 call / -1 put)%s", "");
    dev_tensor(v, "flag", at::kChar);
    if (t->numel() != n) raise(PyExc_ValueError, "flag length mismatch%s", "");
    p = (const int8_t*)ptr(*t);
  }

  at::TensorOptions like(at::ScalarType type) const {
    return at::TensorOptions().dtype(type).device(at::Device(at::kCUDA, (c10::DeviceIndex)device));
  }
  at::Tensor empty(at::ScalarType type) const { return at::empty({n}, like(type)); }
  at::Tensor rows(int count) const { return at::empty({count, n}, like(at::kDouble)); }
};

// Other Python threads run during the allocations and the launch.
struct NoGil {
  PyThreadState* const state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

void* stream_of(PyObject* given, int device) {
  PyObject* s = given;
  if (given == Py_None) {
    s = PyObject_CallFunction(g_stream, "i", device);
    if (!s) throw Raised{};
  }
  void* p = PyLong_AsVoidPtr(s);
  if (s != given) Py_DECREF(s);
  if (!p && PyErr_Occurred()) throw Raised{};
  return p;
}

void check(int rc, int which) {
  if (rc == FV_OK) return;
  PyErr_Format(g_error, "%s failed (%d): %s", kFnName[which], rc,
               fn<const char* (*)()>(kLastError)());
  throw Raised{};
}

double* row(const at::Tensor& t, int64_t n, int i) { return (double*)ptr(t) + i * n; }

PyObject* wrap(const at::Tensor& t) {
  PyObject* o = THPVariable_Wrap(t);
  if (!o) throw Raised{};
  return o;
}

PyObject* dict_of_rows(const at::Tensor& t, const char* const* names, int count) {
  PyObject* d = PyDict_New();
  if (!d) throw Raised{};
  for (int i = 0; i < count; ++i) {
    PyObject* o = THPVariable_Wrap(t.select(0, i));
    if (!o || PyDict_SetItemString(d, names[i], o) != 0) {
      Py_XDECREF(o);
      Py_DECREF(d);
      throw Raised{};
    }
    Py_DECREF(o);
  }
  return d;
}

const char* const kGreekNames[] = {"delta", "gamma", "vega", "theta", "rho"};
const char* const kIvGradNames[] = {"price", "fs", "K", "T", "r", "q"};
const char* const kPriceGradNames[] = {"fs", "K", "T", "r", "q", "sigma"};

// What implied_vol returns: a sigma alone or a tuple; kGreekBlock leaves the
// Greeks as the one [5, n] tensor.
enum Option : int { kStatus = 1, kWithGreeks = 2, kGreekBlock = 4 };

// flat(function, model, solver, price, fs, K, T, r, q, sigma, grad, flag,
//      option or out, stream)
PyObject* flat(PyObject* const* a) {
  const int which = integer(a[0]), model = integer(a[1]), solver = integer(a[2]);
  Batch b;
  fv_quotes q{};
  q.price = b.field<fv_arg>(a[3], "price");
  q.fs = b.field<fv_arg>(a[4], "fs");
  q.K = b.field<fv_arg>(a[5], "K");
  q.T = b.field<fv_arg>(a[6], "T");
  q.r = b.field<fv_arg>(a[7], "r");
  q.q = b.field<fv_arg>(a[8], "q");
  const fv_arg sigma = b.field<fv_arg>(a[9], "sigma");
  if (which == kPriceBackward) b.field<fv_arg>(a[10], "grad_price");
  b.some();
  q.n = b.n;
  b.flag(a[11], q.flag, q.flag_value);
  const double *sig = nullptr, *grad = nullptr;
  if (which == kIvBackward)
    sig = (const double*)ptr(whole_tensor(a[9], "sigma", at::kDouble, b.n));
  if (which == kIvBackward || which == kPriceBackward)
    grad = (const double*)ptr(whole_tensor(
        a[10], which == kIvBackward ? "grad_sigma" : "grad_price", at::kDouble, b.n));
  at::Tensor out, status, block;
  int option = 0;
  if (which == kIv) option = integer(a[12]);
  if (which == kPrice && a[12] != Py_None) out = whole_tensor(a[12], "out", at::kDouble, b.n);
  void* s = stream_of(a[13], b.device);
  int rc = 0;
  {
    const NoGil free;
    switch (which) {
      case kIv: {
        out = b.empty(at::kDouble);
        if (option & kStatus) status = b.empty(at::kByte);
        double* g[5];
        if (option & kWithGreeks) {
          block = b.rows(5);
          for (int i = 0; i < 5; ++i) g[i] = row(block, b.n, i);
        }
        rc = fn<decltype(&fv_implied_vol)>(kIv)(
            model, solver, &q, (double*)ptr(out),
            option & kStatus ? (uint8_t*)ptr(status) : nullptr,
            option & kWithGreeks ? g : nullptr, s);
        break;
      }
      case kPrice:
        if (!out.defined()) out = b.empty(at::kDouble);
        rc = fn<decltype(&fv_price)>(kPrice)(model, &q, sigma, (double*)ptr(out), s);
        break;
      case kGreeks: {
        block = b.rows(5);
        const auto g = [&](int i) { return row(block, b.n, i); };
        rc = fn<decltype(&fv_greeks)>(kGreeks)(model, &q, sigma, g(0), g(1), g(2), g(3), g(4), s);
        break;
      }
      case kIvBackward: {
        block = b.rows(6);
        const auto g = [&](int i) { return row(block, b.n, i); };
        rc = fn<decltype(&fv_implied_vol_backward)>(kIvBackward)(
            model, &q, sig, grad, g(0), g(1), g(2), g(3), g(4), g(5), s);
        break;
      }
      case kPriceBackward: {
        block = b.rows(6);
        const auto g = [&](int i) { return row(block, b.n, i); };
        rc = fn<decltype(&fv_price_backward)>(kPriceBackward)(
            model, &q, sigma, grad, g(0), g(1), g(2), g(3), g(4), g(5), s);
        break;
      }
      case kLbrTrace:
      case kHalleyTrace:
        out = b.empty(at::kInt);
        rc = fn<decltype(&fv_lbr_trace)>(which)(model, &q, (uint32_t*)ptr(out), s);
        break;
    }
  }
  check(rc, which);
  switch (which) {
    case kGreeks: return dict_of_rows(block, kGreekNames, 5);
    case kIvBackward: return dict_of_rows(block, kIvGradNames, 6);
    case kPriceBackward: return dict_of_rows(block, kPriceGradNames, 6);
    case kPrice:
      if (a[12] != Py_None) {
        Py_INCREF(a[12]);
        return a[12];
      }
      return wrap(out);
    case kIv: break;
    default: return wrap(out);
  }
  if (option == 0) return wrap(out);
  const int count = 1 + (option & kStatus ? 1 : 0) + (option & kWithGreeks ? 1 : 0);
  PyObject* res = PyTuple_New(count);
  if (!res) throw Raised{};
  try {
    int i = 0;
    PyTuple_SET_ITEM(res, i++, wrap(out));
    if (option & kStatus) PyTuple_SET_ITEM(res, i++, wrap(status));
    if (option & kWithGreeks)
      PyTuple_SET_ITEM(res, i, option & kGreekBlock ? wrap(block)
                                                    : dict_of_rows(block, kGreekNames, 5));
  } catch (...) {
    Py_DECREF(res);
    throw;
  }
  return res;
}

PyObject* sigma_and_status(const at::Tensor& sigma, const at::Tensor& status) {
  if (!status.defined()) return wrap(sigma);
  PyObject* res = PyTuple_New(2);
  if (!res) throw Raised{};
  try {
    PyTuple_SET_ITEM(res, 0, wrap(sigma));
    PyTuple_SET_ITEM(res, 1, wrap(status));
  } catch (...) {
    Py_DECREF(res);
    throw;
  }
  return res;
}

// flat_f32(model, price, fs, K, T, r, q, flag, with_status, stream)
PyObject* flat_f32(PyObject* const* a) {
  const int model = integer(a[0]);
  Batch b;
  fv_quotes_f32 q{};
  q.price = b.field<fv_arg_f32>(a[1], "price");
  q.fs = b.field<fv_arg_f32>(a[2], "fs");
  q.K = b.field<fv_arg_f32>(a[3], "K");
  q.T = b.field<fv_arg_f32>(a[4], "T");
  q.r = b.field<fv_arg_f32>(a[5], "r");
  q.q = b.field<fv_arg_f32>(a[6], "q");
  b.some();
  q.n = b.n;
  b.flag(a[7], q.flag, q.flag_value);
  const bool with_status = integer(a[8]) != 0;
  void* s = stream_of(a[9], b.device);
  at::Tensor sigma, status;
  int rc;
  {
    const NoGil free;
    sigma = b.empty(at::kFloat);
    if (with_status) status = b.empty(at::kByte);
    rc = fn<decltype(&fv_implied_vol_f32)>(kIvF32)(
        model, &q, (float*)ptr(sigma), with_status ? (uint8_t*)ptr(status) : nullptr, s);
  }
  check(rc, kIvF32);
  return sigma_and_status(sigma, status);
}

// chains(solver, chain_mat_off, mat_quote_off, F, r, T, price, K, flag,
//        with_status, stream)
PyObject* chains(PyObject* const* a) {
  const int solver = integer(a[0]);
  const at::Tensor& cmo = dev_tensor(a[1], "chain_mat_off", at::kLong);
  const at::Tensor& mqo = dev_tensor(a[2], "mat_quote_off", at::kLong);
  const at::Tensor& F = dev_tensor(a[3], "F", at::kDouble);
  const at::Tensor& r = dev_tensor(a[4], "r", at::kDouble);
  const at::Tensor& T = dev_tensor(a[5], "T", at::kDouble);
  const at::Tensor& price = dev_tensor(a[6], "price", at::kDouble);
  const at::Tensor& K = dev_tensor(a[7], "K", at::kDouble);
  const at::Tensor& flag = dev_tensor(a[8], "flag", at::kChar);
  if (cmo.numel() != F.numel() + 1 || mqo.numel() != T.numel() + 1)
    raise(PyExc_ValueError, "offset arrays must have n_chains+1 and n_maturities+1 %s", "entries");
  if (K.numel() != price.numel() || flag.numel() != price.numel() || r.numel() != F.numel())
    raise(PyExc_ValueError, "per-quote / per-chain array lengths %s", "disagree");
  const bool with_status = integer(a[9]) != 0;
  fv_chains c{};
  c.n_chains = F.numel();
  c.n_maturities = T.numel();
  c.n_quotes = price.numel();
  c.chain_mat_off = (const int64_t*)ptr(cmo);
  c.mat_quote_off = (const int64_t*)ptr(mqo);
  c.F = (const double*)ptr(F);
  c.r = (const double*)ptr(r);
  c.T = (const double*)ptr(T);
  c.price = (const double*)ptr(price);
  c.K = (const double*)ptr(K);
  c.flag = (const int8_t*)ptr(flag);
  Batch b;
  b.n = c.n_quotes;
  b.device = price.get_device();
  void* s = stream_of(a[10], b.device);
  at::Tensor sigma, status;
  int rc;
  {
    const NoGil free;
    sigma = b.empty(at::kDouble);
    if (with_status) status = b.empty(at::kByte);
    rc = fn<decltype(&fv_implied_vol_chains)>(kChains)(
        solver, &c, (double*)ptr(sigma), with_status ? (uint8_t*)ptr(status) : nullptr, s);
  }
  check(rc, kChains);
  return sigma_and_status(sigma, status);
}

// init((addresses in the order of Fn), exception class, stream function)
PyObject* init(PyObject* const* a) {
  if (!PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != kFnCount)
    raise(PyExc_ValueError, "init takes the addresses of the library's %s", "functions");
  for (int i = 0; i < kFnCount; ++i) {
    g_fn[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[0], i));
    if (!g_fn[i]) raise(PyExc_ValueError, "%s has no address", kFnName[i]);
  }
  Py_INCREF(a[1]);
  Py_INCREF(a[2]);
  Py_XDECREF(g_error);
  Py_XDECREF(g_stream);
  g_error = a[1];
  g_stream = a[2];
  Py_RETURN_NONE;
}

// No C++ exception leaves through the interpreter.
template <PyObject* (*BODY)(PyObject* const*), int COUNT>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != COUNT) {
    PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", COUNT, nargs);
    return nullptr;
  }
  try {
    return BODY(args);
  } catch (const Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

template <PyObject* (*BODY)(PyObject* const*), int COUNT>
constexpr PyMethodDef method(const char* name) {
  return {name, (PyCFunction)(void*)&entry<BODY, COUNT>, METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method<init, 3>("init"), method<flat, 14>("flat"),
                         method<flat_f32, 10>("flat_f32"), method<chains, 11>("chains"),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "fv_bind", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_fv_bind() { return PyModule_Create(&module); }
