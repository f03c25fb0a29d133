// Host side of the per-call entry points of the Python binding (module
// _dptq_torch): checks the tensors, allocates the outputs the caller did not
// pass, and calls the C ABI on the current stream.  The same checks, in the
// same order and with the same errors, as the Python they replace; written
// against the CPython API and the tensor type directly because a pass of a few
// launches is bound by this work: two calls with fresh outputs took 24 us of
// host time in Python (interpreting the checks, two torch.empty, a stream
// object and the ctypes marshalling), of which the two launches are 6.6 us.

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <array>
#include <initializer_list>
#include <string>

#include "dptq.h"

namespace {

// Set by init(): raises DptqError(status, what); returns the raw stream of a
// device index.
PyObject* g_raise = nullptr;
PyObject* g_stream = nullptr;

// A Python error is set.
struct Raised {};

const char* dtype_name(at::ScalarType t) {
  switch (t) {
    case at::kHalf: return "torch.float16";
    case at::kFloat: return "torch.float32";
    case at::kDouble: return "torch.float64";
    case at::kByte: return "torch.uint8";
    case at::kChar: return "torch.int8";
    case at::kInt: return "torch.int32";
    default: return "?";
  }
}

[[noreturn]] void fail(PyObject* type, const std::string& msg) {
  PyErr_SetString(type, msg.c_str());
  throw Raised{};
}

std::string shape_text(at::IntArrayRef s) {
  std::string r = "(";
  for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
  return r + (s.size() == 1 ? ",)" : ")");
}

// The tensor o after its checks; shape only when `has_shape`.
const at::Tensor& tensor(PyObject* o, const char* name, at::ScalarType dtype, at::IntArrayRef shape = {},
                         bool has_shape = false) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, std::string(name) + " must be a torch.Tensor");
  const at::Tensor& t = THPVariable_Unpack(o);
  if (t.scalar_type() != dtype) {
    PyObject* d = PyObject_GetAttrString(o, "dtype");
    if (!d) throw Raised{};
    PyErr_Format(PyExc_TypeError, "%s must have dtype %s, got %S", name, dtype_name(dtype), d);
    Py_DECREF(d);
    throw Raised{};
  }
  if (!t.is_cuda()) fail(PyExc_ValueError, std::string(name) + " must be a GPU tensor");
  if (!t.is_contiguous()) fail(PyExc_ValueError, std::string(name) + " must be contiguous");
  if (has_shape && t.sizes() != shape)
    fail(PyExc_ValueError, std::string(name) + " must have shape " + shape_text(shape) + ", got " +
                               shape_text(t.sizes()));
  return t;
}

const at::Tensor& tensor_of(PyObject* o, const char* name, at::ScalarType dtype,
                            std::initializer_list<int64_t> shape) {
  return tensor(o, name, dtype, at::IntArrayRef(shape.begin(), shape.size()), true);
}

void two_d(const at::Tensor& t, const char* what) {
  if (t.dim() != 2) fail(PyExc_ValueError, what);
}

int64_t dim(const at::Tensor& t, int i) {
  if (i >= t.dim()) fail(PyExc_IndexError, "tuple index out of range");
  return t.size(i);
}

// An integer argument; any_number: also another number of an integer's value.
int64_t integer(PyObject* o, const char* name, bool any_number = false) {
  PyObject* n = PyIndex_Check(o) ? PyNumber_Index(o) : any_number && PyNumber_Check(o) ? PyNumber_Long(o) : nullptr;
  if (!n) {
    if (!PyErr_Occurred()) PyErr_Format(PyExc_TypeError, "%s must be an integer, got %R", name, o);
    throw Raised{};
  }
  const int eq = PyIndex_Check(o) ? 1 : PyObject_RichCompareBool(o, n, Py_EQ);
  const int64_t v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (PyErr_Occurred()) throw Raised{};
  if (eq != 1) {
    PyErr_Format(PyExc_ValueError, "%s must be an integer, got %R", name, o);
    throw Raised{};
  }
  return v;
}

// int(o) as a C int32 argument (taken modulo 2^32, as ctypes does).
int32_t integer32(PyObject* o) {
  if (PyLong_CheckExact(o)) return (int32_t)PyLong_AsUnsignedLongLongMask(o);
  PyObject* n = PyNumber_Long(o);
  if (!n) throw Raised{};
  const int32_t v = (int32_t)PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  return v;
}

// o == v, by value.
bool equals(PyObject* o, long v) {
  PyObject* n = PyLong_FromLong(v);
  const int eq = n ? PyObject_RichCompareBool(o, n, Py_EQ) : -1;
  Py_XDECREF(n);
  if (eq < 0) throw Raised{};
  return eq == 1;
}

int32_t bits_4_or_8(PyObject* o) {
  if (equals(o, 4)) return 4;
  if (equals(o, 8)) return 8;
  fail(PyExc_ValueError, "bits must be 4 or 8");
}

// Codes of the entry points that leave the check of bits to the library: packed
// where bits == 4, bytes for any other value.
at::ScalarType code_dtype(int32_t bits) { return bits == 4 ? at::kByte : at::kChar; }
int32_t code_bits(PyObject* bits) { return equals(bits, 4) ? 4 : 8; }

// The interpreter lock released for a scope, also when an exception leaves it.
class Unlocked {
 public:
  Unlocked() : state_(PyEval_SaveThread()) {}
  ~Unlocked() { PyEval_RestoreThread(state_); }
  Unlocked(const Unlocked&) = delete;

 private:
  PyThreadState* state_;
};

// An output: the caller's tensor after its checks, or a new one (allocate).
struct Out {
  PyObject* o = nullptr;   // a new reference
  at::Tensor t;
  std::array<int64_t, 2> shape{};
  int dims;
  at::TensorOptions options;
  Out(PyObject* given, const char* name, at::ScalarType dtype, std::initializer_list<int64_t> s,
      const at::Tensor& like)
      : dims((int)s.size()) {
    if (given != Py_None) {
      t = tensor_of(given, name, dtype, s);
      Py_INCREF(given);
      o = given;
    } else {
      std::copy(s.begin(), s.end(), shape.begin());
      options = at::TensorOptions().dtype(dtype).device(like.device());
    }
  }
  Out(const Out&) = delete;
  ~Out() { Py_XDECREF(o); }
  template <typename T = void>
  T* ptr() const { return static_cast<T*>(t.data_ptr()); }
  PyObject* release() {
    PyObject* r = o;
    o = nullptr;
    return r;
  }
};

// Allocates the outputs that the caller did not pass.  Without the interpreter
// lock: an allocation may wait for the device.
template <typename... O>
void allocate(O&... outs) {
  if ((outs.o && ...)) return;
  {
    Unlocked unlocked;
    const auto one = [](Out& out) {
      if (!out.o) out.t = at::empty(at::IntArrayRef(out.shape.data(), out.dims), out.options);
    };
    (one(outs), ...);
  }
  const auto wrap = [](Out& out) {
    if (!out.o) out.o = THPVariable_Wrap(out.t);
    if (!out.o) throw Raised{};
  };
  (wrap(outs), ...);
}

template <typename T = void>
T* ptr(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }

void* stream_of(const at::Tensor& t) {
  PyObject* idx = PyLong_FromLong(t.device().index());
  if (!idx) throw Raised{};
  PyObject* s = PyObject_CallOneArg(g_stream, idx);
  Py_DECREF(idx);
  if (!s) throw Raised{};
  void* p = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  if (!p && PyErr_Occurred()) throw Raised{};
  return p;
}

// Calls the C entry f(args..., stream) on the current stream of t's device,
// without the interpreter lock, and raises on a nonzero status.  The arguments,
// data pointers among them, are values by then: what a tensor without storage
// throws leaves with the lock held.
template <typename F, typename... A>
void call(const char* what, const at::Tensor& t, F f, A... args) {
  void* stream = stream_of(t);
  int st;
  {
    Unlocked unlocked;
    st = f(args..., stream);
  }
  if (st == DPTQ_OK) return;
  PyObject* r = PyObject_CallFunction(g_raise, "is", st, what);
  Py_XDECREF(r);
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, what);
  throw Raised{};
}

template <typename... O>
PyObject* tuple(O&... outs) {
  PyObject* r = PyTuple_New(sizeof...(outs));
  if (!r) throw Raised{};
  Py_ssize_t i = 0;
  (PyTuple_SET_ITEM(r, i++, outs.release()), ...);
  return r;
}

const at::Tensor* signs_of(PyObject* o, int64_t K, const at::Tensor& x) {
  if (o == Py_None) return nullptr;
  const at::Tensor& s = tensor_of(o, "signs", at::kByte, {(K + 7) / 8});
  if (s.device() != x.device()) fail(PyExc_ValueError, "signs must be on the same device as x");
  return &s;
}

int64_t fp6_bytes(int64_t rows, int64_t K) {
  const int64_t n = dptq_fp6_bytes(rows, K);
  if (n < 0)
    fail(PyExc_ValueError, "no FP6 layout for rows=" + std::to_string(rows) + ", K=" + std::to_string(K) +
                               " (K must be a multiple of 128)");
  return n;
}

// rotate_quant(x, had_size, bits, codes, scales, signs)
PyObject* rotate_quant(PyObject* const* a) {
  const at::Tensor& x = tensor(a[0], "x", at::kHalf);
  two_d(x, "x must be 2-D [M, K]");
  const int64_t M = x.size(0), K = x.size(1);
  const int32_t bits = bits_4_or_8(a[2]);
  Out codes(a[3], "codes", code_dtype(bits), {M, bits == 4 ? K / 2 : K}, x);
  Out scales(a[4], "scales", at::kFloat, {M}, x);
  allocate(codes, scales);
  const at::Tensor* signs = signs_of(a[5], K, x);
  const int32_t h = integer32(a[1]);
  if (!signs)
    call("dptq_rotate_quant", x, dptq_rotate_quant, ptr(x), M, K, h, bits, codes.ptr(), scales.ptr<float>());
  else
    call("dptq_rotate_quant_ex", x, dptq_rotate_quant_ex, ptr(x), M, K, h, bits, ptr<uint8_t>(*signs),
         DPTQ_LAYOUT_PACKED, codes.ptr(), scales.ptr<float>());
  return tuple(codes, scales);
}

// rotate_quant_fp6(x, had_size, out, scales, signs)
PyObject* rotate_quant_fp6(PyObject* const* a) {
  const at::Tensor& x = tensor(a[0], "x", at::kHalf);
  two_d(x, "x must be 2-D [M, K]");
  const int64_t M = x.size(0), K = x.size(1);
  Out out(a[2], "out", at::kByte, {fp6_bytes(M, K)}, x);
  Out scales(a[3], "scales", at::kFloat, {M}, x);
  allocate(out, scales);
  const at::Tensor* signs = signs_of(a[4], K, x);
  const int32_t h = integer32(a[1]);
  if (!signs)
    call("dptq_rotate_quant_fp6", x, dptq_rotate_quant_fp6, ptr(x), M, K, h, out.ptr<uint8_t>(),
         scales.ptr<float>());
  else
    call("dptq_rotate_quant_ex", x, dptq_rotate_quant_ex, ptr(x), M, K, h, 4, ptr<uint8_t>(*signs),
         DPTQ_LAYOUT_FP6, out.ptr(), scales.ptr<float>());
  return tuple(out, scales);
}

// rotate_quant_range(x, had_size, bits, codes, scales, zeros)
PyObject* rotate_quant_range(PyObject* const* a) {
  const at::Tensor& x = tensor(a[0], "x", at::kHalf);
  if (x.dim() != 2) fail(PyExc_ValueError, "x must be 2-D [M, K]");
  const int64_t M = x.size(0), K = x.size(1);
  const int32_t cb = code_bits(a[2]);
  Out codes(a[3], "codes", code_dtype(cb), {M, cb == 4 ? K / 2 : K}, x);
  Out scales(a[4], "scales", at::kFloat, {M}, x);
  Out zeros(a[5], "zeros", at::kInt, {M}, x);
  allocate(codes, scales, zeros);
  const int32_t h = integer32(a[1]), bits = integer32(a[2]);
  call("dptq_rotate_quant_range", x, dptq_rotate_quant_range, ptr(x), M, K, h, bits, codes.ptr(),
       scales.ptr<float>(), zeros.ptr<int32_t>());
  return tuple(codes, scales, zeros);
}

struct Gemm {
  const at::Tensor &codes, &w;
  int64_t M, K, N;
};

Gemm gemm_args(PyObject* codes_o, int32_t bits, PyObject* w_o) {
  const at::Tensor& codes = tensor(codes_o, "codes", code_dtype(bits));
  const at::Tensor& w = tensor(w_o, "w_packed", at::kByte);
  const int64_t M = dim(codes, 0), K = dim(codes, 1) * (bits == 4 ? 2 : 1), N = dim(w, 0);
  if (dim(w, 1) * 2 != K)
    fail(PyExc_ValueError, "w_packed must be [N, K/2] with K = " + std::to_string(K));
  return Gemm{codes, w, M, K, N};
}

// qlinear(codes, a_scales, bits, w_packed, w_scales, y, kernel)
PyObject* qlinear(PyObject* const* a) {
  const int32_t bits = bits_4_or_8(a[2]);
  const Gemm g = gemm_args(a[0], bits, a[3]);
  const at::Tensor& as = tensor_of(a[1], "a_scales", at::kFloat, {g.M});
  const at::Tensor& ws = tensor_of(a[4], "w_scales", at::kFloat, {g.N});
  Out y(a[5], "y", at::kHalf, {g.M, g.N}, g.codes);
  allocate(y);
  const int32_t kernel = integer32(a[6]);
  if (kernel == DPTQ_GEMM_AUTO)
    call("dptq_qlinear", g.codes, dptq_qlinear, ptr(g.codes), ptr<float>(as), g.M, g.K, bits,
         ptr<uint8_t>(g.w), ptr<float>(ws), g.N, y.ptr());
  else
    call("dptq_qlinear_kernel", g.codes, dptq_qlinear_kernel, ptr(g.codes), ptr<float>(as), g.M, g.K, bits,
         ptr<uint8_t>(g.w), ptr<float>(ws), g.N, y.ptr(), nullptr, kernel);
  return y.release();
}

// qlinear_a8(codes, a_scales, w_a8, w_scales, y, kernel)
PyObject* qlinear_a8(PyObject* const* a) {
  const Gemm g = gemm_args(a[0], 8, a[2]);
  const at::Tensor& as = tensor_of(a[1], "a_scales", at::kFloat, {g.M});
  const at::Tensor& ws = tensor_of(a[3], "w_scales", at::kFloat, {g.N});
  Out y(a[4], "y", at::kHalf, {g.M, g.N}, g.codes);
  allocate(y);
  const int32_t kernel = integer32(a[5]);
  call("dptq_qlinear_a8", g.codes, dptq_qlinear_a8, ptr(g.codes), ptr<float>(as), g.M, g.K, ptr<uint8_t>(g.w),
       ptr<float>(ws), g.N, y.ptr(), kernel);
  return y.release();
}

// qlinear_decode_native(codes, a_scales, bits, w_dec, w_scales, y)
PyObject* qlinear_decode_native(PyObject* const* a) {
  if (!THPVariable_Check(a[4])) fail(PyExc_TypeError, "w_scales must be a torch.Tensor");
  const int64_t N = dim(THPVariable_Unpack(a[4]), 0);
  const int32_t bits = bits_4_or_8(a[2]);
  const at::Tensor& codes = tensor(a[0], "codes", code_dtype(bits));
  const int64_t M = dim(codes, 0), K = dim(codes, 1) * (bits == 4 ? 2 : 1);
  const int64_t n = dptq_prepacked_bytes(N, K, DPTQ_WEIGHTS_DECODE);
  if (n < 0)
    fail(PyExc_ValueError, "no layout 3 for N=" + std::to_string(N) + ", K=" + std::to_string(K) +
                               " (K must be a multiple of 128; the decode layout also needs N % 16 == 0)");
  const at::Tensor& w = tensor_of(a[3], "w_dec", at::kByte, {n});
  const at::Tensor& as = tensor_of(a[1], "a_scales", at::kFloat, {M});
  const at::Tensor& ws = tensor_of(a[4], "w_scales", at::kFloat, {N});
  Out y(a[5], "y", at::kHalf, {M, N}, codes);
  allocate(y);
  call("dptq_qlinear_decode_native", codes, dptq_qlinear_decode_native, ptr(codes), ptr<float>(as), M, K,
       bits, ptr<uint8_t>(w), ptr<float>(ws), N, y.ptr(), nullptr);
  return y.release();
}

// qlinear_fp6(a6, a_scales, w6, w_scales, M, K, N, y)
PyObject* qlinear_fp6(PyObject* const* a) {
  const int64_t M = integer(a[4], "M"), K = integer(a[5], "K"), N = integer(a[6], "N");
  const at::Tensor& a6 = tensor_of(a[0], "a_fp6", at::kByte, {fp6_bytes(M, K)});
  const at::Tensor& w6 = tensor_of(a[2], "w_fp6", at::kByte, {fp6_bytes(N, K)});
  const at::Tensor& as = tensor_of(a[1], "a_scales", at::kFloat, {M});
  const at::Tensor& ws = tensor_of(a[3], "w_scales", at::kFloat, {N});
  Out y(a[7], "y", at::kHalf, {M, N}, a6);
  allocate(y);
  call("dptq_qlinear_fp6", a6, dptq_qlinear_fp6, ptr<uint8_t>(a6), ptr<float>(as), M, K, ptr<uint8_t>(w6),
       ptr<float>(ws), N, y.ptr(), nullptr);
  return y.release();
}

// qlinear_decode_fused(x, had_size, bits, w_packed, w_scales, y, codes, scales, mode)
PyObject* qlinear_decode_fused(PyObject* const* a) {
  const at::Tensor& x = tensor(a[0], "x", at::kHalf);
  two_d(x, "x must be 2-D [M, K]");
  const int64_t M = x.size(0), K = x.size(1);
  if (!THPVariable_Check(a[3])) fail(PyExc_TypeError, "w_packed must be a torch.Tensor");
  const int64_t N = dim(THPVariable_Unpack(a[3]), 0);
  const at::Tensor& w = tensor_of(a[3], "w_packed", at::kByte, {N, K / 2});
  const at::Tensor& ws = tensor_of(a[4], "w_scales", at::kFloat, {N});
  const int32_t cb = code_bits(a[2]);
  Out y(a[5], "y", at::kHalf, {M, N}, x);
  Out codes(a[6], "codes", code_dtype(cb), {M, cb == 4 ? K / 2 : K}, x);
  Out scales(a[7], "scales", at::kFloat, {M}, x);
  allocate(y, codes, scales);
  const int32_t h = integer32(a[1]), bits = integer32(a[2]), mode = integer32(a[8]);
  call("dptq_qlinear_decode_fused", x, dptq_qlinear_decode_fused, ptr(x), M, K, h, bits, ptr<uint8_t>(w),
       ptr<float>(ws), N, y.ptr(), codes.ptr(), scales.ptr<float>(), mode);
  return tuple(y, codes, scales);
}

// qlinear_range(codes, scales, zeros, bits, w_packed, w_scales, w_sums, y)
PyObject* qlinear_range(PyObject* const* a) {
  if (!THPVariable_Check(a[1])) fail(PyExc_TypeError, "scales must be a torch.Tensor");
  if (!THPVariable_Check(a[4])) fail(PyExc_TypeError, "w_packed must be a torch.Tensor");
  const int64_t M = dim(THPVariable_Unpack(a[1]), 0);
  const at::Tensor& wt = THPVariable_Unpack(a[4]);
  if (wt.dim() != 2) fail(PyExc_ValueError, "w_packed must be 2-D [N, K/2]");
  const int64_t N = wt.size(0), K = 2 * wt.size(1);
  const int32_t cb = code_bits(a[3]);
  const at::Tensor& codes = tensor_of(a[0], "codes", code_dtype(cb), {M, cb == 4 ? K / 2 : K});
  const at::Tensor& s = tensor_of(a[1], "scales", at::kFloat, {M});
  const at::Tensor& z = tensor_of(a[2], "zeros", at::kInt, {M});
  const at::Tensor& w = tensor_of(a[4], "w_packed", at::kByte, {N, K / 2});
  const at::Tensor& ws = tensor_of(a[5], "w_scales", at::kFloat, {N});
  const at::Tensor& sums = tensor_of(a[6], "w_sums", at::kInt, {N});
  Out y(a[7], "y", at::kHalf, {M, N}, codes);
  allocate(y);
  const int32_t bits = integer32(a[3]);
  call("dptq_qlinear_range", codes, dptq_qlinear_range, ptr(codes), ptr<float>(s), ptr<int32_t>(z), M, K,
       bits, ptr<uint8_t>(w), ptr<float>(ws), ptr<int32_t>(sums), N, y.ptr());
  return y.release();
}

// residual_dynamics(x, dx, had_size, bits, eps, jr, snr, means)
PyObject* residual_dynamics(PyObject* const* a) {
  const at::Tensor& x = tensor(a[0], "x", at::kHalf);
  two_d(x, "x must be 2-D [T, K]");
  const int64_t T = x.size(0), K = x.size(1);
  const at::Tensor& dx = tensor_of(a[1], "dx", at::kHalf, {T, K});
  const int32_t bits = bits_4_or_8(a[3]);
  Out jr(a[5], "jr", at::kFloat, {T}, x);
  Out snr(a[6], "snr", at::kFloat, {T}, x);
  Out means(a[7], "means", at::kDouble, {2}, x);
  allocate(jr, snr, means);
  const int32_t h = integer32(a[2]);
  PyObject* f = PyNumber_Float(a[4]);
  if (!f) throw Raised{};
  const double eps = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  call("dptq_residual_dynamics", x, dptq_residual_dynamics, ptr(x), ptr(dx), T, K, h, bits, (float)eps,
       jr.ptr<float>(), snr.ptr<float>(), means.ptr<double>());
  return tuple(jr, snr, means);
}

// kv_quant(kv, group, codes, scales, mins)
PyObject* kv_quant(PyObject* const* a) {
  const at::Tensor& kv = tensor(a[0], "kv", at::kHalf);
  two_d(kv, "kv must be 2-D [T, D]");
  const int64_t T = kv.size(0), D = kv.size(1), group = integer(a[1], "group", true);
  if (group <= 0 || D % group) fail(PyExc_ValueError, "D must be a multiple of group");
  if (a[3] == Py_None || a[4] == Py_None) integer(a[1], "group");   // sizes the new buffers
  Out codes(a[2], "codes", at::kByte, {T, D / 2}, kv);
  Out scales(a[3], "scales", at::kFloat, {T, D / group}, kv);
  Out mins(a[4], "mins", at::kFloat, {T, D / group}, kv);
  allocate(codes, scales, mins);
  const int32_t g = integer32(a[1]);
  call("dptq_kv_quant", kv, dptq_kv_quant, ptr(kv), T, D, g, codes.ptr<uint8_t>(), scales.ptr<float>(),
       mins.ptr<float>());
  return tuple(codes, scales, mins);
}

// kv_dequant(codes, scales, mins, group, out)
PyObject* kv_dequant(PyObject* const* a) {
  const at::Tensor& codes = tensor(a[0], "codes", at::kByte);
  two_d(codes, "codes must be 2-D [T, D/2]");
  const int64_t T = codes.size(0), D = 2 * codes.size(1), group = integer(a[3], "group", true);
  if (group <= 0 || D % group) fail(PyExc_ValueError, "D must be a multiple of group");
  const at::Tensor& scales = tensor_of(a[1], "scales", at::kFloat, {T, D / group});
  const at::Tensor& mins = tensor_of(a[2], "mins", at::kFloat, {T, D / group});
  Out out(a[4], "out", at::kHalf, {T, D}, codes);
  allocate(out);
  const int32_t g = integer32(a[3]);
  call("dptq_kv_dequant", codes, dptq_kv_dequant, ptr<uint8_t>(codes), ptr<float>(scales), ptr<float>(mins),
       T, D, g, out.ptr());
  return out.release();
}

// init(raise_error, raw_stream)
PyObject* init(PyObject* const* a) {
  Py_INCREF(a[0]);
  Py_INCREF(a[1]);
  Py_XSETREF(g_raise, a[0]);
  Py_XSETREF(g_stream, a[1]);
  Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject* const*), int NARGS>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != NARGS) {
    PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", NARGS, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

#define DPTQ_ENTRY(f, n) \
  {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&entry<f, n>)), METH_FASTCALL, nullptr}

PyMethodDef kMethods[] = {
    DPTQ_ENTRY(init, 2),
    DPTQ_ENTRY(rotate_quant, 6),
    DPTQ_ENTRY(rotate_quant_fp6, 5),
    DPTQ_ENTRY(rotate_quant_range, 6),
    DPTQ_ENTRY(qlinear, 7),
    DPTQ_ENTRY(qlinear_a8, 6),
    DPTQ_ENTRY(qlinear_decode_native, 6),
    DPTQ_ENTRY(qlinear_fp6, 8),
    DPTQ_ENTRY(qlinear_decode_fused, 9),
    DPTQ_ENTRY(qlinear_range, 8),
    DPTQ_ENTRY(residual_dynamics, 8),
    DPTQ_ENTRY(kv_quant, 5),
    DPTQ_ENTRY(kv_dequant, 5),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_dptq_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr,
                       nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dptq_torch() { return PyModule_Create(&kModule); }
