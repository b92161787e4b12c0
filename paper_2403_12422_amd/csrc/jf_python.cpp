// The Python side of the C ABI as a CPython extension module (_native): what binding.py's functions do per call --
// checking the tensors, allocating the outputs, reading pointers and the current stream -- in C++.  A call costs the
// host 4-5 us here, of which the kernel launch is 3; the same steps through ctypes and torch's Python API cost 8 us
// (outputs given) to 20 us (outputs allocated, several results), which is more than the kernels of a small layer take.
// The module computes nothing and exports nothing of its own: every function ends in one jf_* call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/EmptyTensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/hip/impl/HIPCachingAllocatorMasqueradingAsCUDA.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <utility>

#include "jetfire.h"

namespace {

PyObject* g_error = nullptr;   // binding.JetfireError, set by init()

[[noreturn]] void raise(long code, const std::string& message) {
  PyObject* e = PyObject_CallFunction(g_error, "ls", code, message.c_str());
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  throw python_error();
}

void check(int32_t rc) {
  if (rc == JF_OK) return;
  std::string msg = jf_error_string(rc);
  if (rc == JF_ERR_LAUNCH) msg += " (hip error " + std::to_string(jf_last_hip_error()) + ")";
  raise(rc, msg);
}

int64_t integer(PyObject* o) {
  PyObject* i = PyNumber_Index(o);
  if (!i) throw python_error();
  const int64_t v = PyLong_AsLongLong(i);
  Py_DECREF(i);
  if (v == -1 && PyErr_Occurred()) throw python_error();
  return v;
}

// The quantization block; sizes of outputs are divided by it, so what the library would refuse is refused first.
int32_t block_size(PyObject* o) {
  const int64_t b = integer(o);
  if (b != 32 && b != 64 && b != 128) check(JF_ERR_BLOCK);
  return (int32_t)b;
}

float real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw python_error();
  return (float)v;
}

bool flag(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw python_error();
  return v != 0;
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a torch.Tensor, got %s", Py_TYPE(o)->tp_name);
    throw python_error();
  }
  return THPVariable_Unpack(o);
}

// An operand: on the GPU, contiguous, of the given type and number of dimensions.
const at::Tensor& operand(PyObject* o, at::ScalarType dtype, int64_t ndim) {
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda()) raise(-2, "tensors must live on the GPU; this library has no CPU path");
  if (t.scalar_type() != dtype || t.dim() != ndim || !t.is_contiguous()) {
    std::string shape = "(";
    for (int64_t d : t.sizes()) shape += std::to_string(d) + ", ";
    raise(-2, std::string("expected contiguous ") + std::to_string(ndim) + "-d " + c10::toString(dtype) + " tensor, got " +
                  c10::toString(t.scalar_type()) + " " + shape + ")");
  }
  return t;
}
const at::Tensor& codes(PyObject* o) { return operand(o, at::kChar, 2); }
const at::Tensor& grid(PyObject* o) { return operand(o, at::kFloat, 2); }
const at::Tensor& vector(PyObject* o) { return operand(o, at::kFloat, 1); }

template <class T>
const T* in(const at::Tensor& t) { return static_cast<const T*>(t.const_data_ptr()); }
// pointer of an optional tensor argument (None = absent)
template <class T>
T* pointer(PyObject* o) { return o == Py_None ? nullptr : static_cast<T*>(tensor(o).mutable_data_ptr()); }

// A new reference that is dropped unless it is handed over with release().
struct Ref {
  PyObject* p;
  explicit Ref(PyObject* o = nullptr) : p(o) {}
  Ref(Ref&& o) noexcept : p(o.p) { o.p = nullptr; }
  Ref& operator=(Ref&& o) noexcept { std::swap(p, o.p); return *this; }
  ~Ref() { Py_XDECREF(p); }
  PyObject* release() { PyObject* o = p; p = nullptr; return o; }
};

Ref owned(PyObject* o) {
  if (!o) throw python_error();
  return Ref(o);
}
Ref same(PyObject* o) { Py_INCREF(o); return Ref(o); }
Ref none() { return same(Py_None); }
// New outputs on the device of `like`, from torch's caching allocator.  On the current device, where a tensor of that device
// exists already, the generic constructor does: empty_cuda's lazy initialisation and device guards take 0.17 of its 0.51 us.
// Which device is current belongs to the calling thread and is read for each call.
class Outputs {
  const at::Tensor& like;
  bool here;

 public:
  explicit Outputs(const at::Tensor& t) : like(t) {
    c10::DeviceIndex device = -1;
    here = c10::hip::GetDevice(&device) == hipSuccess && t.device().index() == device;
  }
  Ref tensor(std::initializer_list<int64_t> size, at::ScalarType dtype) const {
    const at::IntArrayRef s(size.begin(), size.size());
    if (!here) return owned(THPVariable_Wrap(at::Tensor(at::detail::empty_cuda(s, dtype, like.device(), std::nullopt))));
    at::Allocator* const allocator = c10::hip::HIPCachingAllocatorMasqueradingAsCUDA::get();   // torch's for its "cuda" devices
    return owned(THPVariable_Wrap(
        at::Tensor(at::detail::empty_generic(s, allocator, c10::DispatchKeySet(c10::DispatchKey::CUDA), dtype, std::nullopt))));
  }
  Ref floats(std::initializer_list<int64_t> size) const { return tensor(size, at::kFloat); }
  Ref codes(int64_t r, int64_t c) const { return tensor({r, c}, at::kChar); }
  Ref grid(int64_t r, int64_t c, int64_t b) const { return floats({r / b, c / b}); }
};

// The caller's preallocated outputs: item i of a sequence that must hold `n` items (n < 0: at least -n).
struct Given {
  Ref seq;
  Given(PyObject* o, Py_ssize_t n) : seq(owned(PySequence_Fast(o, "out must be a sequence of tensors"))) {
    const Py_ssize_t have = PySequence_Fast_GET_SIZE(seq.p);
    if (n >= 0 ? have != n : have < -n) {
      PyErr_Format(PyExc_ValueError, "out must hold %zd tensors, got %zd", n >= 0 ? n : -n, have);
      throw python_error();
    }
  }
  PyObject* item(Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(seq.p, i); }
  Ref operator[](Py_ssize_t i) const { return same(item(i)); }
};

template <class... R>
PyObject* tuple(R&&... refs) {
  PyObject* t = PyTuple_New(sizeof...(refs));
  if (!t) throw python_error();
  Py_ssize_t i = 0;
  (PyTuple_SET_ITEM(t, i++, refs.release()), ...);
  return t;
}

// The launch itself, without the interpreter lock: it may wait for room in the stream's queue.
template <class F>
void launch(F&& f) {
  void* const stream = c10::hip::getCurrentHIPStream().stream();
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f(stream);
  Py_END_ALLOW_THREADS
  check(rc);
}

void expect(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    throw python_error();
  }
}

// quantize(x, block, transposed_copy, out)
PyObject* quantize(PyObject* const* a, Py_ssize_t n) {
  expect(n, 4);
  const at::Tensor& x0 = tensor(a[0]);
  const at::ScalarType dtype = x0.scalar_type();
  if (dtype != at::kFloat && dtype != at::kHalf) raise(JF_ERR_DTYPE, "source must be float32 or float16");
  const at::Tensor& x = operand(a[0], dtype, 2);
  const int32_t b = block_size(a[1]);
  const bool transposed = flag(a[2]);
  const int64_t rows = x.size(0), cols = x.size(1);
  Ref q, s, qT, sT;
  if (a[3] != Py_None) {
    const Given out(a[3], transposed ? -4 : -2);
    q = out[0], s = out[1];
    qT = (transposed ? out[2] : none()), sT = (transposed ? out[3] : none());
  } else {
    const Outputs make(x);
    q = make.codes(rows, cols), s = make.grid(rows, cols, b);
    qT = (transposed ? make.codes(cols, rows) : none());
    sT = (transposed ? make.grid(cols, rows, b) : none());
  }
  const void* px = x.const_data_ptr();
  int8_t *pq = pointer<int8_t>(q.p), *pqT = pointer<int8_t>(qT.p);
  float *ps = pointer<float>(s.p), *psT = pointer<float>(sT.p);
  launch([&](void* st) { return jf_quantize_block(px, dtype == at::kFloat ? 0 : 1, rows, cols, cols, b, pq, cols, ps, pqT, rows, psT, st); });
  return transposed ? tuple(q, s, qT, sT) : tuple(q, s);
}

// dequantize(q, s, block, half, out)
PyObject* dequantize(PyObject* const* a, Py_ssize_t n) {
  expect(n, 5);
  const at::Tensor &q = codes(a[0]), &s = grid(a[1]);
  const int32_t b = (int32_t)integer(a[2]);
  const bool half = flag(a[3]);
  const int64_t rows = q.size(0), cols = q.size(1);
  Ref out = a[4] != Py_None ? same(a[4]) : Outputs(q).tensor({rows, cols}, half ? at::kHalf : at::kFloat);
  void* po = pointer<void>(out.p);
  launch([&](void* st) { return jf_dequantize_block(in<int8_t>(q), in<float>(s), rows, cols, b, po, half ? 1 : 0, cols, st); });
  return out.release();
}

typedef int32_t (*linear_fn)(const int8_t*, const float*, const int8_t*, const float*, int64_t, int64_t, int64_t, int32_t, int8_t*,
                             float*, float*, void*, size_t, void*);

PyObject* linear(linear_fn fn, const at::Tensor& p, const at::Tensor& sp, const at::Tensor& w, const at::Tensor& sw, int64_t N,
                 int64_t C, int64_t D, int32_t b, int64_t rows, int64_t cols, bool want_q, bool want_f32, PyObject* given) {
  Ref q, s, f;
  if (given != Py_None) {
    const Given out(given, 3);
    q = out[0], s = out[1], f = out[2];
  } else {
    const Outputs make(p);
    q = (want_q ? make.codes(rows, cols) : none());
    s = (want_q ? make.grid(rows, cols, b) : none());
    f = (want_f32 ? make.floats({rows, cols}) : none());
  }
  int8_t* pq = pointer<int8_t>(q.p);
  float *ps = pointer<float>(s.p), *pf = pointer<float>(f.p);
  launch([&](void* st) { return fn(in<int8_t>(p), in<float>(sp), in<int8_t>(w), in<float>(sw), N, C, D, b, pq, ps, pf, nullptr, 0, st); });
  return tuple(q, s, f);
}

// linear_fwd(X, SX, W, SW, block, want_f32, out)
PyObject* linear_fwd(PyObject* const* a, Py_ssize_t n) {
  expect(n, 7);
  const at::Tensor &X = codes(a[0]), &W = codes(a[2]), &SX = grid(a[1]), &SW = grid(a[3]);
  const int64_t N = X.size(0), C = X.size(1), D = W.size(0);
  if (W.size(1) != C) raise(JF_ERR_SHAPE, "X and W disagree on C");
  return linear(jf_linear_fwd, X, SX, W, SW, N, C, D, block_size(a[4]), N, D, true, flag(a[5]), a[6]);
}

// linear_dgrad(dY, SdY, W, SW, block, want_f32, out)
PyObject* linear_dgrad(PyObject* const* a, Py_ssize_t n) {
  expect(n, 7);
  const at::Tensor &dY = codes(a[0]), &W = codes(a[2]), &SdY = grid(a[1]), &SW = grid(a[3]);
  const int64_t N = dY.size(0), D = dY.size(1), C = W.size(1);
  if (W.size(0) != D) raise(JF_ERR_SHAPE, "dY and W disagree on D");
  return linear(jf_linear_dgrad, dY, SdY, W, SW, N, C, D, block_size(a[4]), N, C, true, flag(a[5]), a[6]);
}

// linear_wgrad(dY, SdY, X, SX, block, want_q, want_f32, out)
PyObject* linear_wgrad(PyObject* const* a, Py_ssize_t n) {
  expect(n, 8);
  const at::Tensor &dY = codes(a[0]), &X = codes(a[2]), &SdY = grid(a[1]), &SX = grid(a[3]);
  const int64_t N = dY.size(0), D = dY.size(1), C = X.size(1);
  if (X.size(0) != N) raise(JF_ERR_SHAPE, "dY and X disagree on N");
  return linear(jf_linear_wgrad, dY, SdY, X, SX, N, C, D, block_size(a[4]), D, C, flag(a[5]), flag(a[6]), a[7]);
}

// linear_bwd(dY, SdY, W, SW, X, SX, block, want_f32, out)
PyObject* linear_bwd(PyObject* const* a, Py_ssize_t n) {
  expect(n, 9);
  const at::Tensor &dY = codes(a[0]), &W = codes(a[2]), &X = codes(a[4]), &SdY = grid(a[1]), &SW = grid(a[3]), &SX = grid(a[5]);
  const int64_t N = dY.size(0), D = dY.size(1), C = W.size(1);
  if (W.size(0) != D || X.size(0) != N || X.size(1) != C) raise(JF_ERR_SHAPE, "dY, W and X disagree on N, C, D");
  const int32_t b = block_size(a[6]);
  const bool want_f32 = flag(a[7]);
  Ref o[6];   // dX, SdX, dX_f32, dW, SdW, dW_f32
  if (a[8] != Py_None) {
    const Given out(a[8], 2);
    for (int i = 0; i < 2; ++i) {
      const Given half(out.item(i), 3);
      for (int j = 0; j < 3; ++j) o[3 * i + j] = half[j];
    }
  } else {
    const Outputs make(dY);
    const int64_t rows[2] = {N, D};
    for (int i = 0; i < 2; ++i) {
      o[3 * i] = make.codes(rows[i], C);
      o[3 * i + 1] = make.grid(rows[i], C, b);
      o[3 * i + 2] = (want_f32 ? make.floats({rows[i], C}) : none());
    }
  }
  int8_t *dX = pointer<int8_t>(o[0].p), *dW = pointer<int8_t>(o[3].p);
  float *SdX = pointer<float>(o[1].p), *dXf = pointer<float>(o[2].p), *SdW = pointer<float>(o[4].p), *dWf = pointer<float>(o[5].p);
  launch([&](void* st) {
    return jf_linear_bwd(in<int8_t>(dY), in<float>(SdY), in<int8_t>(W), in<float>(SW), in<int8_t>(X), in<float>(SX), N, C, D, b, dX, SdX,
                         dXf, dW, SdW, dWf, nullptr, 0, st);
  });
  Ref first(tuple(o[0], o[1], o[2])), second(tuple(o[3], o[4], o[5]));
  return tuple(first, second);
}

// gelu(X, SX, block, out)
PyObject* gelu(PyObject* const* a, Py_ssize_t n) {
  expect(n, 4);
  const at::Tensor &X = codes(a[0]), &SX = grid(a[1]);
  const int32_t b = (int32_t)integer(a[2]);
  const int64_t N = X.size(0), C = X.size(1);
  Ref Y, SY;
  if (a[3] != Py_None) {
    const Given out(a[3], 2);
    Y = out[0], SY = out[1];
  } else {
    const Outputs make(X);
    Y = make.codes(N, C), SY = make.floats({SX.size(0), SX.size(1)});
  }
  int8_t* y = pointer<int8_t>(Y.p);
  float* sy = pointer<float>(SY.p);
  launch([&](void* st) { return jf_gelu_q(in<int8_t>(X), in<float>(SX), N, C, b, y, sy, st); });
  return tuple(Y, SY);
}

// gelu_bwd(dY, SdY, X, SX, block, out)
PyObject* gelu_bwd(PyObject* const* a, Py_ssize_t n) {
  expect(n, 6);
  const at::Tensor &X = codes(a[2]), &SX = grid(a[3]), &dY = codes(a[0]), &SdY = grid(a[1]);
  const int32_t b = (int32_t)integer(a[4]);
  const int64_t N = X.size(0), C = X.size(1);
  if (dY.sizes() != X.sizes()) raise(JF_ERR_SHAPE, "dY and X shapes differ");
  Ref dX, SdX;
  if (a[5] != Py_None) {
    const Given out(a[5], 2);
    dX = out[0], SdX = out[1];
  } else {
    const Outputs make(X);
    dX = make.codes(N, C), SdX = make.floats({SX.size(0), SX.size(1)});
  }
  int8_t* y = pointer<int8_t>(dX.p);
  float* sy = pointer<float>(SdX.p);
  launch([&](void* st) { return jf_gelu_q_bwd(in<int8_t>(dY), in<float>(SdY), in<int8_t>(X), in<float>(SX), N, C, b, y, sy, st); });
  return tuple(dX, SdX);
}

// layernorm(X, SX, row_mean | None, row_sumsq | None, gamma, beta, eps, block, out): from partials when they are given
PyObject* layernorm(PyObject* const* a, Py_ssize_t n) {
  expect(n, 9);
  const at::Tensor &X = codes(a[0]), &SX = grid(a[1]), &gamma = vector(a[4]), &beta = vector(a[5]);
  const int64_t N = X.size(0), C = X.size(1);
  const float eps = real(a[6]);
  const int32_t b = block_size(a[7]);
  const float *rm = nullptr, *rq = nullptr;
  const bool partials = a[2] != Py_None;
  if (partials) {
    const at::Tensor &m = grid(a[2]), &q = grid(a[3]);
    if (m.size(0) != C / b || m.size(1) != N || q.sizes() != m.sizes())
      raise(JF_ERR_SHAPE, "row partials must be (C / block, N), as jf_add_q writes them");
    rm = in<float>(m), rq = in<float>(q);
  }
  Ref Y, SY, mean, rstd;
  if (a[8] != Py_None) {
    const Given out(a[8], 4);
    Y = out[0], SY = out[1], mean = out[2], rstd = out[3];
  } else {
    const Outputs make(X);
    Y = make.codes(N, C), SY = make.floats({SX.size(0), SX.size(1)});
    mean = make.floats({N}), rstd = make.floats({N});
  }
  int8_t* y = pointer<int8_t>(Y.p);
  float *sy = pointer<float>(SY.p), *mu = pointer<float>(mean.p), *rs = pointer<float>(rstd.p);
  launch([&](void* st) {
    return partials ? jf_layernorm_q_partials(in<int8_t>(X), in<float>(SX), rm, rq, in<float>(gamma), in<float>(beta), eps, N, C, b, y, sy, mu, rs, st)
                    : jf_layernorm_q(in<int8_t>(X), in<float>(SX), in<float>(gamma), in<float>(beta), eps, N, C, b, y, sy, mu, rs, st);
  });
  return tuple(Y, SY, mean, rstd);
}

// dropout(X, SX, mask_bits, p, block, out)
PyObject* dropout(PyObject* const* a, Py_ssize_t n) {
  expect(n, 6);
  const at::Tensor &X = codes(a[0]), &SX = grid(a[1]), &mask = operand(a[2], at::kByte, 2);
  const float p = real(a[3]);
  const int32_t b = (int32_t)integer(a[4]);
  const int64_t N = X.size(0), C = X.size(1);
  if (mask.size(0) != N || mask.size(1) != C / 8) raise(JF_ERR_SHAPE, "mask_bits must be (N, C / 8)");
  Ref Y, SY;
  if (a[5] != Py_None) {
    const Given out(a[5], 2);
    Y = out[0], SY = out[1];
  } else {
    const Outputs make(X);
    Y = make.codes(N, C), SY = make.floats({SX.size(0), SX.size(1)});
  }
  int8_t* y = pointer<int8_t>(Y.p);
  float* sy = pointer<float>(SY.p);
  launch([&](void* st) { return jf_dropout_q(in<int8_t>(X), in<float>(SX), in<uint8_t>(mask), p, N, C, b, y, sy, st); });
  return tuple(Y, SY);
}

// add(X1, S1, X2, S2, block, want_partials, out)
PyObject* add(PyObject* const* a, Py_ssize_t n) {
  expect(n, 7);
  const at::Tensor &X1 = codes(a[0]), &S1 = grid(a[1]), &X2 = codes(a[2]), &S2 = grid(a[3]);
  const int32_t b = block_size(a[4]);
  const bool partials = flag(a[5]);
  const int64_t N = X1.size(0), C = X1.size(1);
  if (X2.sizes() != X1.sizes()) raise(JF_ERR_SHAPE, "X1 and X2 shapes differ");
  Ref Y, SY, rm, rq;
  if (a[6] != Py_None) {
    const Given out(a[6], partials ? -4 : -2);
    Y = out[0], SY = out[1];
    rm = (partials ? out[2] : none()), rq = (partials ? out[3] : none());
  } else {
    const Outputs make(X1);
    Y = make.codes(N, C), SY = make.floats({S1.size(0), S1.size(1)});
    rm = (partials ? make.floats({C / b, N}) : none());
    rq = (partials ? make.floats({C / b, N}) : none());
  }
  int8_t* y = pointer<int8_t>(Y.p);
  float *sy = pointer<float>(SY.p), *m = pointer<float>(rm.p), *q = pointer<float>(rq.p);
  launch([&](void* st) { return jf_add_q(in<int8_t>(X1), in<float>(S1), in<int8_t>(X2), in<float>(S2), N, C, b, y, sy, m, q, st); });
  return partials ? tuple(Y, SY, rm, rq) : tuple(Y, SY);
}

// layernorm_bwd(dY, SdY, X, SX, gamma, mean, rstd, block, workspace | None, out | None, static)
PyObject* layernorm_bwd(PyObject* const* a, Py_ssize_t n) {
  expect(n, 11);
  const at::Tensor &X = codes(a[2]), &SX = grid(a[3]), &dY = codes(a[0]), &SdY = grid(a[1]);
  const at::Tensor &gamma = vector(a[4]), &mean = vector(a[5]), &rstd = vector(a[6]);
  const int32_t b = (int32_t)integer(a[7]);
  const bool fixed = flag(a[10]);
  const int64_t N = X.size(0), C = X.size(1);
  if (dY.sizes() != X.sizes()) raise(JF_ERR_SHAPE, "dY and X shapes differ");
  Ref ws = none();
  if (!fixed) {
    if (a[8] != Py_None) {
      ws = same(a[8]);
    } else {
      const int64_t need = (int64_t)jf_workspace_bytes(JF_OP_LAYERNORM_BWD, N, C, 0, b);
      ws = Outputs(X).tensor({need > 16 ? need : 16}, at::kByte);
    }
  }
  Ref dX, SdX, dg, db;
  if (fixed || a[9] != Py_None) {
    const Given out(a[9], 4);
    dX = out[0], SdX = out[1], dg = out[2], db = out[3];
    if (fixed) codes(dX.p), grid(SdX.p), vector(dg.p), vector(db.p);
  } else {
    const Outputs make(X);
    dX = make.codes(N, C), SdX = make.floats({SX.size(0), SX.size(1)});
    dg = make.floats({C}), db = make.floats({C});
  }
  int8_t* y = pointer<int8_t>(dX.p);
  float *sy = pointer<float>(SdX.p), *g = pointer<float>(dg.p), *e = pointer<float>(db.p);
  void* w = pointer<void>(ws.p);
  const size_t bytes = w ? (size_t)tensor(ws.p).numel() : 0;
  launch([&](void* st) {
    return fixed ? jf_layernorm_q_bwd_static(in<int8_t>(dY), in<float>(SdY), in<int8_t>(X), in<float>(SX), in<float>(gamma), in<float>(mean),
                                             in<float>(rstd), N, C, b, y, sy, g, e, st)
                 : jf_layernorm_q_bwd(in<int8_t>(dY), in<float>(SdY), in<int8_t>(X), in<float>(SX), in<float>(gamma), in<float>(mean),
                                      in<float>(rstd), N, C, b, y, sy, g, e, w, bytes, st);
  });
  return tuple(dX, SdX, dg, db);
}

PyObject* init(PyObject* const* a, Py_ssize_t n) {
  expect(n, 1);
  Py_INCREF(a[0]);
  Py_XDECREF(g_error);
  g_error = a[0];
  Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  return F(args, n);
  END_HANDLE_TH_ERRORS
}

template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<F>)), METH_FASTCALL, nullptr};
}

PyMethodDef g_methods[] = {
    method<init>("init"),
    method<quantize>("quantize"),
    method<dequantize>("dequantize"),
    method<linear_fwd>("linear_fwd"),
    method<linear_dgrad>("linear_dgrad"),
    method<linear_wgrad>("linear_wgrad"),
    method<linear_bwd>("linear_bwd"),
    method<gelu>("gelu"),
    method<gelu_bwd>("gelu_bwd"),
    method<layernorm>("layernorm"),
    method<dropout>("dropout"),
    method<add>("add"),
    method<layernorm_bwd>("layernorm_bwd"),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&g_module); }
