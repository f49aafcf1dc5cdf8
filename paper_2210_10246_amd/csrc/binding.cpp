// The calls of binding.py in native code: the same checks on the same arguments, then the C ABI on
// the current stream.  Marshalling one call through ctypes takes 8-10 us of Python, more than the
// kernels of a small layer (float32 LayerNorm of 256 x 768, forward + backward: 23 us a pass, 9 us of
// them on the GPU; through this file 10).
//
// A function here returns the status of the call, or None for anything that is not plainly in
// order: another type, dtype, size or layout, a tensor subclass, a tensor without storage, a number that
// is no float or int.  Nothing has happened then, and binding.py goes through its own checks, which
// raise what they always raised.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/tempo.h"

namespace {

struct NotPlain {};

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotPlain{};
  return THPVariable_Unpack(o);
}
void* pointer(const at::Tensor& t) {
  if (!t.is_cuda() || !t.has_storage() || !t.is_contiguous()) throw NotPlain{};
  return t.data_ptr();
}
// Argument o as a device pointer, if it has that dtype and number of elements (or at least so many).
void* exactly(PyObject* o, at::ScalarType dtype, int64_t numel) {
  const at::Tensor& t = tensor(o);
  if (t.scalar_type() != dtype || t.numel() != numel) throw NotPlain{};
  return pointer(t);
}
void* at_least(PyObject* o, at::ScalarType dtype, int64_t numel) {
  const at::Tensor& t = tensor(o);
  if (t.scalar_type() != dtype || t.numel() < numel) throw NotPlain{};
  return pointer(t);
}
void* optional(PyObject* o, at::ScalarType dtype, int64_t numel) {
  return o == Py_None ? nullptr : exactly(o, dtype, numel);
}
float* floats(PyObject* o, int64_t numel) {
  return static_cast<float*>(exactly(o, at::kFloat, numel));
}
uint32_t* mask_words(PyObject* o, int64_t n) {
  return static_cast<uint32_t*>(at_least(o, at::kInt, (n + 31) / 32));
}

float real(PyObject* o) {
  if (PyFloat_Check(o)) return static_cast<float>(PyFloat_AS_DOUBLE(o));
  if (PyLong_CheckExact(o)) {
    const double v = PyLong_AsDouble(o);
    if (!PyErr_Occurred()) return static_cast<float>(v);
  }
  throw NotPlain{};
}
uint64_t bits64(PyObject* o) {
  if (PyLong_CheckExact(o)) return PyLong_AsUnsignedLongLongMask(o);
  throw NotPlain{};
}
tempo_gelu_kind gelu_kind(PyObject* o) {
  if (PyUnicode_CheckExact(o)) {
    if (PyUnicode_CompareWithASCIIString(o, "erf") == 0) return TEMPO_GELU_ERF;
    if (PyUnicode_CompareWithASCIIString(o, "tanh") == 0) return TEMPO_GELU_TANH;
  }
  throw NotPlain{};
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// An activation tensor: its pointer, element count, and dtype in both vocabularies.
struct Act {
  const at::Tensor& t;
  void* p;
  int64_t n;
  at::ScalarType scalar;
  tempo_dtype dt;
  explicit Act(PyObject* o) : t(tensor(o)), p(pointer(t)), n(t.numel()), scalar(t.scalar_type()) {
    if (scalar != at::kFloat && scalar != at::kBFloat16) throw NotPlain{};
    dt = scalar == at::kFloat ? TEMPO_F32 : TEMPO_BF16;
  }
  void* same(PyObject* o) const { return exactly(o, scalar, n); }
  void* same_or_none(PyObject* o) const { return optional(o, scalar, n); }
};
struct Rows : Act {  // [N, M]
  int64_t M, N;
  explicit Rows(PyObject* o) : Act(o) {
    if (t.dim() < 1) throw NotPlain{};
    M = t.size(-1);
    N = M ? n / M : 0;
  }
};
struct Slices : Act {  // [B, A, Sq, Sk]
  explicit Slices(PyObject* o) : Act(o) {
    if (t.dim() != 4) throw NotPlain{};
  }
};

// Runs `prepare` (checks; may throw) and the call it returns, with the interpreter released as
// ctypes does.
template <int ARGS, typename F>
PyObject* plain_call(Py_ssize_t nargs, F&& prepare) {
  if (nargs != ARGS) Py_RETURN_NONE;
  try {
    auto call = prepare();
    tempo_status status;
    PyThreadState* state = PyEval_SaveThread();
    status = call();  // a C function: returns a status, throws nothing
    PyEval_RestoreThread(state);
    return PyLong_FromLong(status);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

#define TEMPO_METHOD(name) PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t nargs)

TEMPO_METHOD(gelu_fwd) {  // x, y, mask, kind
  return plain_call<4>(nargs, [&] {
    const Act x(a[0]);
    return [p = x.p, y = x.same(a[1]), m = mask_words(a[2], x.n), n = x.n, dt = x.dt,
            k = gelu_kind(a[3]), st = stream()] { return tempo_gelu_fwd(p, y, m, n, dt, k, st); };
  });
}
TEMPO_METHOD(gelu_bwd) {  // dy, y, mask, dx, kind
  return plain_call<5>(nargs, [&] {
    const Act y(a[1]);
    return [dy = y.same(a[0]), p = y.p, m = mask_words(a[2], y.n), dx = y.same(a[3]), n = y.n, dt = y.dt,
            k = gelu_kind(a[4]), st = stream()] { return tempo_gelu_bwd(dy, p, m, dx, n, dt, k, st); };
  });
}
TEMPO_METHOD(silu_fwd) {  // x, y, mask
  return plain_call<3>(nargs, [&] {
    const Act x(a[0]);
    return [p = x.p, y = x.same(a[1]), m = mask_words(a[2], x.n), n = x.n, dt = x.dt, st = stream()] {
      return tempo_silu_fwd(p, y, m, n, dt, st);
    };
  });
}
TEMPO_METHOD(silu_bwd) {  // dy, y, mask, dx
  return plain_call<4>(nargs, [&] {
    const Act y(a[1]);
    return [dy = y.same(a[0]), p = y.p, m = mask_words(a[2], y.n), dx = y.same(a[3]), n = y.n, dt = y.dt,
            st = stream()] { return tempo_silu_bwd(dy, p, m, dx, n, dt, st); };
  });
}
TEMPO_METHOD(layernorm_fwd) {  // x, gamma, beta, y, rstd, mean, eps
  return plain_call<7>(nargs, [&] {
    const Rows x(a[0]);
    return [p = x.p, ga = floats(a[1], x.M), be = floats(a[2], x.M), y = x.same(a[3]),
            rs = floats(a[4], x.N), mu = static_cast<float*>(optional(a[5], at::kFloat, x.N)), N = x.N,
            M = x.M, eps = real(a[6]), dt = x.dt, st = stream()] {
      return tempo_layernorm_fwd(p, ga, be, y, rs, mu, N, M, eps, dt, st);
    };
  });
}
TEMPO_METHOD(layernorm_bwd) {  // dy, y, gamma, beta, rstd, dx, dgamma, dbeta, workspace
  return plain_call<9>(nargs, [&] {
    const Rows y(a[1]);
    const at::Tensor& ws = tensor(a[8]);
    return [dy = y.same(a[0]), p = y.p, ga = floats(a[2], y.M), be = floats(a[3], y.M),
            rs = floats(a[4], y.N), dx = y.same(a[5]), dg = floats(a[6], y.M), db = floats(a[7], y.M),
            w = pointer(ws), size = static_cast<size_t>(ws.numel()) * ws.element_size(), N = y.N, M = y.M,
            dt = y.dt, st = stream()] {
      return tempo_layernorm_bwd(dy, p, ga, be, rs, dx, dg, db, w, size, N, M, dt, st);
    };
  });
}
TEMPO_METHOD(layernorm_bwd_static) {  // dy, y, gamma, beta, rstd, dx, dgamma, dbeta
  return plain_call<8>(nargs, [&] {
    const Rows y(a[1]);
    return [dy = y.same(a[0]), p = y.p, ga = floats(a[2], y.M), be = floats(a[3], y.M),
            rs = floats(a[4], y.N), dx = y.same(a[5]), dg = floats(a[6], y.M), db = floats(a[7], y.M),
            N = y.N, M = y.M, dt = y.dt, st = stream()] {
      return tempo_layernorm_bwd_static(dy, p, ga, be, rs, dx, dg, db, N, M, dt, st);
    };
  });
}
// scores, key_len, causal, probs, out, keep_bits, p, seed, offset
TEMPO_METHOD(attn_softmax_dropout_fwd) {
  return plain_call<9>(nargs, [&] {
    const Slices s(a[0]);
    const int causal = PyObject_IsTrue(a[2]);
    if (causal < 0) throw NotPlain{};
    return [sc = s.p, kl = static_cast<int32_t*>(optional(a[1], at::kInt, s.t.size(0))), causal,
            pr = s.same(a[3]), out = s.same_or_none(a[4]), kb = mask_words(a[5], s.n), B = s.t.size(0),
            A = s.t.size(1), Sq = s.t.size(2), Sk = s.t.size(3), p = real(a[6]), seed = bits64(a[7]),
            offset = bits64(a[8]), dt = s.dt, st = stream()] {
      return tempo_attn_softmax_dropout_fwd(sc, kl, causal, pr, out, kb, B, A, Sq, Sk, p, seed, offset, dt,
                                            st);
    };
  });
}
TEMPO_METHOD(attn_softmax_dropout_bwd) {  // dout, probs, keep_bits, dscores, out_recomputed, p
  return plain_call<6>(nargs, [&] {
    const Slices s(a[1]);
    return [dout = s.same(a[0]), pr = s.p, kb = mask_words(a[2], s.n), ds = s.same(a[3]),
            re = s.same_or_none(a[4]), B = s.t.size(0), A = s.t.size(1), Sq = s.t.size(2),
            Sk = s.t.size(3), p = real(a[5]), dt = s.dt, st = stream()] {
      return tempo_attn_softmax_dropout_bwd(dout, pr, kb, ds, re, B, A, Sq, Sk, p, dt, st);
    };
  });
}
// dout, probs, dscores, out_recomputed, p, seed, offset
TEMPO_METHOD(attn_softmax_dropout_bwd_regen) {
  return plain_call<7>(nargs, [&] {
    const Slices s(a[1]);
    return [dout = s.same(a[0]), pr = s.p, ds = s.same(a[2]), re = s.same_or_none(a[3]), B = s.t.size(0),
            A = s.t.size(1), Sq = s.t.size(2), Sk = s.t.size(3), p = real(a[4]), seed = bits64(a[5]),
            offset = bits64(a[6]), dt = s.dt, st = stream()] {
      return tempo_attn_softmax_dropout_bwd_regen(dout, pr, ds, re, B, A, Sq, Sk, p, seed, offset, dt, st);
    };
  });
}
TEMPO_METHOD(attn_softmax_dropout_bwd_bytemask) {  // dout, probs, keep_bytes, dscores, out_recomputed, p
  return plain_call<6>(nargs, [&] {
    const Slices s(a[1]);
    const at::Tensor& k = tensor(a[2]);
    if ((k.scalar_type() != at::kByte && k.scalar_type() != at::kBool) || k.numel() != s.n) throw NotPlain{};
    return [dout = s.same(a[0]), pr = s.p, kb = static_cast<const uint8_t*>(pointer(k)), ds = s.same(a[3]),
            re = s.same_or_none(a[4]), B = s.t.size(0), A = s.t.size(1), Sq = s.t.size(2),
            Sk = s.t.size(3), p = real(a[5]), dt = s.dt, st = stream()] {
      return tempo_attn_softmax_dropout_bwd_bytemask(dout, pr, kb, ds, re, B, A, Sq, Sk, p, dt, st);
    };
  });
}

#define TEMPO_ENTRY(name) {"tempo_" #name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {TEMPO_ENTRY(gelu_fwd),
                         TEMPO_ENTRY(gelu_bwd),
                         TEMPO_ENTRY(silu_fwd),
                         TEMPO_ENTRY(silu_bwd),
                         TEMPO_ENTRY(layernorm_fwd),
                         TEMPO_ENTRY(layernorm_bwd),
                         TEMPO_ENTRY(layernorm_bwd_static),
                         TEMPO_ENTRY(attn_softmax_dropout_fwd),
                         TEMPO_ENTRY(attn_softmax_dropout_bwd),
                         TEMPO_ENTRY(attn_softmax_dropout_bwd_regen),
                         TEMPO_ENTRY(attn_softmax_dropout_bwd_bytemask),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
