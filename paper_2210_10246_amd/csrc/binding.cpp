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
#include <ATen/ops/empty.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/tempo.h"
#include "encoder.h"

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

// ---- the encoder layer of modules.py ---------------------------------------------------------------------------
// A float32 tensor of these sizes beside x.
float* beside(const at::Tensor& x, PyObject* o, std::initializer_list<int64_t> sizes) {
  const at::Tensor& t = tensor(o);
  if (t.scalar_type() != at::kFloat || t.device() != x.device() || t.sizes() != at::IntArrayRef(sizes) || t.is_neg()) throw NotPlain{};
  return static_cast<float*>(pointer(t));
}
constexpr int kEncoderParams = 12;
// x, or a tensor of its sizes, on the current device: its pointer, and the sizes into e.
float* input(const at::Tensor& x, tempo_encoder* e) {
  if (x.scalar_type() != at::kFloat || x.dim() != 3 || x.is_neg()) throw NotPlain{};
  float* p = static_cast<float*>(pointer(x));
  if (x.device().index() != c10::hip::current_device()) throw NotPlain{};
  e->batch = x.size(0);
  e->seq = x.size(1);
  e->hidden = x.size(2);
  return p;
}
int64_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw NotPlain{};
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw NotPlain{};
  return v;
}
// The layer of x with heads, eps1, eps2, p, seed and kind at a[0 .. 5], and its parameters at w.
tempo_encoder encoder(const at::Tensor& x, PyObject* const* a, PyObject* const* w) {
  tempo_encoder e{};
  e.x = input(x, &e);
  e.heads = integer(a[0]);
  e.eps1 = real(a[1]);
  e.eps2 = real(a[2]);
  e.p = real(a[3]);
  e.seed = bits64(a[4]);
  e.kind = gelu_kind(a[5]);
  const at::Tensor& w1 = tensor(w[4]);
  if (w1.dim() != 2) throw NotPlain{};
  e.ffn = w1.size(0);
  const int64_t H = e.hidden, F = e.ffn;
  e.wqkv = beside(x, w[0], {3 * H, H});
  e.bqkv = beside(x, w[1], {3 * H});
  e.wproj = beside(x, w[2], {H, H});
  e.bproj = beside(x, w[3], {H});
  e.w1 = beside(x, w[4], {F, H});
  e.b1 = beside(x, w[5], {F});
  e.w2 = beside(x, w[6], {H, F});
  e.b2 = beside(x, w[7], {H});
  e.gamma1 = beside(x, w[8], {H});
  e.beta1 = beside(x, w[9], {H});
  e.gamma2 = beside(x, w[10], {H});
  e.beta2 = beside(x, w[11], {H});
  if (!tempo_encoder_takes(&e)) throw NotPlain{};
  return e;
}
float* data(const at::Tensor& t) { return t.defined() ? static_cast<float*>(t.data_ptr()) : nullptr; }
// The next offset of the generator, from where a module keeps the last one.  Taken under the interpreter's lock, once nothing
// can send the call elsewhere any more: threads that share the module draw other bits, and a call made of its parts takes its own.
PyObject* next_offset(PyObject* module, uint64_t* offset) {
  PyObject* last = PyDict_CheckExact(module) ? PyDict_GetItemString(module, "offset") : nullptr;
  if (!last || !PyLong_CheckExact(last)) throw NotPlain{};
  PyObject* one = PyLong_FromLong(1);
  PyObject* next = one ? PyNumber_Add(last, one) : nullptr;
  Py_XDECREF(one);
  if (!next || PyDict_SetItemString(module, "offset", next) != 0) {
    Py_XDECREF(next);
    throw NotPlain{};
  }
  *offset = bits64(next);
  return next;
}
// What `front` owns, then the tensors, an undefined one as None.
template <size_t F, size_t N>
PyObject* result(PyObject* const (&front)[F], const at::Tensor* const (&t)[N]) {
  PyObject* r = PyTuple_New(F + N);
  for (size_t i = 0; i < F; ++i) {
    if (r) PyTuple_SET_ITEM(r, i, front[i]);
    else Py_XDECREF(front[i]);
  }
  for (size_t i = 0; r && i < N; ++i) PyTuple_SET_ITEM(r, F + i, THPVariable_Wrap(*t[i]));  // None for an undefined one
  return r;
}

// x, key_len, the attention core's __dict__, heads, eps1, eps2, p, seed, kind, 12 parameters -> status, offset and what the
// backward needs
TEMPO_METHOD(encoder_fwd) {
  if (nargs != 9 + kEncoderParams) Py_RETURN_NONE;
  at::Tensor qkv, probs, keep, ctxt, y1, rstd1, h, side, y2, rstd2;
  tempo_status status;
  PyObject* offset;
  HANDLE_TH_ERRORS
  try {
    const at::Tensor& x = tensor(a[0]);
    tempo_encoder e = encoder(x, a + 3, a + 9);
    if (a[1] != Py_None) {
      const at::Tensor& k = tensor(a[1]);
      if (k.scalar_type() != at::kInt || k.numel() != e.batch || k.device() != x.device()) throw NotPlain{};
      e.key_len = static_cast<int32_t*>(pointer(k));
    }
    const int64_t B = e.batch, S = e.seq, T = B * S, n = B * e.heads * S * S;
    const auto floats = x.options().requires_grad(false), words = floats.dtype(at::kInt);
    qkv = at::empty({T, 3 * e.hidden}, floats);
    probs = at::empty({B, e.heads, S, S}, floats);
    at::Tensor out = at::empty({B, e.heads, S, S}, floats);
    keep = at::empty({(n + 31) / 32}, words);
    ctxt = at::empty({T, e.hidden}, floats);
    y1 = at::empty({T, e.hidden}, floats);
    rstd1 = at::empty({T}, floats);
    h = at::empty({T, e.ffn}, floats);
    side = at::empty({(T * e.ffn + 31) / 32}, words);
    y2 = at::empty({B, S, e.hidden}, floats);
    rstd2 = at::empty({T}, floats);
    e.qkv = data(qkv);
    e.probs = data(probs);
    e.keep = reinterpret_cast<uint32_t*>(keep.data_ptr());
    e.ctxt = data(ctxt);
    e.y1 = data(y1);
    e.rstd1 = data(rstd1);
    e.h = data(h);
    e.side = reinterpret_cast<uint32_t*>(side.data_ptr());
    e.y2 = data(y2);
    e.rstd2 = data(rstd2);
    void* st = stream();
    offset = next_offset(a[2], &e.offset);
    PyThreadState* state = PyEval_SaveThread();
    status = tempo_encoder_fwd(&e, data(out), st);
    PyEval_RestoreThread(state);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  const at::Tensor* all[] = {&qkv, &probs, &keep, &ctxt, &y1, &rstd1, &h, &side, &y2, &rstd2};
  PyObject* front[] = {PyLong_FromLong(status), offset};
  return result(front, all);
  END_HANDLE_TH_ERRORS
}

// dy, wanted (bits: x, then the parameters), heads, ffn, p, seed, offset, kind, and of the forward x, wqkv, wproj, w1, w2, gamma1, beta1,
// gamma2, beta2, qkv, probs, keep (or None: drawn again), ctxt, y1, rstd1, h, side, y2, rstd2, of which only those are looked at
// that the wanted gradients need -> status and the 13 gradients
TEMPO_METHOD(encoder_bwd) {
  if (nargs != 8 + 19) Py_RETURN_NONE;
  at::Tensor dx, dw[kEncoderParams];
  tempo_status status = TEMPO_OK;
  HANDLE_TH_ERRORS  // out of memory, as torch raises it
  try {
    const at::Tensor& out_grad = tensor(a[0]);
    const uint64_t wanted = bits64(a[1]);
    tempo_encoder e{};
    const float* dy = input(out_grad, &e);
    e.heads = integer(a[2]);
    e.ffn = integer(a[3]);
    e.p = real(a[4]);
    e.seed = bits64(a[5]);
    e.offset = bits64(a[6]);
    e.kind = gelu_kind(a[7]);
    if (!tempo_encoder_takes(&e)) throw NotPlain{};
    const int64_t B = e.batch, S = e.seq, T = B * S, H = e.hidden, F = e.ffn, n = B * e.heads * S * S;
    auto want = [&](int first, int last) { return (wanted >> first & ((uint64_t{2} << (last - first)) - 1)) != 0; };
    // bits: 0 x, 1 2 qkv, 3 4 proj, 5 6 fc1, 7 8 fc2, 9 10 ln1, 11 12 ln2
    const bool attention = want(0, 2), first = want(0, 4) || want(9, 10), second = first || want(5, 6);
    PyObject* const* o = a + 8;
    auto kept = [&](bool needed, std::initializer_list<int64_t> sizes) {
      PyObject* t = *o++;
      return needed ? beside(out_grad, t, sizes) : nullptr;
    };
    auto bits = [&](bool needed, int64_t elements) {
      PyObject* t = *o++;
      if (!needed) return static_cast<uint32_t*>(nullptr);
      if (tensor(t).device() != out_grad.device()) throw NotPlain{};
      return mask_words(t, elements);
    };
    e.x = kept(want(1, 1), {B, S, H});
    e.wqkv = kept(want(0, 0), {3 * H, H});
    e.wproj = kept(attention, {H, H});
    e.w1 = kept(first, {F, H});
    e.w2 = kept(second, {H, F});
    e.gamma1 = kept(first, {H});
    e.beta1 = kept(first, {H});
    e.gamma2 = kept(true, {H});
    e.beta2 = kept(true, {H});
    e.qkv = kept(attention, {T, 3 * H});
    e.probs = kept(attention, {B, e.heads, S, S});
    e.keep = bits(attention && *o != Py_None, n);
    e.ctxt = kept(want(3, 3), {T, H});
    e.y1 = kept(first || want(5, 5), {T, H});
    e.rstd1 = kept(first, {T});
    e.h = kept(second || want(7, 7), {T, F});
    e.side = bits(second, T * F);
    e.y2 = kept(true, {B, S, H});
    e.rstd2 = kept(true, {T});
    const auto floats = out_grad.options().requires_grad(false);
    auto grad = [&](int i, at::IntArrayRef sizes) { return data(dw[i] = at::empty(sizes, floats)); };
    auto wanted_grad = [&](int i, at::IntArrayRef sizes) { return want(i + 1, i + 1) ? grad(i, sizes) : nullptr; };
    tempo_encoder_grads g{};
    at::Tensor ds = at::empty({T, H}, floats), dh, dy1;
    at::Tensor workspace = at::empty({static_cast<int64_t>(tempo_layernorm_bwd_workspace_bytes(T, H))}, floats.dtype(at::kByte));
    const size_t workspace_bytes = workspace.numel();
    void* st = stream();
    auto run = [&](auto&& call) {
      if (status != TEMPO_OK) return;
      PyThreadState* state = PyEval_SaveThread();
      status = call();
      PyEval_RestoreThread(state);
    };
    g.dgamma2 = grad(10, {H});
    g.dbeta2 = grad(11, {H});
    g.dw2 = wanted_grad(6, {H, F});
    g.db2 = wanted_grad(7, {H});
    g.dw1 = wanted_grad(4, {F, H});
    g.db1 = wanted_grad(5, {F});
    if (first) dy1 = at::empty({T, H}, floats);
    if (second) dh = at::empty({T, F}, floats);
    run([&] {
      return tempo_encoder_bwd_ffn(&e, &g, dy, data(ds), data(dh), data(dy1), workspace.data_ptr(), workspace_bytes, st);
    });
    dh.reset();
    if (first) {
      g.dgamma1 = grad(8, {H});
      g.dbeta1 = grad(9, {H});
      run([&] {
        return tempo_encoder_bwd_norm(&e, &g, data(dy1), data(ds), workspace.data_ptr(), workspace_bytes, st);
      });
    }
    workspace.reset();
    if (want(0, 4)) {
      at::Tensor dctxt, dqkv, dout, out;
      g.dwproj = wanted_grad(2, {H, H});
      g.dbproj = wanted_grad(3, {H});
      if (attention) {
        dctxt = dy1;  // has been read
        dqkv = at::empty({T, 3 * H}, floats);
        dout = at::empty({B, e.heads, S, S}, floats);
        out = at::empty({B, e.heads, S, S}, floats);
        g.dwqkv = wanted_grad(0, {3 * H, H});
        g.dbqkv = wanted_grad(1, {3 * H});
        if (want(0, 0)) g.dx = data(dx = at::empty({B, S, H}, floats));
      }
      run([&] {
        return tempo_encoder_bwd_attention(&e, &g, data(ds), data(dctxt), data(dqkv), data(dout), data(out), st);
      });
    }
    for (int i = 8; i < kEncoderParams; ++i)  // the LayerNorms'
      if (!want(i + 1, i + 1)) dw[i].reset();
  } catch (const NotPlain&) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  const at::Tensor* all[] = {&dx, dw, dw + 1, dw + 2, dw + 3, dw + 4, dw + 5, dw + 6, dw + 7, dw + 8, dw + 9, dw + 10, dw + 11};
  PyObject* front[] = {PyLong_FromLong(status)};
  return result(front, all);
  END_HANDLE_TH_ERRORS
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
                         TEMPO_ENTRY(encoder_fwd),
                         TEMPO_ENTRY(encoder_bwd),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
