// Float32 activations and the derivatives of their inverses on the device: for the kernels of gelu.hip and for the
// products of an encoder layer that end or begin with one.
#pragma once

#include <type_traits>

#include "tempo_device.h"
#include "tempo_host.h"

#define TEMPO_TABLE_QUAL __device__
#include "gelu_tables.inc"

namespace tempo {
namespace {

template <int KIND>
struct GeluConst;
// Per activation: the minimum (x* as compared in float32, y* split hi + lo), the number of
// right-branch and left-near pieces of the backward table, the rows of that table, and how many
// bf16 patterns lower the left branch's lookup window starts.
#define TEMPO_ACT_CONST(KIND, UPPER, lower)                                                  \
  template <>                                                                                \
  struct GeluConst<KIND> {                                                                   \
    static constexpr uint32_t xstar = TEMPO_GELU_##UPPER##_XSTAR_F32;                        \
    static constexpr uint32_t ys_hi = TEMPO_GELU_##UPPER##_YSTAR_HI;                         \
    static constexpr uint32_t ys_lo = TEMPO_GELU_##UPPER##_YSTAR_LO;                         \
    static constexpr int NR = TEMPO_GELU_##UPPER##_NR;                                       \
    static constexpr int NL = TEMPO_GELU_##UPPER##_NL;                                       \
    static constexpr int kBwdRows = TEMPO_GELU_##UPPER##_BWD_ROWS;                           \
    static constexpr int kLutLeftShift = TEMPO_GELU_##UPPER##_LUT_LEFT_SHIFT;                \
    __device__ static const uint32_t (*bwd_table())[4] { return tempo_gelu_bwd_table_##lower; } \
    __device__ static const uint32_t* lut_fwd() { return tempo_gelu_lut_fwd_##lower; }       \
    __device__ static const uint32_t* lut_bwd() { return tempo_gelu_lut_bwd_##lower; }       \
  };
TEMPO_ACT_CONST(TEMPO_GELU_ERF, ERF, erf)
TEMPO_ACT_CONST(TEMPO_GELU_TANH, TANH, tanh)
TEMPO_ACT_CONST(kActSilu, SILU, silu)
#undef TEMPO_ACT_CONST

__device__ __forceinline__ float cubic(const f32x4 c, float z) {
  return fmaf(fmaf(fmaf(c.w, z, c.z), z, c.y), z, c.x);
}

// GELU(x) = x Phi(x), erf form.  Phi(x) = 1/2 erfc(-x / sqrt 2); for z >= 0,
// erfc(z) = exp(-z^2) erfcx(z), and 1/2 erfcx(z) (1 + z/2) is one polynomial of degree 8 in
// t = 1 / (1 + z/2) (relative error 9e-8 up to |x| = 9; beyond, the exponential has long made
// Phi 0 or 1).  With w = |x| sqrt(log2(e)/2) the exponential is exp2(-w^2).  x < 0 takes the
// small value itself, so the left tail keeps its relative accuracy, and the product with x comes
// last, so the zero at x = 0 is exact.  No table: the kernel needs no LDS.
__device__ __forceinline__ float gelu_erf_value(float x) {
  const float w = fabsf(x) * as_f32(TEMPO_GELU_ERFC_W_SCALE);
  const float t = __builtin_amdgcn_rcpf(fmaf(w, as_f32(TEMPO_GELU_ERFC_T_FACTOR), 1.0f));
  const float u = fmaf(t, as_f32(TEMPO_GELU_ERFC_UA), as_f32(TEMPO_GELU_ERFC_UB));
  static_assert(TEMPO_GELU_ERFC_DEG == 8, "Horner chain below");
  float q = as_f32(TEMPO_GELU_ERFC_Q8);
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q7));
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q6));
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q5));
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q4));
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q3));
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q2));
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q1));
  q = fmaf(q, u, as_f32(TEMPO_GELU_ERFC_Q0));
  const float half_erfc = t * q * __builtin_amdgcn_exp2f(-(w * w));  // 1/2 erfc(|x| / sqrt 2)
  const float phi = (x < 0.0f) ? half_erfc : 1.0f - half_erfc;
  return x * phi;  // NaN stays NaN
}

// GELU(x), tanh form written as x * sigmoid(2u): no cancellation on the left tail.
__device__ __forceinline__ float gelu_tanh_value(float x) {
  const float k = 0.7978845608028654f;      // sqrt(2/pi)
  const float ka = 0.7978845608028654f * 0.044715f;
  const float m2log2e = -2.0f * 1.4426950408889634f;
  const float inner = fmaf(x * x, ka, k);
  const float e = __builtin_amdgcn_exp2f(m2log2e * x * inner);  // exp(-2u)
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

// SiLU(x) = x * sigmoid(x); exp overflows to +inf on the far left, which gives -0.
__device__ __forceinline__ float silu_value(float x) {
  const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * x);  // exp(-x)
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

template <int KIND>
__device__ __forceinline__ float act_value(float x) {
  if constexpr (KIND == TEMPO_GELU_ERF) return gelu_erf_value(x);
  else if constexpr (KIND == TEMPO_GELU_TANH) return gelu_tanh_value(x);
  else return silu_value(x);
}

// d(y, m) = GELU'(GELU*^-1(y, m)).
template <int KIND>
__device__ __forceinline__ float gelu_composite(float y, bool right, const f32x4* tab) {
  const float ys_hi = as_f32(GeluConst<KIND>::ys_hi);
  const float ys_lo = as_f32(GeluConst<KIND>::ys_lo);
  const float t = fmaxf((y - ys_hi) - ys_lo, 0.0f);
  const float s = __builtin_amdgcn_sqrtf(t);
  const float c = right ? static_cast<float>(TEMPO_GELU_CR) : static_cast<float>(TEMPO_GELU_CL);
  constexpr int NR = GeluConst<KIND>::NR, NL = GeluConst<KIND>::NL;
  const float umax = right ? (NR - 0.00001f) : (NL - 0.00001f);
  const int base = right ? 0 : NR;
  const float u = fminf(s * c, umax);
  const float fl = floorf(u);
  const float z_s = u - fl;
  const int idx_s = static_cast<int>(fl) + base;
  // left tail: quarter-octaves of -y below 2^TAIL_TOP_EXP
  const float ny = -y;
  const uint32_t bits = as_u32(ny);
  constexpr int kRem = 23 - TEMPO_GELU_TAIL_SUB_BITS;
  constexpr uint32_t kTop =
      ((127u + TEMPO_GELU_TAIL_TOP_EXP - 1u) << TEMPO_GELU_TAIL_SUB_BITS) |
      ((1u << TEMPO_GELU_TAIL_SUB_BITS) - 1u);
  const uint32_t it = min(kTop - (bits >> kRem), static_cast<uint32_t>(TEMPO_GELU_NT - 1));
  const float z_t = static_cast<float>(bits & ((1u << kRem) - 1u));
  const bool tail = !right && (ny < 0.0625f);
  static_assert(TEMPO_GELU_TAIL_TOP_EXP == -4, "tail threshold literal");
  const int idx = tail ? static_cast<int>(it) + (NR + NL) : idx_s;
  const float z = tail ? z_t : z_s;
  float d = cubic(tab[idx], z);
  return (y != y) ? y : d;
}

}  // namespace
}  // namespace tempo
