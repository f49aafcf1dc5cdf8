// Float32 matrix products of the encoder layer (no HIP in here beyond the stream).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/tempo.h"

namespace tempo {

constexpr int kTile = 32;  // rows and columns of a matrix instruction, and of the smallest tile

// One operand of a product: element (row, k) at p[row * ld + k], or at p[k * ld + row] if k_major.  The slice b of a
// batch starts (b / inner) * outer_stride + (b % inner) * inner_stride elements further on.
struct MatSide {
  const float* p;
  int64_t ld;
  int64_t outer_stride, inner_stride;
  bool k_major;
};

// c[m][n] = alpha * sum_k a(m, k) b(n, k) + bias[n] + add[m][n]
struct Matmul {
  MatSide a, b;
  float* c;            // null in a group: not computed, but for the sums below
  int64_t ldc, c_outer, c_inner;
  const float* bias;   // [N] or null
  const float* add;    // laid out as c, or null; may be c
  float* a_sums;       // [M]: sum_k a(m, k), or null (k-major a, a single slice)
  float alpha;
  int M, N, K, batch, inner;
  int n_counted;       // what the choice of a tile takes for N
  // Float32 GELU of c, or its backward from the outputs act_y, laid out as c; side: the bits at or right of the minimum,
  // written or read (N a multiple of 8, a single slice, no addend).
  enum Act { kNone, kForward, kBackward } act = kNone;
  tempo_gelu_kind kind = TEMPO_GELU_ERF;
  const float* act_y = nullptr;
  uint8_t* side = nullptr;
};
tempo_status launch_matmul(const Matmul& g, hipStream_t st);
// g (k-major b only) and one or two products of one size with two k-major operands, none of which needs another.  g or h0
// may have no c; everything else gets the bits that it has beside it.
tempo_status launch_matmul_group(const Matmul& g, const Matmul& h0, const Matmul* h1, hipStream_t st);

}  // namespace tempo
