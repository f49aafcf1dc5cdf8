// Float32 matrix products of the encoder layer on the matrix cores (v_mfma_f32_32x32x2_f32): small ones, whose operands come
// from the L2s and the Infinity Cache, where what a library call costs the host is more than the product takes.
//
// Bound by what a wave waits for between its matrix instructions (operands through LDS, one barrier a step) and by uneven
// numbers of tiles per compute unit, then by the matrix cores: [256, 768] x [768, 2304] 15.0 us, 5.9 at their rate (154
// TFLOP/s measured; rocBLAS 16.2), [256, 3072] x [3072, 768] 19.3 (7.8; 16.7), [2304, 256] x [256, 768] 14.8 (5.9; 12.5), 24
// heads of [128, 64] x [64, 128] 4.1 (8.0 and two copies).  At [2048, 1024] x [1024, 4096] 152 (112; 125).
// Steps of k are fetched DEPTH + 2 ahead, written to LDS two ahead and read from there one ahead of the matrix instructions.
// With one step fetched ahead and everything else in sequence [256, 768] x [768, 2304] takes 17.5, [256, 3072] x [3072, 768] 28.
#include "gelu_f32.h"
#include "matmul.h"

namespace tempo {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef f32x4 f32x4_word __attribute__((aligned(4)));  // 16 bytes at any float's address

// R rows by KT values of k of one operand: DEPTH steps ahead in registers, then LDS.
template <bool KM, int R, int KT, int THREADS, int DEPTH>
struct Stage {
  static constexpr int kLd = KM ? R + 8 : KT + 4;  // row pitch in LDS: reads of a wave meet each bank once
  static constexpr int kFloats = KM ? KT * kLd : R * kLd;
  static constexpr int kPieces = R * KT / 4 / THREADS;
  static_assert(kPieces * 4 * THREADS == R * KT, "whole pieces per lane");
  static constexpr int kRun = (KM ? R : KT) / 4;  // pieces side by side

  const float* p[kPieces];
  int64_t step;  // elements from one step to the next
  f32x4 v[DEPTH][kPieces];

  // Pieces of rows that do not exist read the last ones that do: they make elements of c that nothing stores.
  __device__ __forceinline__ Stage(const MatSide& s, int outer, int inner, int row0, int rows) {
    const float* base = s.p + outer * s.outer_stride + inner * s.inner_stride;
    step = KM ? KT * s.ld : KT;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int at = i * THREADS + static_cast<int>(threadIdx.x);
      if constexpr (KM) p[i] = base + at / kRun * s.ld + min(row0 + at % kRun * 4, (rows - 1) & ~3);
      else p[i] = base + min(row0 + at / kRun, rows - 1) * s.ld + at % kRun * 4;
    }
  }
  // Whole steps (see full_steps()).
  __device__ __forceinline__ void load(int slot, int s) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) v[slot][i] = *reinterpret_cast<const f32x4_word*>(p[i] + s * step);
  }
  // The last step: zeros for the values of k that do not exist.
  __device__ __forceinline__ void load_rest(f32x4 (&rest)[kPieces], int s, int row0, int rows, int K) const {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int at = i * THREADS + static_cast<int>(threadIdx.x);
      const int k = s * KT + (KM ? at / kRun : at % kRun * 4);
      const int left = KM ? (k < K ? rows - min(row0 + at % kRun * 4, (rows - 1) & ~3) : 0) : K - k;
      const float* q = p[i] + s * step;
      rest[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (left >= 4) {
        rest[i] = *reinterpret_cast<const f32x4_word*>(q);
      } else if (left > 0) {
        rest[i].x = q[0];
        if (left > 1) rest[i].y = q[1];
        if (left > 2) rest[i].z = q[2];
      }
    }
  }
  __device__ static __forceinline__ void store(float* lds, const f32x4 (&w)[kPieces]) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int at = i * THREADS + static_cast<int>(threadIdx.x);
      *reinterpret_cast<f32x4*>(lds + at / kRun * kLd + at % kRun * 4) = w[i];
    }
  }
  // Values k .. k + 3 of row `row`
  __device__ static __forceinline__ f32x4 read(const float* lds, int row, int k) {
    if constexpr (KM) {
      const float* q = lds + k * kLd + row;
      return f32x4{q[0], q[kLd], q[2 * kLd], q[3 * kLd]};
    } else {
      return *reinterpret_cast<const f32x4*>(lds + row * kLd + k);
    }
  }
};

// Steps of KT values of k that are loaded in whole 16-byte pieces.  Where the rows of a k-major operand are no multiple of
// a piece, their last piece ends in the next row, so that the last row takes no part.
__device__ __forceinline__ int full_steps(const Matmul& g, bool akm, bool bkm, int KT) {
  const bool over = (akm && g.M % 4 != 0) || (bkm && g.N % 4 != 0);
  return (over ? g.K - 1 : g.K) / KT;
}

// A workgroup owns BM x BN elements of c.  Each of its waves owns 32 x 32 of them for a KS-th of every KT values of k.
template <bool AKM_, bool BKM_, int BM_, int BN_, int KS_, int KT_, int DEPTH_>
struct Config {
  static constexpr bool AKM = AKM_, BKM = BKM_;
  static constexpr int BM = BM_, BN = BN_, KS = KS_, KT = KT_, DEPTH = DEPTH_;
  static constexpr int kWavesM = BM / kTile, kWavesN = BN / kTile;
  static constexpr int kThreads = kWave * kWavesM * kWavesN * KS;
  using A = Stage<AKM, BM, KT, kThreads, DEPTH>;
  using B = Stage<BKM, BN, KT, kThreads, DEPTH>;
  static constexpr int kBuffer = A::kFloats + B::kFloats;
  static constexpr int kExchange = KS > 1 ? KS * kWavesM * kWavesN * 16 * kWave : 0;
  static constexpr int kStaged = 2 * kBuffer > kExchange ? 2 * kBuffer : kExchange;
  static constexpr int kLds = kStaged + (AKM ? KS * BM : 0);  // floats
  static int64_t tiles(const Matmul& g) { return int64_t{(g.M + BM - 1) / BM} * ((g.N + BN - 1) / BN) * g.batch; }
};

// Tile `block` of `total`, in the order of the launch.
// ACT, KIND: g.act and g.kind.  table: rows of the backward's cubics in LDS.
template <typename C, int ACT, int KIND>
__device__ __forceinline__ void matmul_tile(const Matmul& g, int block, int total, float* lds, const f32x4* table) {
  constexpr bool AKM = C::AKM, BKM = C::BKM;
  constexpr int BM = C::BM, BN = C::BN, KS = C::KS, KT = C::KT, DEPTH = C::DEPTH;
  constexpr int kWavesM = C::kWavesM, kThreads = C::kThreads;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  constexpr int KW = KT / KS;
  static_assert(KW % 8 == 0, "whole steps of 8");
  using A = typename C::A;
  using B = typename C::B;
  constexpr int kBuffer = C::kBuffer;
  float* const sums = lds + C::kStaged;  // AKM: [KS][BM]

  // Neighbouring workgroups go to different XCDs, each of which has its own L2: every XCD takes a run of tiles, which
  // share columns of c.
  constexpr int kXcds = 8;
  const int xcd = block % kXcds, each = total / kXcds, more = total % kXcds;
  const int tile = xcd * each + min(xcd, more) + block / kXcds;
  const int slice = tile / (tiles_m * tiles_n), in_slice = tile % (tiles_m * tiles_n);
  const int n0 = in_slice / tiles_m * BN, m0 = in_slice % tiles_m * BM;
  const int outer = slice / g.inner, inner = slice % g.inner;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const int ks = wave % KS, at = wave / KS, wm = at % kWavesM, wn = at / kWavesM;
  const int l32 = lane % kTile, half = lane / kTile;

  A a(g.a, outer, inner, m0, g.M);
  B b(g.b, outer, inner, n0, g.N);
  const int steps = full_steps(g, AKM, BKM, KT);
  const bool rest = steps * KT < g.K;
  f32x4 rest_a[A::kPieces], rest_b[B::kPieces];
  if (rest) {
    a.load_rest(rest_a, steps, m0, g.M, g.K);
    b.load_rest(rest_b, steps, n0, g.N, g.K);
  }
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  // AKM: the sums of a, of a few steps and of all before, so that long columns do not add up in one chain
  f32x4 asum = {0.0f, 0.0f, 0.0f, 0.0f}, asum_before = asum;
  constexpr int kFrags = KW / 8;
  f32x4 fa[2][kFrags], fb[2][kFrags];
  // No branch around the loads: behind one, the compiler waits for all that are under way.  Beyond the last step they
  // read that one again.
  auto fetch = [&](int slot, int s) {
    a.load(slot, min(s, steps - 1));
    b.load(slot, min(s, steps - 1));
  };
  auto put = [&](int slot, int parity) {
    A::store(lds + parity * kBuffer, a.v[slot]);
    B::store(lds + parity * kBuffer + A::kFloats, b.v[slot]);
  };
  auto get = [&](int parity) {
    const float* la = lds + parity * kBuffer;
    const float* lb = la + A::kFloats;
#pragma unroll
    for (int kk = 0; kk < kFrags; ++kk) {
      const int k = ks * KW + kk * 8 + half * 4;
      fa[parity][kk] = A::read(la, wm * kTile + l32, k);
      fb[parity][kk] = B::read(lb, wn * kTile + l32, k);
    }
  };
  auto multiply = [&](int parity, int from, int to) {
#pragma unroll
    for (int kk = from; kk < to; ++kk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[parity][kk][i], fa[parity][kk][i], acc, 0, 0, 0);
        if constexpr (AKM) asum[i] += fa[parity][kk][i];
      }
    }
  };
  // While the matrix cores work on step s, the operands of s + 1 come from LDS and step s + 2 is written there: into the
  // buffer of s, which all waves have read before the last barrier.
  static_assert(DEPTH % 2 == 0, "parities below");
  if (steps > 0) {
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) fetch(j, j);
    put(0, 0);
    fetch(0, DEPTH);
    put(1, 1);
    fetch(1, DEPTH + 1);
    lds_barrier();
    get(0);
    lds_barrier();
    auto one = [&](int j, int s) {
      get((j + 1) & 1);
      multiply(j & 1, 0, (kFrags + 1) / 2);
      put((j + 2) % DEPTH, j & 1);
      fetch((j + 2) % DEPTH, s + 2 + DEPTH);
      multiply(j & 1, (kFrags + 1) / 2, kFrags);
      lds_barrier();
    };
    const int whole = steps / DEPTH * DEPTH;
    for (int s = 0; s < whole; s += DEPTH) {
#pragma unroll
      for (int j = 0; j < DEPTH; ++j) one(j, s + j);
      if constexpr (AKM) {
        asum_before += asum;
        asum = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
#pragma unroll
    for (int j = 0; j < DEPTH - 1; ++j) {
      if (whole + j < steps) one(j, whole + j);
    }
  }
  if (rest) {
    A::store(lds, rest_a);
    B::store(lds + A::kFloats, rest_b);
    lds_barrier();
    get(0);
    multiply(0, 0, kFrags);
    lds_barrier();
  }

  if constexpr (AKM) {
    if (g.a_sums && n0 == 0) {  // uniform over the workgroup
      asum += asum_before;
      float v = (asum[0] + asum[1]) + (asum[2] + asum[3]);
      v = across_rows<32>(v, [](float x, float y) { return x + y; });
      if (wn == 0 && half == 0) sums[ks * BM + wm * kTile + l32] = v;
    }
  }
  // Register r of a lane is element (m = lane % 32, n = 8 (r / 4) + 4 (lane / 32) + r % 4) of the wave's 32 x 32: four
  // adjacent ones per r / 4.  With KS > 1 the waves of an element exchange their sums; each adds up 4 / KS of the four
  // groups.
  const int m = m0 + wm * kTile + l32;
  auto finish = [&](int q, f32x4 v) {
    const int n = n0 + wn * kTile + 8 * q + 4 * half;
    const int left = m < g.M && (!AKM || g.c) ? g.N - n : 0;
    const int64_t e = outer * g.c_outer + inner * g.c_inner + m * g.ldc + n;
    v *= g.alpha;
    if constexpr (ACT == Matmul::kForward) {
      // a group of both halves of the wave is 8 adjacent elements: a byte of the mask
      if (g.bias && left > 0) v += *reinterpret_cast<const f32x4_word*>(g.bias + n);
      uint32_t bits = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bits |= (v[i] >= as_f32(GeluConst<KIND>::xstar) ? 1u : 0u) << (4 * half + i);
        v[i] = act_value<KIND>(v[i]);
      }
      const auto both = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
      if (left <= 0) return;
      *reinterpret_cast<f32x4_word*>(g.c + e) = v;
      if (half == 0) g.side[e >> 3] = static_cast<uint8_t>(both[0] | both[1]);
      return;
    }
    if (left <= 0) return;
    if constexpr (ACT == Matmul::kBackward) {
      const f32x4 y = *reinterpret_cast<const f32x4_word*>(g.act_y + e);
      const uint32_t bits = g.side[e >> 3] >> (4 * half);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] *= gelu_composite<KIND>(y[i], (bits >> i) & 1u, table);
    }
    if (left >= 4) {
      if (g.bias) v += *reinterpret_cast<const f32x4_word*>(g.bias + n);
      if (g.add) v += *reinterpret_cast<const f32x4_word*>(g.add + e);
      *reinterpret_cast<f32x4_word*>(g.c + e) = v;
    } else {
      for (int i = 0; i < left; ++i) {
        float w = v[i];
        if (g.bias) w += g.bias[n + i];
        if (g.add) w += g.add[e + i];
        g.c[e + i] = w;
      }
    }
  };
  if constexpr (KS == 1) {
    if constexpr (AKM) lds_barrier();
#pragma unroll
    for (int q = 0; q < 4; ++q) finish(q, f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]});
  } else {
    f32x4* const x = reinterpret_cast<f32x4*>(lds) + static_cast<size_t>(at) * KS * 4 * kWave;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      x[(ks * 4 + q) * kWave + lane] =
          f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    lds_barrier();
#pragma unroll
    for (int q0 = 0; q0 < 4; q0 += KS) {
      const int q = q0 + ks;
      if (q < 4) {
        f32x4 v = x[q * kWave + lane];
#pragma unroll
        for (int s = 1; s < KS; ++s) v += x[(s * 4 + q) * kWave + lane];
        finish(q, v);
      }
    }
  }
  if constexpr (AKM) {
    if (g.a_sums && n0 == 0) {
      for (int i = threadIdx.x; i < BM && m0 + i < g.M; i += kThreads) {
        float v = sums[i];
#pragma unroll
        for (int s = 1; s < KS; ++s) v += sums[s * BM + i];
        g.a_sums[m0 + i] = v;
      }
    }
  }
}

template <typename C, int ACT, int KIND>
__global__ __launch_bounds__(C::kThreads) void matmul_kernel(Matmul g) {
  __shared__ __attribute__((aligned(16))) float lds[C::kLds];
  matmul_tile<C, ACT, KIND>(g, blockIdx.x, gridDim.x, lds, nullptr);
}
template <typename C>
tempo_status go(const Matmul& g, hipStream_t st) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(C::tiles(g)), dim3(C::kThreads), 0, st, g);
    return launch_status();
  };
  if (g.act == Matmul::kNone) return launch(matmul_kernel<C, Matmul::kNone, 0>);
  if constexpr (!C::BKM) {
    if (g.act == Matmul::kForward)
      return launch(g.kind == TEMPO_GELU_TANH ? matmul_kernel<C, Matmul::kForward, TEMPO_GELU_TANH>
                                              : matmul_kernel<C, Matmul::kForward, TEMPO_GELU_ERF>);
  }
  return TEMPO_ERR_UNSUPPORTED;
}

// Products that need nothing of each other in one launch: g, and one or two of the same size.
template <typename C, typename D, int ACT, int KIND>
__global__ __launch_bounds__(C::kThreads) void matmul_group_kernel(Matmul g, Matmul h0, Matmul h1, int g_tiles, int h_tiles) {
  static_assert(C::kThreads == D::kThreads, "one workgroup size");
  constexpr int kRows = ACT == Matmul::kBackward ? GeluConst<KIND>::kBwdRows : 0;
  constexpr int kStaged = C::kLds > D::kLds ? C::kLds : D::kLds;
  static_assert(kStaged % 4 == 0, "table rows of 16 bytes behind it");
  __shared__ __attribute__((aligned(16))) float lds[kStaged + 4 * kRows];
  const int block = blockIdx.x;
  if (block < g_tiles) {  // none of it if g is not computed
    f32x4* const table = reinterpret_cast<f32x4*>(lds + kStaged);
    if constexpr (ACT == Matmul::kBackward) {  // ordered by the barriers of the loop
      for (int i = threadIdx.x; i < kRows; i += C::kThreads)
        table[i] = *reinterpret_cast<const f32x4*>(GeluConst<KIND>::bwd_table()[i]);
    }
    return matmul_tile<C, ACT, KIND>(g, block, g_tiles, lds, table);
  }
  const int rest = block - g_tiles;
  if (rest < h_tiles) matmul_tile<D, Matmul::kNone, 0>(h0, rest, h_tiles, lds, nullptr);
  else matmul_tile<D, Matmul::kNone, 0>(h1, rest - h_tiles, h_tiles, lds, nullptr);
}
template <typename C, typename D>
tempo_status go_group(const Matmul& g, const Matmul& h0, const Matmul* h1, hipStream_t st) {
  // The sums are made by the tiles of the first columns, which come first.
  const int64_t g_tiles = g.c ? C::tiles(g) : 0;
  const int64_t h_tiles = h0.c ? D::tiles(h0) : h0.a_sums ? (h0.M + D::BM - 1) / D::BM : 0;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g_tiles + (h1 ? 2 : 1) * h_tiles), dim3(C::kThreads), 0, st, g, h0, h1 ? *h1 : h0,
                       static_cast<int>(g_tiles), static_cast<int>(h_tiles));
    return launch_status();
  };
  if (g.act == Matmul::kNone) return launch(matmul_group_kernel<C, D, Matmul::kNone, 0>);
  if (g.act != Matmul::kBackward) return TEMPO_ERR_UNSUPPORTED;
  return launch(g.kind == TEMPO_GELU_TANH ? matmul_group_kernel<C, D, Matmul::kBackward, TEMPO_GELU_TANH>
                                          : matmul_group_kernel<C, D, Matmul::kBackward, TEMPO_GELU_ERF>);
}

template <bool AKM, bool BKM>
using Large = Config<AKM, BKM, 64, 64, 1, 16, 4>;
template <bool AKM, bool BKM>
using Middle = Config<AKM, BKM, 64, 32, 2, 32, 4>;
template <bool AKM, bool BKM>
using Small = Config<AKM, BKM, 32, 32, 4, 32, 4>;
template <bool AKM, bool BKM>
using SmallLong = Config<AKM, BKM, 32, 32, 8, 64, 4>;

// Tiles of 64 x 64, 64 x 32 or 32 x 32 elements: whichever gives the compute unit with the most of them the least to do,
// where a smaller tile takes 8 % more time for its elements, and a workgroup alone on its compute unit 15 %.  us with 64 x 64 /
// 64 x 32 / 32 x 32 tiles: [256, 768] x [768, 2304] 18.8 / 17.9 / 15.2, [512, 1024] x [1024, 3072] 38.6 / 31.5 / 33.7, [1024, 768]
// x [768, 3072] 43.8 / 46.8 / 49.6.  Where each compute unit has at most one 32 x 32 tile with many values of k, 8 instead of 4
// waves share those: [256, 3072] x [3072, 768] k-major 23.5 / 19.7, 768 values 8.4 / 7.9, but 7.7 / 8.3 with rows of k side by side
// and, 2048 values, 15.4 / 15.5.  Larger tiles per wave or workgroup (64 x 128, 128 x 128) gain 5 % on [2048, 1024] x [1024, 4096]
// and lose everywhere below.
template <bool BKM>
tempo_status by_shape(const Matmul& g, hipStream_t st) {
  const int64_t cus = compute_units();
  auto rounds = [&](int bm, int bn) {
    return (int64_t{(g.M + bm - 1) / bm} * ((g.N + bn - 1) / bn) * g.batch + cus - 1) / cus;
  };
  auto cost = [&](int bm, int bn, int percent) {
    const int64_t r = rounds(bm, bn);
    return r * (bm * bn / 1024) * (100 + percent) + (bm * bn / 1024) * 15;
  };
  const int64_t large = cost(64, 64, 0), middle = cost(64, 32, 8), least = cost(32, 32, 16);
  if (large <= middle && large <= least) return go<Large<false, BKM>>(g, st);
  if (middle <= least) return go<Middle<false, BKM>>(g, st);
  if (rounds(32, 32) == 1 && g.K >= (BKM ? 512 : 2560)) return go<SmallLong<false, BKM>>(g, st);
  return go<Small<false, BKM>>(g, st);
}

}  // namespace

tempo_status launch_matmul(const Matmul& g, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return TEMPO_OK;
  if (g.a.k_major) return TEMPO_ERR_UNSUPPORTED;  // in groups only
  return g.b.k_major ? by_shape<true>(g, st) : by_shape<false>(g, st);
}
// The tile of each by how many of 64 x 64 it has per compute unit: together they are some per compute unit, and the sizes
// that suit a product by itself (by_shape()) are too small or too large.  The rule counts both also where one of them is not
// computed: tiles decide in which order the products of an element add up, and so its bits.  us apart / with the product of the rows in large,
// middle, small tiles and the others' tile this gives: dx and dw of a [256, 768] x [768, 3072] layer (192 and 576 tiles) 37.0 /
// 28.7, 30.3, 32.3; [256, 768] x [768, 768] (48, 144) 16.7 / 20.7, 13.9, 10.9; [128, 768] x [768, 3072] (96, 576) 26.1 / 24.3, 18.0,
// 21.3; [512, 1024] x [1024, 3072] (128, 768) 69.5 / 77.1, 63.6, 66.4; [2048, 1024] x [1024, 4096] (512, 1024) 305 / 301, 327,
// 341.  The others' tile, large / middle / small: (48, 576) 31.3 / 32.4 / 33.9; (48, 144) 13.4 / 10.9 / 11.3; (64, 64) 17.5 / 12.7 /
// 10.0.  Three products of 24 heads of 128 x 128 x 64 11.1 / 6.3.
tempo_status launch_matmul_group(const Matmul& g, const Matmul& h0, const Matmul* h1, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0 || h0.M <= 0 || h0.N <= 0 || h0.batch <= 0) return TEMPO_ERR_UNSUPPORTED;
  using GL = Large<false, true>;
  using GM = Middle<false, true>;
  using GS = Small<false, true>;
  using HL = Large<true, true>;
  using HM = Middle<true, true>;
  using HS = Small<true, true>;
  Matmul counted = h0;
  counted.N = h0.n_counted;
  const int64_t cus = compute_units(), g_tiles = GL::tiles(g), h_tiles = HL::tiles(counted);
  if (g_tiles * 8 >= cus * 5)
    return h_tiles >= cus ? go_group<GL, HL>(g, h0, h1, st) : go_group<GL, HM>(g, h0, h1, st);
  if (g_tiles * 16 >= cus * 5)
    return h_tiles >= cus ? go_group<GM, HL>(g, h0, h1, st) : go_group<GM, HM>(g, h0, h1, st);
  if (h_tiles >= cus) return go_group<GS, HL>(g, h0, h1, st);
  return h_tiles * 8 >= cus * 3 ? go_group<GS, HM>(g, h0, h1, st) : go_group<GS, HS>(g, h0, h1, st);
}

}  // namespace tempo
