// In-place LayerNorm for gfx950 (Sec. 3.2; App. D.2, D.3).
//
// Forward: a group of LANES lanes owns one row, held entirely in registers (CH 16-byte pieces
// per lane, piece c of lane t = c*LANES + t), so x is read once; mean and the biased variance are taken in two
// register passes; gamma/beta stay in registers across the rows a group walks.
// Backward: same ownership; xhat is rebuilt from the OUTPUT as (y - beta)/gamma, the two row
// sums are butterfly-reduced, and the column sums for dgamma/dbeta are carried in registers
// across rows, tree-reduced over the workgroup through LDS in a fixed order and written as
// one partial per workgroup; a second small kernel adds the partials in a fixed order.  Few rows take one
// launch, in which workgroups that own columns walk all rows (ln_bwd_few_kernel).
#include <atomic>
#include <type_traits>

#include "tempo_device.h"
#include "tempo_host.h"

namespace tempo {
namespace {

constexpr int kFwdThreads = 256;
constexpr int kBwdWaves = 8;
constexpr int kBwdThreads = kBwdWaves * kWave;
// ln_bwd_few_kernel: lanes per workgroup, and those of them side by side on a row's columns.
constexpr int kFewThreads = 512;
constexpr int kFewColLanes = 4;
// Rows of more than 1024 pieces in bfloat16 (8192 columns: 4 pieces per lane of 4 waves) or 2048
// pieces in float32 (8192 columns: 6 or 8 pieces per lane of 4 waves, float32 only, whose pieces
// need half the registers per column) take the generic kernels.  Dynamic LDS of the backward: the column sums' slots (all
// of them, 64*M bytes while a row fits one wave, when that is at most kOneStepLdsBytes; else
// half of them for a tree: 32*M bytes while a row fits one wave, 128 KiB at M = 4096; 16*M over
// two waves; 8*M over four), or gamma, 1/gamma and beta/gamma (12*M bytes, 96 KiB at M = 8192)
// when a lane's share of them does not fit its registers, whichever is more.
constexpr int kMaxFastPieces = 1024;
constexpr int kMaxFastPiecesF32 = 2048;
// Most LDS the backward's column sums may take in one step (every wave's sums at once); two
// workgroups of that size still fit a compute unit.
constexpr size_t kOneStepLdsBytes = 64 * 1024;

// The V parameters or column sums of a piece, at a 16-byte aligned address unless RAG.
template <bool RAG, int V>
__device__ __forceinline__ void load_cols(const float* p, float (&v)[V]) {
  if constexpr (RAG) load_floats_any<V>(p, v);
  else load_floats<V>(p, v);
}
// Column sums of piece ch of a row of M columns -> p[0 .. M).  The first `dup` sums of the last
// piece of a ragged row belong to the piece before.  ALIGNED: p is 16-byte aligned.
template <bool RAG, bool ALIGNED, int V>
__device__ __forceinline__ void store_col_sums(float* p, int ch, int chunks, int M, const float (&v)[V]) {
  if (RAG && ch == chunks - 1) {
    const int col = piece_col<RAG, V>(ch, chunks, M), dup = piece_dup<RAG, V>(ch, chunks, M);
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (i >= dup) p[col + i] = v[i];
  } else if constexpr (ALIGNED) {
    store_floats<V>(p + ch * V, v);
  } else {
    store_floats_any<V>(p + ch * V, v);
  }
}
// A division by gamma may be done by multiplication with its reciprocal if neither that nor a residual
// leaves the range of float32: if |gamma| is in 2^-60 .. 2^60, here its offset in that range.
constexpr uint32_t kTameLow = (127u - 60u) << 24, kTameRange = 120u << 24;
__device__ __forceinline__ uint32_t tame_offset(float gamma) { return (as_u32(gamma) << 1) - kTameLow; }
// 1 / g by the hardware estimate and one Newton step (within 1 ulp): a lane does this for each of its columns
// in every workgroup, and the IEEE division costs four times as much.
__device__ __forceinline__ float reciprocal(float g) {
  const float est = __builtin_amdgcn_rcpf(g);
  return fmaf(fmaf(-g, est, 1.0f), est, est);
}
// d / g for a tame g: the product with the reciprocal, one residual step, which rounds it as a division
// does, and the division's own treatment of infinities.
__device__ __forceinline__ float tame_quotient(float d, float g, float rcp) {
  const float q = d * rcp;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-g, q, d), rcp, q), g, d);
}
// Whether all of a wave's gammas are tame: scalar, so that the choice is a branch and not a select.
__device__ __forceinline__ bool all_tame(uint32_t offset) {
  return __builtin_amdgcn_ballot_w64(offset > kTameRange) == 0;
}
// xhat of an element from the stored output.  The fused form loses 2^-24 |beta / gamma| to the rounding of
// beta / gamma; ragged rows subtract first and divide (tame_quotient).  What this / a division per element takes
// beyond the fused form, us: 8192 x 1001 f32 0.3 / 0.2, bf16 0.9 / 2.7; 4096 x 4100 bf16 1.1 / 4.8.
// wave_tame: all_tame(); if not, the choice is per column, so that the two lanes which share one find the same value.
// (Per element: with a loop over the piece inside the branch the few-row kernel is slower, f32 64x4100 4.0 -> 5.9 us.)
template <bool RAG>
__device__ __forceinline__ float xhat_of(float y, float ga, float rg, float bg, bool wave_tame) {
  if constexpr (!RAG) return fmaf(y, rg, -bg);
  if (wave_tame || tame_offset(ga) <= kTameRange) return tame_quotient(y - bg, ga, rg);
  return (y - bg) / ga;
}
// Length of a row of column sums in LDS: whole 16-byte pieces.
__host__ __device__ constexpr int64_t lds_row(int64_t M) { return (M + 3) & ~int64_t{3}; }

// Forward.  A batch is kGroups*R consecutive rows; lane group g takes rows base + r*kGroups + g
// and fetches all R of them (packed) before any arithmetic, so that short rows still keep
// several 16-byte loads per lane in flight.  LOOP = false: one batch per workgroup (the grid
// must cover every batch).  LOOP = true: workgroups walk the batches grid-stride, fetching the
// next batch before they compute on the current one, and load gamma/beta once: for long rows
// the parameters (8 bytes per column from L2) otherwise outweigh the row itself.
// RAG: rows of any length that is no multiple of the piece (see piece_col): 16-byte accesses at
// element-aligned addresses, columns on fixed lanes.  Bound by memory like the aligned rows: 8192 x 1001
// f32 15.1 -> 13.1 us against element-wise accesses (1000 columns: 13.2), 4096 x 4100 bf16 40.6 -> 16.8.
template <typename T, int LANES, int CH, int R, bool LOOP, bool RAG>
__global__ __launch_bounds__(kFwdThreads) void ln_fwd_kernel(
    const T* x, const float* __restrict__ gamma, const float* __restrict__ beta, T* y,
    float* __restrict__ rstd_out, float* __restrict__ mean_out, int64_t N, int M, float eps) {
  constexpr int kGroups = kFwdThreads / LANES;
  constexpr int V = Store<T>::kVec;
  const int g = threadIdx.x / LANES;
  const int t = threadIdx.x % LANES;
  const int chunks = RAG ? (M + V - 1) / V : M / V;
  // mean and variance by a true division: a row of equal values c then has the mean c exactly
  // (its sum c*M is exact) and zero variance, whatever the rounding of 1/M would do
  const float m_f = static_cast<float>(M);
  __shared__ float red[2][kFwdThreads / kWave];
  static_assert(LANES <= kWave || R == 1, "rows over several waves: one row per group");

  auto fetch = [&](int64_t base, Raw<T> (&f)[R][CH]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = base + r * kGroups + g;
      if (row < N) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const int ch = c * LANES + t;
          if (ch < chunks) f[r][c].a = ldg_piece<RAG>(x + row * M + piece_col<RAG, V>(ch, chunks, M));
        }
      }
    }
  };

  int64_t base = static_cast<int64_t>(blockIdx.x) * (kGroups * R);
  if (base >= N) return;  // uniform over the workgroup
  Raw<T> raw[R][CH];
  fetch(base, raw);
  // parameters after the first rows are on their way; they stay in registers for every batch
  float ga[CH][V], be[CH][V];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = c * LANES + t;
    if (ch < chunks) {
      load_cols<RAG, V>(gamma + piece_col<RAG, V>(ch, chunks, M), ga[c]);
      load_cols<RAG, V>(beta + piece_col<RAG, V>(ch, chunks, M), be[c]);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i) ga[c][i] = be[c][i] = 0.0f;
    }
  }
  while (true) {
    const int64_t next = base + static_cast<int64_t>(gridDim.x) * (kGroups * R);
    Raw<T> ahead[R][CH];  // unused (and eliminated) without LOOP
    if constexpr (LOOP) {
      if (next < N) fetch(next, ahead);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = base + r * kGroups + g;
      // no row: uniform over the lane group; a group of several waves walks on with zeros
      // (the reductions hold workgroup barriers) and stores nothing
      const bool live = row < N;
      if (LANES <= kWave && !live) continue;
      float v[CH][V];
      float sum = 0.0f;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
        if (live && ch < chunks) {
          raw[r][c].unpack(v[c]);
        } else {
#pragma unroll
          for (int i = 0; i < V; ++i) v[c][i] = 0.0f;
        }
#pragma unroll
        for (int i = 0; i < V; ++i)
          sum += (RAG && i < piece_dup<RAG, V>(ch, chunks, M)) ? 0.0f : v[c][i];
      }
      const float mu = row_reduce<LANES, false>(sum, red[0]) / m_f;
      float sq = 0.0f;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float d = v[c][i] - mu;
          v[c][i] = d;
          sq += (ch < chunks && i >= piece_dup<RAG, V>(ch, chunks, M)) ? d * d : 0.0f;
        }
      }
      const float var = row_reduce<LANES, false>(sq, red[1]) / m_f;
      const float rs = 1.0f / sqrtf(var + eps);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
        if (live && ch < chunks) {
          float o[V];
#pragma unroll
          for (int i = 0; i < V; ++i) o[i] = fmaf(v[c][i] * rs, ga[c][i], be[c][i]);
          stg_piece<RAG>(y + row * M + piece_col<RAG, V>(ch, chunks, M), Store<T>::pack(o));
        }
      }
      if (t == 0 && live) {
        rstd_out[row] = rs;
        if (mean_out) mean_out[row] = mu;
      }
    }
    if constexpr (!LOOP) {
      break;
    } else {
      if (next >= N) break;  // uniform over the workgroup
#pragma unroll
      for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int c = 0; c < CH; ++c) raw[r][c] = ahead[r][c];
      }
      base = next;
    }
  }
}

// Sum over a 256-thread workgroup; every thread gets the result.
__device__ __forceinline__ float block_sum_256(float v, float* lds) {
  v = group_sum<kWave>(v);
  const int w = threadIdx.x / kWave;
  lds_barrier();
  if ((threadIdx.x & (kWave - 1)) == 0) lds[w] = v;
  lds_barrier();
  return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// Any M (fewer columns than a piece, or more than the register-resident kernels hold): one workgroup per
// row, scalar accesses.  KC > 0: rows of at most 256 * KC columns, held in registers and read once.
// KC == 0: any length, x re-read from cache for each pass.
template <typename T, int KC>
__global__ __launch_bounds__(256) void ln_fwd_generic_kernel(
    const T* x, const float* __restrict__ gamma, const float* __restrict__ beta, T* y,
    float* __restrict__ rstd_out, float* __restrict__ mean_out, int64_t N, int64_t M, float eps) {
  __shared__ float lds[4];
  const float m_f = static_cast<float>(M);
  for (int64_t row = blockIdx.x; row < N; row += gridDim.x) {
    const T* xr = x + row * M;
    T* yr = y + row * M;
    float mu, rs;
    if constexpr (KC > 0) {
      // rows of at most 256 * KC columns: read once, thread t holds columns t, t + 256, ...
      float v[KC];
      float s = 0.0f;
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        const int64_t j = k * 256 + threadIdx.x;
        v[k] = j < M ? Store<T>::load1(xr + j) : 0.0f;
        s += v[k];
      }
      mu = block_sum_256(s, lds) / m_f;
      float q = 0.0f;
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        const int64_t j = k * 256 + threadIdx.x;
        const float d = v[k] - mu;
        v[k] = d;
        q += j < M ? d * d : 0.0f;
      }
      const float var = block_sum_256(q, lds) / m_f;
      rs = 1.0f / sqrtf(var + eps);
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        const int64_t j = k * 256 + threadIdx.x;
        if (j < M) Store<T>::store1(yr + j, fmaf(v[k] * rs, gamma[j], beta[j]));
      }
    } else {
      float s = 0.0f;
      for (int64_t j = threadIdx.x; j < M; j += 256) s += Store<T>::load1(xr + j);
      mu = block_sum_256(s, lds) / m_f;
      float q = 0.0f;
      for (int64_t j = threadIdx.x; j < M; j += 256) {
        const float d = Store<T>::load1(xr + j) - mu;
        q += d * d;
      }
      const float var = block_sum_256(q, lds) / m_f;
      rs = 1.0f / sqrtf(var + eps);
      for (int64_t j = threadIdx.x; j < M; j += 256) {
        const float d = Store<T>::load1(xr + j) - mu;
        Store<T>::store1(yr + j, fmaf(d * rs, gamma[j], beta[j]));
      }
    }
    if (threadIdx.x == 0) {
      rstd_out[row] = rs;
      if (mean_out) mean_out[row] = mu;
    }
  }
}

// A "batch" is kGroups*R consecutive rows: lane group g takes rows base + r*kGroups + g, r < R.
// All R rows of a group are fetched (kept packed) before any arithmetic, so a group waits
// for memory once per batch.  LOOP = false: one batch per workgroup (grid = batches).
// LOOP = true: workgroups walk the batches grid-stride and fetch the next batch before they
// compute on the current one; the column sums stay in registers across batches, so the LDS
// tree and the partial store are paid once per workgroup however many rows it walks.
// RAG: rows of any length that is no multiple of the piece (see piece_col), parameters in registers,
// and xhat as the quotient (y - beta) / gamma itself.  8192 x 1001 f32 50.0 -> 23.7 us against
// element-wise accesses (1000 columns: 22.4), 4096 x 4100 bf16 97.8 -> 28.5.
template <typename T, int LANES, int CH, int R, bool LOOP, bool RAG>
__global__ __launch_bounds__(kBwdThreads) void ln_bwd_kernel(
    const T* dy, const T* __restrict__ y, const float* __restrict__ gamma,
    const float* __restrict__ beta, const float* __restrict__ rstd, T* dx,
    float* __restrict__ partial, int64_t N, int M, int slot_row) {
  extern __shared__ float lds[];  // bwd_lds_bytes(): the tree's [slots][2][M] floats, >= 3*M
  constexpr int kGroups = kBwdThreads / LANES;
  constexpr int V = Store<T>::kVec;
  const int g = threadIdx.x / LANES;
  const int t = threadIdx.x % LANES;
  const int wave = threadIdx.x / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int chunks = RAG ? (M + V - 1) / V : M / V;
  const int Ml = RAG ? static_cast<int>(lds_row(M)) : M;  // a row of column sums in LDS
  const float inv_m = 1.0f / static_cast<float>(M);
  const int64_t batch_rows = kGroups * R;
  __shared__ float2 red[2][kBwdWaves];
  static_assert(LANES <= kWave || R == 1, "rows over several waves: one row per group");
  int flip = 0;
  // gamma, 1/gamma and beta/gamma (beta if RAG) of the lane's columns live in its registers when that share
  // is at most 24 columns; otherwise in LDS (the first 3*M floats; the
  // same memory is reused by the reduction tree at the end), where every row re-reads the three
  // vectors twice: at 8 waves per compute unit that is microseconds of LDS time per batch.
  // The column sums are always in registers.
  constexpr bool kRegParams = CH * V <= 24;
  static_assert(!RAG || kRegParams, "ragged rows: parameters in registers");
  float* p_ga = lds;
  float* p_rg = lds + M;
  float* p_bg = lds + 2 * M;
  float r_ga[kRegParams ? CH : 1][V], r_rg[kRegParams ? CH : 1][V], r_bg[kRegParams ? CH : 1][V];
  // xhat and dy*gamma of the batch stay in registers between the two passes when they fit (128
  // registers; a workgroup of 8 waves has 256 per lane however few it uses): the second pass
  // then neither unpacks nor recomputes them.  Same arithmetic either way.
  constexpr bool kKeep = kRegParams && R * CH * V <= 64 && R * CH * 8 * (LOOP ? 2 : 1) <= 64;
  float k_h[kKeep ? R : 1][kKeep ? CH : 1][V], k_q[kKeep ? R : 1][kKeep ? CH : 1][V];
  float acc_g[CH][V], acc_b[CH][V];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
#pragma unroll
    for (int i = 0; i < V; ++i) acc_g[c][i] = acc_b[c][i] = 0.0f;
  }

  auto fetch = [&](int64_t base, Raw<T> (&fd)[R][CH], Raw<T> (&fy)[R][CH], float (&fs)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = base + r * kGroups + g;
      fs[r] = 0.0f;
      if (row < N) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const int ch = c * LANES + t;
          if (ch < chunks) {
            const int64_t e = row * M + piece_col<RAG, V>(ch, chunks, M);
            fd[r][c].a = ldg_piece<RAG>(dy + e);
            fy[r][c].a = ldg_piece<RAG>(y + e);
          }
        }
        fs[r] = rstd[row];
      }
    }
  };

  int64_t base = static_cast<int64_t>(blockIdx.x) * batch_rows;
  Raw<T> rd[R][CH], ry[R][CH];
  float rs[R];
  fetch(base, rd, ry, rs);
  // parameters after the first rows are on their way
  uint32_t offset = 0;  // the largest of the lane's gammas
  if constexpr (kRegParams) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int ch = c * LANES + t;
      float be[V];
      if (ch < chunks) {
        load_cols<RAG, V>(gamma + piece_col<RAG, V>(ch, chunks, M), r_ga[c]);
        load_cols<RAG, V>(beta + piece_col<RAG, V>(ch, chunks, M), be);
      } else {
#pragma unroll
        for (int i = 0; i < V; ++i) {
          r_ga[c][i] = 1.0f;
          be[i] = 0.0f;
        }
      }
#pragma unroll
      for (int i = 0; i < V; ++i) {
        r_rg[c][i] = reciprocal(r_ga[c][i]);
        if constexpr (RAG) {
          r_bg[c][i] = be[i];
          // waits for beta here: first used inside the loop, it would make the loop wait for every
          // load under way, the rows fetched ahead included (8192 x 1001 f32: 38 -> 42 us)
          asm volatile("" : "+v"(r_bg[c][i]));
          offset = max(offset, tame_offset(r_ga[c][i]));
        } else {
          r_bg[c][i] = be[i] * r_rg[c][i];
        }
      }
    }
  } else {
    for (int j = threadIdx.x; j < M; j += kBwdThreads) {
      const float gj = gamma[j];
      const float rj = 1.0f / gj;
      p_ga[j] = gj;
      p_rg[j] = rj;
      p_bg[j] = beta[j] * rj;
    }
    lds_barrier();
  }
  const bool wave_tame = all_tame(offset);
  auto xhat = [&](const float (&y8)[V], const float (&ga)[V], const float (&rg)[V], const float (&bg)[V],
                  float (&h)[V]) {
    if (!RAG || wave_tame) {
#pragma unroll
      for (int i = 0; i < V; ++i) h[i] = xhat_of<RAG>(y8[i], ga[i], rg[i], bg[i], true);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i) h[i] = xhat_of<RAG>(y8[i], ga[i], rg[i], bg[i], false);
    }
  };
  while (base < N) {
    const int64_t next = base + static_cast<int64_t>(gridDim.x) * batch_rows;
    Raw<T> nd[R][CH], ny[R][CH];  // unused (and eliminated) without LOOP
    float ns[R];
    if constexpr (LOOP) {
      if (next < N) fetch(next, nd, ny, ns);
    }
    // pass 1: the two row sums of every row (and the column accumulators); the R butterfly
    // chains are independent, so their latencies overlap
    float c1[R], c2[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = base + r * kGroups + g;
      c1[r] = c2[r] = 0.0f;
      if (row >= N) continue;  // uniform over the lane group
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
        if (ch < chunks) {
          float d8[V], y8[V], ga[V], rg[V], bg[V];
          rd[r][c].unpack(d8);
          ry[r][c].unpack(y8);
          if constexpr (kRegParams) {
#pragma unroll
            for (int i = 0; i < V; ++i) {
              ga[i] = r_ga[c][i];
              rg[i] = r_rg[c][i];
              bg[i] = r_bg[c][i];
            }
          } else {
            load_floats<V>(p_ga + ch * V, ga);
            load_floats<V>(p_rg + ch * V, rg);
            load_floats<V>(p_bg + ch * V, bg);
          }
          float h[V];
          xhat(y8, ga, rg, bg, h);
#pragma unroll
          for (int i = 0; i < V; ++i) {
            const float q = d8[i] * ga[i];
            if (!RAG || i >= piece_dup<RAG, V>(ch, chunks, M)) {
              c1[r] = fmaf(q, h[i], c1[r]);
              c2[r] += q;
            }
            acc_g[c][i] = fmaf(d8[i], h[i], acc_g[c][i]);
            acc_b[c][i] += d8[i];
            if constexpr (kKeep) {
              k_h[r][c][i] = h[i];
              k_q[r][c][i] = q;
            }
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      row_sum2<LANES>(c1[r], c2[r], red[flip]);
      flip ^= 1;
      c1[r] *= inv_m;
      c2[r] *= inv_m;
    }
    // pass 2: dx, from the kept xhat and dy*gamma or recomputing them from the packed registers
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = base + r * kGroups + g;
      if (row >= N) continue;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
        if (ch < chunks) {
          float o[V];
          if constexpr (kKeep) {
#pragma unroll
            for (int i = 0; i < V; ++i)
              o[i] = rs[r] * (k_q[r][c][i] - fmaf(k_h[r][c][i], c1[r], c2[r]));
          } else {
            float d8[V], y8[V], ga[V], rg[V], bg[V];
            rd[r][c].unpack(d8);
            ry[r][c].unpack(y8);
            if constexpr (kRegParams) {
#pragma unroll
              for (int i = 0; i < V; ++i) {
                ga[i] = r_ga[c][i];
                rg[i] = r_rg[c][i];
                bg[i] = r_bg[c][i];
              }
            } else {
              load_floats<V>(p_ga + ch * V, ga);
              load_floats<V>(p_rg + ch * V, rg);
              load_floats<V>(p_bg + ch * V, bg);
            }
            float h[V];
            xhat(y8, ga, rg, bg, h);
#pragma unroll
            for (int i = 0; i < V; ++i) o[i] = rs[r] * (d8[i] * ga[i] - fmaf(h[i], c1[r], c2[r]));
          }
          stg_piece<RAG>(dx + row * M + piece_col<RAG, V>(ch, chunks, M), Store<T>::pack(o));
        }
      }
    }
    if constexpr (!LOOP) {
      break;
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          rd[r][c] = nd[r][c];
          ry[r][c] = ny[r][c];
        }
        rs[r] = ns[r];
      }
      base = next;
    }
  }
  // Column sums of the workgroup -> its [2][M] slot of `partial`.  First over the lane groups
  // that share a wave (fixed butterfly), then over the waves through LDS.  When a row takes
  // W > 1 waves, wave w holds the columns of part w % W of the row; the W waves of one row, whose
  // columns are disjoint, share one [2][M] LDS slot, so there are S = kBwdWaves / W slots to add.
  // The association is the same on both routes, a binary tree that pairs slot s with s + S/2,
  // then s + S/4, ...:
  //  - all S slots fit kOneStepLdsBytes: every wave writes its sums, one barrier, and each lane
  //    of the workgroup adds one 16-byte piece of the S slots and stores it;
  //  - else the tree runs through S/2 slots, a barrier pair per level, and the waves of slot 0
  //    store the result.
  // This tail is on the critical path of the kernel (the tree and the slot's store were each
  // measured at about a microsecond of it); running it before the last batch's dx is stored
  // hides the store but puts a barrier between the waves' loads and stores, and was slower.
#pragma unroll
  for (int c = 0; c < CH; ++c) {
#pragma unroll
    for (int i = 0; i < V; ++i) {
#pragma unroll
      for (int m = LANES; m < kWave; m <<= 1) {
        acc_g[c][i] += __shfl_xor(acc_g[c][i], m, kWave);
        acc_b[c][i] += __shfl_xor(acc_b[c][i], m, kWave);
      }
    }
  }
  const bool owner = lane < LANES;  // one copy per wave
  constexpr int kRowWaves = LANES > kWave ? LANES / kWave : 1;
  constexpr int S = kBwdWaves / kRowWaves;
  float* out = partial + static_cast<size_t>(blockIdx.x) * 2 * slot_row;
  if (static_cast<size_t>(S) * 2 * Ml * sizeof(float) <= kOneStepLdsBytes) {
    if constexpr (!kRegParams) lds_barrier();  // the parameters in LDS are no longer read
    if (owner) {
      float* slot = lds + static_cast<size_t>(wave / kRowWaves) * 2 * Ml;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
        if (ch < chunks) {
          store_col_sums<RAG, true, V>(slot, ch, chunks, M, acc_g[c]);
          store_col_sums<RAG, true, V>(slot + Ml, ch, chunks, M, acc_b[c]);
        }
      }
    }
    lds_barrier();
    for (int j = threadIdx.x * 4; j < 2 * Ml; j += kBwdThreads * 4) {
      float v[S][4];
#pragma unroll
      for (int k = 0; k < S; ++k) load_floats<4>(lds + static_cast<size_t>(k) * 2 * Ml + j, v[k]);
#pragma unroll
      for (int half = S / 2; half >= 1; half >>= 1) {
#pragma unroll
        for (int k = 0; k < half; ++k) {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[k][i] += v[k + half][i];
        }
      }
      if (RAG && slot_row != Ml) {  // from LDS rows of Ml to slot rows of M floats
        const int col = j < Ml ? j : j - Ml;
        float* o = out + (j < Ml ? 0 : slot_row) + col;
        if (col + 4 <= M) {
          store_floats_any<4>(o, v[0]);
        } else {
          for (int i = 0; col + i < M; ++i) o[i] = v[0][i];
        }
      } else {
        store_floats<4>(out + j, v[0]);
      }
    }
    return;
  }
#pragma unroll
  for (int half = kBwdWaves / 2; half >= kRowWaves; half >>= 1) {
    lds_barrier();
    if (wave >= half && wave < 2 * half && owner) {
      float* slot = lds + static_cast<size_t>((wave - half) / kRowWaves) * 2 * Ml;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
        if (ch < chunks) {
          store_col_sums<RAG, true, V>(slot, ch, chunks, M, acc_g[c]);
          store_col_sums<RAG, true, V>(slot + Ml, ch, chunks, M, acc_b[c]);
        }
      }
    }
    lds_barrier();
    if (wave < half && owner) {
      const float* slot = lds + static_cast<size_t>(wave / kRowWaves) * 2 * Ml;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = c * LANES + t;
        if (ch < chunks) {
          float a[V], b[V];
          load_cols<RAG, V>(slot + piece_col<RAG, V>(ch, chunks, M), a);
          load_cols<RAG, V>(slot + Ml + piece_col<RAG, V>(ch, chunks, M), b);
#pragma unroll
          for (int i = 0; i < V; ++i) {
            acc_g[c][i] += a[i];
            acc_b[c][i] += b[i];
          }
        }
      }
    }
  }
  if (wave < kRowWaves && owner) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int ch = c * LANES + t;
      if (ch < chunks) {
        store_col_sums<RAG, !RAG, V>(out, ch, chunks, M, acc_g[c]);
        store_col_sums<RAG, !RAG, V>(out + slot_row, ch, chunks, M, acc_b[c]);
      }
    }
  }
}

// Any M: one workgroup per row for dx; per-workgroup column partials are accumulated by
// walking rows blockIdx.x, blockIdx.x + gridDim.x, ... with thread j owning columns j, j+256...
// KC > 0: rows of at most 256 * KC columns; the thread's column sums and the gamma and beta of
// its columns live in registers and the partial slot is written once at the end.  KC == 0: any
// length; the sums are kept in the partial slot itself (private to the workgroup).
template <typename T, int KC>
__global__ __launch_bounds__(256) void ln_bwd_generic_kernel(
    const T* dy, const T* __restrict__ y, const float* __restrict__ gamma,
    const float* __restrict__ beta, const float* __restrict__ rstd, T* dx,
    float* __restrict__ partial, int64_t N, int64_t M) {
  __shared__ float lds[4];
  const float inv_m = 1.0f / static_cast<float>(M);
  float* pg = partial + static_cast<size_t>(blockIdx.x) * 2 * M;
  float* pb = pg + M;
  if constexpr (KC > 0) {
    float ag[KC], ab[KC], ga[KC], be[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const int64_t j = k * 256 + threadIdx.x;
      ag[k] = ab[k] = 0.0f;
      ga[k] = j < M ? gamma[j] : 1.0f;
      be[k] = j < M ? beta[j] : 0.0f;
    }
    for (int64_t row = blockIdx.x; row < N; row += gridDim.x) {
      const T* dyr = dy + row * M;
      const T* yr = y + row * M;
      T* dxr = dx + row * M;
      float c1 = 0.0f, c2 = 0.0f;
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        const int64_t j = k * 256 + threadIdx.x;
        if (j < M) {
          const float d = Store<T>::load1(dyr + j);
          const float h = (Store<T>::load1(yr + j) - be[k]) / ga[k];
          const float q = d * ga[k];
          c1 = fmaf(q, h, c1);
          c2 += q;
          ag[k] = fmaf(d, h, ag[k]);
          ab[k] += d;
        }
      }
      c1 = block_sum_256(c1, lds) * inv_m;
      c2 = block_sum_256(c2, lds) * inv_m;
      const float rs = rstd[row];
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        const int64_t j = k * 256 + threadIdx.x;
        if (j < M) {
          const float d = Store<T>::load1(dyr + j);
          const float h = (Store<T>::load1(yr + j) - be[k]) / ga[k];
          Store<T>::store1(dxr + j, rs * (d * ga[k] - fmaf(h, c1, c2)));
        }
      }
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const int64_t j = k * 256 + threadIdx.x;
      if (j < M) {
        pg[j] = ag[k];
        pb[j] = ab[k];
      }
    }
  } else {
    for (int64_t j = threadIdx.x; j < M; j += 256) {
      pg[j] = 0.0f;
      pb[j] = 0.0f;
    }
    for (int64_t row = blockIdx.x; row < N; row += gridDim.x) {
      const T* dyr = dy + row * M;
      const T* yr = y + row * M;
      T* dxr = dx + row * M;
      float c1 = 0.0f, c2 = 0.0f;
      for (int64_t j = threadIdx.x; j < M; j += 256) {
        const float d = Store<T>::load1(dyr + j);
        const float h = (Store<T>::load1(yr + j) - beta[j]) / gamma[j];
        const float q = d * gamma[j];
        c1 = fmaf(q, h, c1);
        c2 += q;
        pg[j] = fmaf(d, h, pg[j]);
        pb[j] += d;
      }
      c1 = block_sum_256(c1, lds) * inv_m;
      c2 = block_sum_256(c2, lds) * inv_m;
      const float rs = rstd[row];
      for (int64_t j = threadIdx.x; j < M; j += 256) {
        const float d = Store<T>::load1(dyr + j);
        const float h = (Store<T>::load1(yr + j) - beta[j]) / gamma[j];
        Store<T>::store1(dxr + j, rs * (d * gamma[j] - fmaf(h, c1, c2)));
      }
    }
  }
}

// dgamma[j] = sum_p partial[p][0][j], dbeta[j] = sum_p partial[p][1][j], slots of [2][slot_row >= M].  A workgroup of
// 4 waves owns 32 adjacent columns of the [2][slot_row] row, 8 lanes x 4 floats; its 32 slices each add every
// 32nd partial (all loads of a lane are independent and issued together), then the slices are
// combined through LDS in a fixed order.  ANY (slot_row odd): slots start at any float's address and the
// last 16-byte piece of a slot is half a piece.
constexpr int kFinCols = 32;   // 128 contiguous bytes per partial row
constexpr int kFinSlices = 32;
constexpr int kFinVecLanes = kFinCols / 4;
template <bool ANY>
__global__ __launch_bounds__(kFinVecLanes* kFinSlices) void ln_bwd_finalize_kernel(
    const float* __restrict__ partial, float* __restrict__ dgamma, float* __restrict__ dbeta,
    int parts, int64_t M, int64_t slot_row) {
  __shared__ float lds[kFinSlices][kFinCols + 4];
  const int q = threadIdx.x % kFinVecLanes;
  const int slice = threadIdx.x / kFinVecLanes;
  const int64_t j2 = static_cast<int64_t>(blockIdx.x) * kFinCols + q * 4;  // index into [2][slot_row]
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  auto add_up = [&](auto load) {  // load(address, four values)
    const float* p0 = partial + j2;
    auto at = [&](int p) { return p0 + static_cast<size_t>(p) * 2 * slot_row; };
    int p = slice;
    for (; p + 7 * kFinSlices < parts; p += 8 * kFinSlices) {
      float v[8][4];
#pragma unroll
      for (int u = 0; u < 8; ++u) load(at(p + u * kFinSlices), v[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] += v[u][i];
      }
    }
    // The rest all at once too: with 250 partials the last slices have 7, and cost 1.5 us when they added
    // them up one memory latency after the other (2000 x 1024 bf16 backward 10.2 -> 8.7 us).
    if (p + kFinSlices < parts) {
      float v[7][4];
#pragma unroll
      for (int u = 0; u < 7; ++u)
        if (p + u * kFinSlices < parts) load(at(p + u * kFinSlices), v[u]);
#pragma unroll
      for (int u = 0; u < 7; ++u) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (p + u * kFinSlices < parts) s[i] += v[u][i];
      }
    } else if (p < parts) {
      float v[4];
      load(at(p), v);
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] += v[i];
    }
  };
  if (j2 + 4 <= 2 * slot_row) {
    add_up([](const float* p, float (&v)[4]) { load_cols<ANY, 4>(p, v); });
  } else if (ANY && j2 < 2 * slot_row) {  // 2 * slot_row - j2 is 2: the sums of two columns, as many loads under way
    add_up([](const float* p, float (&v)[4]) {
      v[0] = p[0];
      v[1] = p[1];
      v[2] = v[3] = 0.0f;
    });
  }
  store_floats<4>(&lds[slice][q * 4], s);
  lds_barrier();
  const int col = threadIdx.x;
  const int64_t j = static_cast<int64_t>(blockIdx.x) * kFinCols + col;
  if (col < kFinCols && (j < M || (j >= slot_row && j < slot_row + M))) {
    float tot = 0.0f;
#pragma unroll
    for (int k = 0; k < kFinSlices; ++k) tot += lds[k][col];
    if (j < M) dgamma[j] = tot;
    else dbeta[j - slot_row] = tot;
  }
}

// The columns of a piece and xhat of its rows.
template <bool RAG, int V>
struct Xhat {
  float ga[V], rg[V], bg[V];
  bool tame;
  __device__ __forceinline__ Xhat(const float (&gamma)[V], const float (&beta)[V]) {
    uint32_t offset = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      ga[i] = gamma[i];
      rg[i] = reciprocal(gamma[i]);
      bg[i] = RAG ? beta[i] : beta[i] * rg[i];
      offset = max(offset, tame_offset(gamma[i]));
    }
    tame = all_tame(offset);
  }
  __device__ __forceinline__ void operator()(const float (&y8)[V], float (&h)[V]) const {
#pragma unroll
    for (int i = 0; i < V; ++i) h[i] = xhat_of<RAG>(y8[i], ga[i], rg[i], bg[i], tame);
  }
};

// Few rows: the whole backward in one launch.  The first col_blocks workgroups own 64 bytes of columns each
// (4 lanes x a piece, 128 rows at a time) and walk all rows for dgamma and dbeta, which need no row sums; the
// others own rows (LANES lanes, CH pieces per lane) and write dx.  dy and y are read twice, the second
// time from a cache; in return there are no partials and no second dispatch.  In place (dx is dy) the two halves
// are launched one after the other; `first` is the launch's first workgroup.
// Bound by latency: a launch that does nothing takes 1.7 us, and a wave alone on its SIMD 4-8 cycles an
// instruction, so that the column walk has one row per lane under way and the next fetched: with 2, 4 or 8 rows
// unrolled 64x768 f32 takes 3.0, 3.5 and 5.3 us (256 lanes) instead of 2.9.
template <typename T, int LANES, int CH, bool RAG>
__global__ __launch_bounds__(kFewThreads) void ln_bwd_few_kernel(
    const T* dy, const T* y, const float* __restrict__ gamma,
    const float* __restrict__ beta, const float* __restrict__ rstd, T* dx,
    float* __restrict__ dgamma, float* __restrict__ dbeta, int N, int M, int col_blocks, int first) {
  constexpr int V = Store<T>::kVec;
  constexpr int kWaves = kFewThreads / kWave;
  const int chunks = RAG ? (M + V - 1) / V : M / V;
  auto load = [](const T* p) {  // cached: the other half of the grid reads it too
    if constexpr (RAG) return *reinterpret_cast<const u32x4_any*>(p);
    else return *reinterpret_cast<const u32x4*>(p);
  };
  const int block = first + static_cast<int>(blockIdx.x);
  if (block < col_blocks) {
    constexpr int kSlices = kFewThreads / kFewColLanes;
    static_assert(kFewColLanes == 4, "the sums over a wave's lanes below");
    __shared__ float sums[kWaves][kFewColLanes][2 * V];
    const int t = threadIdx.x % kFewColLanes;
    const int slice = threadIdx.x / kFewColLanes;
    const int ch = block * kFewColLanes + t;
    float acc[2 * V];
#pragma unroll
    for (int i = 0; i < 2 * V; ++i) acc[i] = 0.0f;
    if (ch < chunks && slice < N) {
      const int col = piece_col<RAG, V>(ch, chunks, M);
      int64_t e = static_cast<int64_t>(slice) * M + col;
      u32x4 d = load(dy + e), o = load(y + e);
      float ga[V], be[V];
      load_cols<RAG, V>(gamma + col, ga);
      load_cols<RAG, V>(beta + col, be);
      const Xhat<RAG, V> xhat(ga, be);
      for (int row = slice; row < N; row += kSlices) {
        u32x4 next_d = d, next_o = o;
        e += static_cast<int64_t>(kSlices) * M;
        if (row + kSlices < N) {
          next_d = load(dy + e);
          next_o = load(y + e);
        }
        float d8[V], y8[V], h[V];
        Store<T>::unpack(d, d8);
        Store<T>::unpack(o, y8);
        xhat(y8, h);
#pragma unroll
        for (int i = 0; i < V; ++i) {
          acc[i] = fmaf(d8[i], h[i], acc[i]);
          acc[V + i] += d8[i];
        }
        d = next_d;
        o = next_o;
      }
    }
    // over the 16 lanes of the wave that own the same piece, then over the waves
    auto add = [](float a, float b) { return a + b; };
#pragma unroll
    for (int i = 0; i < 2 * V; ++i) {
      acc[i] += dpp_f32<kDppRor4>(acc[i]);
      acc[i] += dpp_f32<kDppRor8>(acc[i]);
      acc[i] = across_rows<32>(across_rows<16>(acc[i], add), add);
    }
    if ((threadIdx.x & (kWave - 1)) < kFewColLanes) {
#pragma unroll
      for (int i = 0; i < 2 * V; ++i) sums[threadIdx.x / kWave][t][i] = acc[i];
    }
    lds_barrier();
    const int k = threadIdx.x / (2 * V), i = threadIdx.x % (2 * V);
    const int sum_ch = block * kFewColLanes + k;
    if (k < kFewColLanes && sum_ch < chunks && i % V >= piece_dup<RAG, V>(sum_ch, chunks, M)) {
      float s = sums[0][k][i];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) s += sums[w][k][i];
      (i < V ? dgamma : dbeta)[piece_col<RAG, V>(sum_ch, chunks, M) + i % V] = s;
    }
    return;
  }
  constexpr int kGroups = kFewThreads / LANES;
  __shared__ float2 red[kWaves];
  const int t = threadIdx.x % LANES;
  const int row = (block - col_blocks) * kGroups + threadIdx.x / LANES;
  const bool live = row < N;  // a group of several waves walks on: the row sums hold a barrier
  if (LANES <= kWave && !live) return;
  const int64_t e = static_cast<int64_t>(row) * M;
  u32x4 d[CH], o[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = c * LANES + t;
    if (live && ch < chunks) {
      d[c] = load(dy + e + piece_col<RAG, V>(ch, chunks, M));
      o[c] = load(y + e + piece_col<RAG, V>(ch, chunks, M));
    }
  }
  const float rs = live ? rstd[row] : 0.0f;
  float h[CH][V], q[CH][V];
  float c1 = 0.0f, c2 = 0.0f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = c * LANES + t;
    if (live && ch < chunks) {
      float ga[V], be[V], d8[V], y8[V];
      load_cols<RAG, V>(gamma + piece_col<RAG, V>(ch, chunks, M), ga);
      load_cols<RAG, V>(beta + piece_col<RAG, V>(ch, chunks, M), be);
      Store<T>::unpack(d[c], d8);
      Store<T>::unpack(o[c], y8);
      Xhat<RAG, V>(ga, be)(y8, h[c]);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        q[c][i] = d8[i] * ga[i];
        if (!RAG || i >= piece_dup<RAG, V>(ch, chunks, M)) {
          c1 = fmaf(q[c][i], h[c][i], c1);
          c2 += q[c][i];
        }
      }
    }
  }
  row_sum2<LANES>(c1, c2, red);
  const float inv_m = 1.0f / static_cast<float>(M);
  c1 *= inv_m;
  c2 *= inv_m;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = c * LANES + t;
    if (live && ch < chunks) {
      float r[V];
#pragma unroll
      for (int i = 0; i < V; ++i) r[i] = rs * (q[c][i] - fmaf(h[c][i], c1, c2));
      stg_piece<RAG>(dx + e + piece_col<RAG, V>(ch, chunks, M), Store<T>::pack(r));
    }
  }
}

struct Shape {
  int lanes;
  int ch;
};

// Lanes per row and pieces per lane for a row of `pieces` 16-byte pieces: least padding, then
// the widest group.  ch == 0: no register-resident shape fits.  full_wave (the backward): a
// whole wave per row counts as unpadded while at most a third of its lanes' pieces are
// padding; one row per wave lets a lane group fetch up to 4 rows at once, which there is
// worth more than the idle lanes (measured at 384 and 768 columns; the forward loses by it).
constexpr Shape pick_shape(int pieces, bool full_wave) {
  constexpr int wide[] = {1, 2, 3, 4, 6, 8, 12, 16};  // 64 lanes
  constexpr int narrow[] = {1, 2, 3};                 // 32 and 16 lanes
  Shape best = {0, 0};
  int best_waste = 1 << 30;
  for (int lanes = 64; lanes >= 16; lanes >>= 1) {
    const int need = (pieces + lanes - 1) / lanes;
    const int* allowed = lanes == 64 ? wide : narrow;
    const int count = lanes == 64 ? 8 : 3;
    for (int k = 0; k < count; ++k) {
      if (allowed[k] >= need) {
        int waste = lanes * allowed[k] - pieces;
        if (full_wave && lanes == 64 && waste * 3 <= lanes * allowed[k]) waste = 0;
        if (waste < best_waste) {
          best_waste = waste;
          best = {lanes, allowed[k]};
        }
        break;
      }
    }
  }
  return best;
}

// A row whose pieces per lane on one wave would exceed max_ch is spread over 2 or 4 waves (at
// most 4 pieces per lane there).
constexpr Shape widen_shape(Shape one, int pieces, int max_ch, int max_lanes) {
  if (one.ch == 0 || (one.lanes == kWave && one.ch > max_ch)) {  // no one-wave shape, or too many pieces
    for (int lanes = 2 * kWave; lanes <= max_lanes; lanes *= 2) {
      const int need = (pieces + lanes - 1) / lanes;
      if (need <= max_ch || lanes == max_lanes) {
        if (need <= 4) return {lanes, need};
        if (lanes == max_lanes && need <= 8) return {lanes, need <= 6 ? 6 : 8};
        break;
      }
    }
  }
  return one;
}

}  // namespace

#define TEMPO_LN_DISPATCH(LAUNCH)                                                          \
  switch (sh.lanes * 100 + sh.ch) {                                                        \
    case 6401: LAUNCH(64, 1); break;                                                       \
    case 6402: LAUNCH(64, 2); break;                                                       \
    case 6403: LAUNCH(64, 3); break;                                                       \
    case 6404: LAUNCH(64, 4); break;                                                       \
    case 6406: LAUNCH(64, 6); break;                                                       \
    case 6408: LAUNCH(64, 8); break;                                                       \
    case 6412: LAUNCH(64, 12); break;                                                      \
    case 6416: LAUNCH(64, 16); break;                                                      \
    case 3201: LAUNCH(32, 1); break;                                                       \
    case 3203: LAUNCH(32, 3); break;                                                       \
    case 1601: LAUNCH(16, 1); break;                                                       \
    case 1603: LAUNCH(16, 3); break;                                                       \
    case 12801: LAUNCH(128, 1); break;                                                     \
    case 12802: LAUNCH(128, 2); break;                                                     \
    case 12803: LAUNCH(128, 3); break;                                                     \
    case 12804: LAUNCH(128, 4); break;                                                     \
    case 25601: LAUNCH(256, 1); break;                                                     \
    case 25602: LAUNCH(256, 2); break;                                                     \
    case 25603: LAUNCH(256, 3); break;                                                     \
    case 25604: LAUNCH(256, 4); break;                                                     \
    case 25606: LAUNCH(256, 6); break;                                                     \
    case 25608: LAUNCH(256, 8); break;                                                     \
    case 51202: LAUNCH(512, 2); break;                                                     \
    case 51204: LAUNCH(512, 4); break;                                                     \
    default: return TEMPO_ERR_UNSUPPORTED;                                                 \
  }

// Rows per lane group that exist as kernels for a shape (keeps the number of instantiations
// down): 4 only for one or two pieces per lane on full-wave groups, 2 up to four pieces.
template <int L, int C>
constexpr int max_rows() {
  return L > 64 ? 1 : ((C <= 2 && L == 64) ? 4 : (C <= 4 ? 2 : 1));
}

// Most pieces a row may have in the register-resident kernels.
constexpr int max_fast_pieces(int vec) { return vec == 4 ? kMaxFastPiecesF32 : kMaxFastPieces; }
// Shape for rows of `pieces` pieces of vec elements; ch == 0: too long.
// Backward: four waves whose lanes would own more than 24 columns each (parameters in LDS, read twice per
// element) give the row to all eight waves, which halves the columns per lane and keeps the parameters
// in registers.  Ragged rows, whose columns also hold a quotient:
//  - so do those of 24 columns in float32, which do not fit the registers: 8000x5001 138 -> 89 us, 2000x4097
//    38 -> 27; in bfloat16 they do, and eight waves lose (8000x5001 56 -> 66);
//  - several rows per wave with three pieces per lane end in long reductions: a row per wave instead.  f32
//    64x129 6.8 -> 4.9, 4000x129 9.0 -> 7.0, 65536x129 28 -> 25; bf16 64x515 8.8 -> 6.8,
//    4000x515 13.4 -> 9.9, 16384x515 19.0 -> 19.2, and not beyond: 65536x515 49 -> 54.  many: 64 rows per compute unit
//    and more.
constexpr Shape shape_of(int pieces, int vec, int max_ch, bool backward, bool ragged, bool many) {
  const Shape sh = widen_shape(pick_shape(pieces, backward), pieces, max_ch, 256);
  if (backward && sh.lanes == 256 && sh.ch * vec > 24) return {kBwdThreads, sh.ch / 2};
  if (backward && ragged) {
    if (sh.lanes == 256 && sh.ch == 6) return {kBwdThreads, 4};
    if (sh.lanes < kWave && sh.ch == 3 && (vec == 4 || !many)) return {kWave, (pieces + kWave - 1) / kWave};
  }
  return sh;
}

// Shapes that ragged rows are dispatched to (no others: ragged_shapes_exist()).
constexpr int kRaggedFwdMaxPieces = 4;
constexpr int kRaggedBwdMaxPieces = 3;
constexpr bool is_ragged_shape(int lanes, int ch, int vec, bool backward) {
  if (lanes < kWave) return ch == 1 || (ch == 3 && !(backward && vec == 4));
  if (lanes == kWave) return ch <= (backward ? kRaggedBwdMaxPieces : kRaggedFwdMaxPieces);
  if (lanes > 256) return backward;
  return backward ? ch == 2 || ch == 3 || (lanes == 256 && vec == 4 && ch == 4)
                  : ch == 3 || ch == 4 || (lanes == 256 && vec == 4 && ch > 4);
}
constexpr bool ragged_shapes_exist(int vec, bool backward) {
  for (int p = 2; p <= max_fast_pieces(vec); ++p) {
    for (bool many : {false, true}) {
      const Shape sh = shape_of(p, vec, backward ? kRaggedBwdMaxPieces : kRaggedFwdMaxPieces, backward, true, many);
      if (sh.ch == 0 || !is_ragged_shape(sh.lanes, sh.ch, vec, backward)) return false;
    }
  }
  return true;
}
static_assert(ragged_shapes_exist(4, false) && ragged_shapes_exist(4, true), "float32");
static_assert(ragged_shapes_exist(8, false) && ragged_shapes_exist(8, true), "bfloat16");

template <typename T, int L, int C>
static void ln_fwd_go(int rr, bool loop, bool ragged, int grid, hipStream_t st, const void* x, const float* gamma,
                      const float* beta, void* y, float* rstd, float* mean, int64_t N, int64_t M,
                      float eps) {
  if constexpr ((std::is_same<T, bf16_t>::value && C > 4 && L > kWave) || L > kFwdThreads) {
    // shapes that exist for float32 only, or for the backward only (fast_shape never picks them here)
  } else {
    auto launch = [&](auto rows, auto lp, auto rag) {
      hipLaunchKernelGGL((ln_fwd_kernel<T, L, C, decltype(rows)::value, decltype(lp)::value,
                                        decltype(rag)::value>),
                         dim3(grid), dim3(kFwdThreads), 0, st, static_cast<const T*>(x), gamma, beta,
                         static_cast<T*>(y), rstd, mean, N, static_cast<int>(M), eps);
    };
    auto go = [&](auto rows, auto lp) {
      if constexpr (is_ragged_shape(L, C, Store<T>::kVec, false)) {
        if (ragged) return launch(rows, lp, std::true_type{});
      }
      launch(rows, lp, std::false_type{});
    };
    using std::integral_constant;
    if constexpr (C == 1 && L <= 64) {
      if (rr == 4) {
        if (loop) return go(integral_constant<int, 4>{}, std::true_type{});
        return go(integral_constant<int, 4>{}, std::false_type{});
      }
    }
    if constexpr (C <= 2 && L <= 64) {
      if (rr == 2) {
        if (loop) return go(integral_constant<int, 2>{}, std::true_type{});
        return go(integral_constant<int, 2>{}, std::false_type{});
      }
    }
    if (loop) return go(integral_constant<int, 1>{}, std::true_type{});
    go(integral_constant<int, 1>{}, std::false_type{});
  }
}

static bool is_ragged(int64_t M, tempo_dtype dt) { return M % (dt == TEMPO_F32 ? 4 : 8) != 0; }

// Longest rows whose column sums fit the LDS of a compute unit when a wave owns a row: half of the waves' sums at once,
// beside 1 KiB for what the kernel declares itself.
constexpr int64_t kOneWaveBwdColumns = 159 * 1024 / (kBwdWaves / 2 * 2 * sizeof(float));  // 5088
static bool fast_shape(int64_t N, int64_t M, tempo_dtype dt, bool backward, Shape* sh) {
  const int vec = dt == TEMPO_F32 ? 4 : 8;
  if (M < vec || (M + vec - 1) / vec > max_fast_pieces(vec)) return false;
  const int pieces = static_cast<int>((M + vec - 1) / vec);
  const bool ragged = is_ragged(M, dt);
  int max_ch = ragged ? (backward ? kRaggedBwdMaxPieces : kRaggedFwdMaxPieces)
                      : tune_get(backward ? kTuneLnBwdMaxPieces : kTuneLnFwdMaxPieces);
  if (backward && M > kOneWaveBwdColumns && max_ch > 4) max_ch = 4;  // several waves, whatever the knob says
  *sh = shape_of(pieces, vec, max_ch, backward, ragged, N >= int64_t{64} * compute_units());
  return sh->ch != 0;
}

constexpr int kFwdFullBlocks = 3;

tempo_status launch_layernorm_fwd(const void* x, const float* gamma, const float* beta, void* y,
                                  float* rstd, float* mean, int64_t N, int64_t M, float eps,
                                  tempo_dtype dt, hipStream_t st) {
  Shape sh;
  int64_t cap = static_cast<int64_t>(compute_units()) * tune_get(kTuneLnFwdBlocksPerCu);
  if (fast_shape(N, M, dt, false, &sh)) {
    // rows per lane group, if the knob allows more than one: 4 for rows of one piece per lane, 2
    // for two pieces, so that a lane has 4 pieces in flight (and as many fetched ahead when the
    // workgroups loop); rows of one piece also take one more workgroup per compute unit.
    // Measured on 16384 x 512 and 65536 x 256 bf16: 9-10 % faster than 2 rows.
    const int tuned = tune_get(kTuneLnFwdRows);
    int rr = (sh.ch <= 2 && sh.lanes <= kWave && tuned >= 2) ? (sh.ch == 1 ? 4 : 2) : 1;
    // Few rows: fewer per lane group as long as that leaves less than kFwdFullBlocks workgroups per
    // compute unit.  Measured, us at 1, 3 and 4 per unit: 5000 x 512 bf16 5.1, 4.2, 4.2; 10000 x 256
    // f32 5.8, 5.5, 5.5; 30000 x 128 bf16 5.0, 4.8, 5.9; 1024 x 256 f32 3.9 with four rows, 2.2 with one.
    while (rr > 1 && (N + kFwdThreads / sh.lanes * rr - 1) / (kFwdThreads / sh.lanes * rr) <
                         kFwdFullBlocks * compute_units())
      rr >>= 1;
    if (rr == 4) cap += compute_units();
    int groups = (kFwdThreads / sh.lanes) * rr;
    int64_t want = (N + groups - 1) / groups;
    // Rows of two pieces whose workgroups would walk five batches of two rows or more: one row
    // at a time and one more workgroup per compute unit instead (32768 and 65536 rows of 1024
    // bf16 columns: 5-6 % faster; up to 16384 rows the two-row form is as fast or faster).
    if (rr == 2 && want >= 5 * cap) {
      rr = 1;
      cap += compute_units();
      groups = kFwdThreads / sh.lanes;
      want = (N + groups - 1) / groups;
    }
    const bool loop = want > cap;
    const int grid = static_cast<int>(loop ? cap : want);
#define TEMPO_LAUNCH(L, C)                                                                   \
  do {                                                                                       \
    if (dt == TEMPO_F32) ln_fwd_go<float, L, C>(rr, loop, is_ragged(M, dt), grid, st, x, gamma, beta, y, rstd, mean, N, M, eps);   \
    else ln_fwd_go<bf16_t, L, C>(rr, loop, is_ragged(M, dt), grid, st, x, gamma, beta, y, rstd, mean, N, M, eps);    \
  } while (0)
    TEMPO_LN_DISPATCH(TEMPO_LAUNCH)
#undef TEMPO_LAUNCH
  } else {
    // one row per workgroup at a time: as many workgroups as a compute unit holds (8 of 256 lanes)
    const int64_t most = static_cast<int64_t>(compute_units()) * 8;
    const int grid = static_cast<int>(N < most ? N : most);
    auto go = [&](auto tag, auto kc) {
      using T = decltype(tag);
      hipLaunchKernelGGL((ln_fwd_generic_kernel<T, decltype(kc)::value>), dim3(grid), dim3(256), 0,
                         st, static_cast<const T*>(x), gamma, beta, static_cast<T*>(y), rstd, mean, N,
                         M, eps);
    };
    auto by_length = [&](auto tag) {  // columns per thread held in registers: 1 (short rows) or none
      if (M <= 256) go(tag, std::integral_constant<int, 1>{});
      else go(tag, std::integral_constant<int, 0>{});
    };
    if (dt == TEMPO_F32) by_length(float{});
    else by_length(bf16_t{});
  }
  return launch_status();
}

// Launch plan of the register-resident backward kernel.  Rows per lane group and batch (r):
// as many as the knob allows while the packed rows stay within ~64 registers and the grid
// keeps one workgroup per compute unit.  If that leaves more batches than the knob's number of
// workgroups per compute unit (default 1), workgroups loop with prefetch instead (two batches
// are then held in registers: half the rows per batch for one-piece rows, one row otherwise) on
// a grid of that many workgroups per compute unit.  A grid that does not loop has exactly one
// workgroup per batch, however many that is.
// Rows that are no multiple of a piece, and rows too long for the register-resident kernel, use at
// most this many partial slots whatever the knobs say: a workspace of 8 KiB x M.
constexpr int kMaxRaggedSlots = 1024;
struct BwdPlan {
  int r;
  bool loop;
  int grid;
};
static BwdPlan bwd_plan(int64_t N, const Shape& sh, bool ragged) {
  const int tuned = tune_get(kTuneLnBwdRowsPerGroup);
  const int regs_per_row = sh.ch * 8;  // dy and y, 4 registers per packed piece
  const int64_t groups = kBwdThreads / sh.lanes;
  const int cus = compute_units();
  auto batches = [&](int r) { return (N + groups * r - 1) / (groups * r); };
  int r = tuned >= 4 ? 4 : (tuned >= 2 ? 2 : 1);
  const int avail =  // max_rows<L, C>()
      sh.lanes > 64 ? 1 : ((sh.ch <= 2 && sh.lanes == 64) ? 4 : (sh.ch <= 4 ? 2 : 1));
  if (r > avail) r = avail;
  while (r > 1 && (r * regs_per_row > 64 || batches(r) < cus)) r >>= 1;
  int64_t most = static_cast<int64_t>(tune_get(kTuneLnBwdLoopBlocksPerCu)) * cus;
  if (ragged && most > kMaxRaggedSlots) most = kMaxRaggedSlots;
  BwdPlan p;
  if (batches(r) > most) {
    p.loop = true;
    p.r = (r > 1 && sh.ch == 1) ? r / 2 : 1;  // measured: rows of 2 pieces per lane loop best alone
    p.grid = static_cast<int>(most);
  } else {
    p.loop = false;
    p.r = r;
    p.grid = static_cast<int>(batches(r));  // <= most <= 65536 * compute units
  }
  if (p.grid < 1) p.grid = 1;
  return p;
}

// Dynamic LDS of the backward kernel: the column sums' slots (one per kRowWaves waves: all of
// them when they fit kOneStepLdsBytes, else those of the upper half of the workgroup for the
// tree), or the three parameter vectors when they live in LDS.
static size_t bwd_lds_bytes(const Shape& sh, int64_t M, tempo_dtype dt) {
  const int row_waves = sh.lanes > kWave ? sh.lanes / kWave : 1;
  const int all = kBwdWaves / row_waves;
  M = lds_row(M);
  const size_t one_step = static_cast<size_t>(all) * 2 * M * sizeof(float);
  const int slots = one_step <= kOneStepLdsBytes ? all : (all / 2 > 0 ? all / 2 : 1);
  const int vec = dt == TEMPO_F32 ? 4 : 8;
  const bool reg_params = sh.ch * vec <= 24;  // kRegParams of ln_bwd_kernel
  size_t floats = static_cast<size_t>(slots) * 2 * M;
  if (!reg_params && floats < static_cast<size_t>(3) * M) floats = static_cast<size_t>(3) * M;
  return floats * sizeof(float);
}

// Launches the register-resident backward kernel; returns the number of workgroups used (the
// number of partial slots written).  A looping launch is trimmed to the workgroups that are
// resident at once, so that no second round of workgroups repeats the reduction epilogue.
template <typename T, int L, int C>
static int ln_bwd_go(const BwdPlan& plan, bool ragged, size_t lds_bytes, hipStream_t st, const void* dy,
                     const void* y, const float* gamma, const float* beta, const float* rstd,
                     void* dx, float* workspace, int64_t N, int64_t M, int slot_row) {
  int grid = plan.grid;
  if constexpr ((std::is_same<T, bf16_t>::value && ((C > 4 && L > kWave) || (C == 16 && L == kWave))) ||
                (L == 4 * kWave && C * Store<T>::kVec > 24) ||
                (L == kBwdThreads && C != (std::is_same<T, bf16_t>::value ? 2 : 4))) {
    return grid;  // shapes that exist for the other dtype or the forward only
  } else {
    auto launch = [&](auto rows, auto loop, auto rag) {
      auto kernel = ln_bwd_kernel<T, L, C, decltype(rows)::value, decltype(loop)::value,
                                  decltype(rag)::value>;
      if (decltype(loop)::value) {
        static std::atomic<int> resident{0};  // workgroups per compute unit, per instantiation
        int per_cu = resident.load(std::memory_order_relaxed);
        if (per_cu == 0) {
          if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBwdThreads,
                                                           lds_bytes) != hipSuccess || per_cu < 1) {
            (void)hipGetLastError();
            per_cu = 1;
          }
          resident.store(per_cu, std::memory_order_relaxed);
        }
        const int fit = per_cu * compute_units();
        if (grid > fit) grid = fit;
      }
      hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBwdThreads), lds_bytes, st,
                         static_cast<const T*>(dy), static_cast<const T*>(y), gamma, beta, rstd,
                         static_cast<T*>(dx), workspace, N, static_cast<int>(M), slot_row);
    };
    auto go = [&](auto rows, auto loop) {
      if constexpr (is_ragged_shape(L, C, Store<T>::kVec, true)) {
        if (ragged) return launch(rows, loop, std::true_type{});
      }
      launch(rows, loop, std::false_type{});
    };
    using std::integral_constant;
    if (plan.loop) {
      if constexpr (max_rows<L, C>() >= 4) {  // looping holds two batches: half the rows
        if (plan.r == 2) {
          go(integral_constant<int, 2>{}, std::true_type{});
          return grid;
        }
      }
      go(integral_constant<int, 1>{}, std::true_type{});
      return grid;
    }
    if constexpr (max_rows<L, C>() >= 4) {
      if (plan.r == 4) {
        go(integral_constant<int, 4>{}, std::false_type{});
        return grid;
      }
    }
    if constexpr (max_rows<L, C>() >= 2) {
      if (plan.r >= 2) {
        go(integral_constant<int, 2>{}, std::false_type{});
        return grid;
      }
    }
    go(integral_constant<int, 1>{}, std::false_type{});
    return grid;
  }
}

// Most rows that ln_bwd_few_kernel takes: a column's rows are walked in steps of 128, and the longest float32
// rows, 6 or 8 pieces per lane, cost more to read twice than the second dispatch.  Backward, two launches / one, us:
// f32 256x768 5.7 / 3.0, 640x768 6.6 / 4.5, 640x1001 7.3 / 6.7, 640x4096 14.0 / 12.7, 640x6144 18.4 / 16.8, 320x8187 18.4 /
// 18.1, 384x8187 18.6 / 20.5, 640x8187 22.5 / 30.3, 320x6143 14.3 / 13.6, 384x6143 14.5 / 15.0, 640x5001 17.0 / 17.8, 576x6148
// 17.3 / 18.1, 640x8192 20.9 / 23.7; bf16 256x1024 6.0 / 2.9, 640x1024 6.5 / 3.4, 640x4096 12.1 / 7.8, 640x8191 19.5 / 19.3.
// Beyond 640 rows, forward + backward: f32 1024x768 10.8 / 10.8, 768x4096 20.9 / 21.6, bf16 1024x1024 10.6 / 11.2.  In place the columns have to be summed before dx is written, in a
// launch of their own, which only 64 rows and the longer bfloat16 ones gain by (f32 64x768 5.6 / 5.4, 256x768 5.7 / 6.8,
// 640x4096 14.0 / 16.7, bf16 640x1024 6.3 / 9.4, 256x4096 8.9 / 7.6); the rule is the same, for dx, dgamma and dbeta to have
// the bits of the call apart.
constexpr int64_t kFewRows = 640;
constexpr int64_t kFewLongRows = 320;  // float32, of more than 4096 columns if ragged, of more than 6144 if not
static bool overlap(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + b_bytes && y < x + a_bytes;
}
// Lanes and pieces per lane of a row in ln_bwd_few_kernel: a wave while that leaves at most four pieces, else
// four waves.
constexpr Shape few_shape(int pieces) {
  for (int ch = 1; ch <= 4; ++ch)
    if (pieces <= ch * kWave) return {kWave, ch};
  for (int ch : {2, 3, 4, 6, 8})
    if (pieces <= ch * 4 * kWave) return {4 * kWave, ch};
  return {0, 0};
}
static bool few_rows(int64_t N, int64_t M, tempo_dtype dt) {
  const int vec = dt == TEMPO_F32 ? 4 : 8;
  const bool is_long = dt == TEMPO_F32 && M > (is_ragged(M, dt) ? 4096 : 6144);
  return N >= 1 && N <= (is_long ? kFewLongRows : kFewRows) && M >= vec && (M + vec - 1) / vec <= max_fast_pieces(vec);
}
template <typename T>
static tempo_status ln_bwd_few(bool ragged, bool in_place, hipStream_t st, const void* dy, const void* y, const float* gamma,
                               const float* beta, const float* rstd, void* dx, float* dgamma, float* dbeta, int64_t N,
                               int64_t M) {
  const int pieces = static_cast<int>((M + Store<T>::kVec - 1) / Store<T>::kVec);
  const Shape sh = few_shape(pieces);
  const int col_blocks = (pieces + kFewColLanes - 1) / kFewColLanes;
  const int groups = kFewThreads / sh.lanes;
  const int grid = col_blocks + static_cast<int>((N + groups - 1) / groups);
  auto go = [&](auto lanes, auto ch) {
    auto launch = [&](auto rag, int first, int count) {
      hipLaunchKernelGGL((ln_bwd_few_kernel<T, decltype(lanes)::value, decltype(ch)::value, decltype(rag)::value>),
                         dim3(count), dim3(kFewThreads), 0, st, static_cast<const T*>(dy), static_cast<const T*>(y),
                         gamma, beta, rstd, static_cast<T*>(dx), dgamma, dbeta, static_cast<int>(N),
                         static_cast<int>(M), col_blocks, first);
      return launch_status();
    };
    auto halves = [&](auto rag) {
      if (!in_place) return launch(rag, 0, grid);
      const tempo_status columns = launch(rag, 0, col_blocks);
      return columns != TEMPO_OK ? columns : launch(rag, col_blocks, grid - col_blocks);
    };
    return ragged ? halves(std::true_type{}) : halves(std::false_type{});
  };
  using std::integral_constant;
  constexpr integral_constant<int, kWave> wave{};
  constexpr integral_constant<int, 4 * kWave> waves{};
  switch (sh.lanes * 100 + sh.ch) {
    case 6401: return go(wave, integral_constant<int, 1>{});
    case 6402: return go(wave, integral_constant<int, 2>{});
    case 6403: return go(wave, integral_constant<int, 3>{});
    case 6404: return go(wave, integral_constant<int, 4>{});
    case 25602: return go(waves, integral_constant<int, 2>{});
    case 25603: return go(waves, integral_constant<int, 3>{});
    case 25604: return go(waves, integral_constant<int, 4>{});
  }
  if constexpr (std::is_same<T, float>::value) {
    if (sh.ch == 6) return go(waves, integral_constant<int, 6>{});
    if (sh.ch == 8) return go(waves, integral_constant<int, 8>{});
  }
  return TEMPO_ERR_UNSUPPORTED;
}

// Everything a backward launch depends on, taken from the knobs once: the workspace check and
// the launch of one call always see the same plan.
struct BwdLaunch {
  bool fast;    // register-resident kernel (else the any-M kernel)
  Shape sh;
  BwdPlan plan;
  int slots;    // partial [2][M] slots the row kernel may write: an upper bound of its grid
};
static BwdLaunch bwd_launch(int64_t N, int64_t M, tempo_dtype dt) {
  BwdLaunch b;
  b.fast = fast_shape(N, M, dt, true, &b.sh);
  // rows that are no multiple of a piece: one slot per row up to kMaxRaggedSlots, for either kernel
  const int per_row = static_cast<int>(N > kMaxRaggedSlots ? kMaxRaggedSlots : (N < 1 ? 1 : N));
  if (b.fast) {
    b.plan = bwd_plan(N, b.sh, is_ragged(M, dt));
    b.slots = is_ragged(M, dt) ? per_row : b.plan.grid;
  } else {
    b.plan = {1, true, per_row};  // one row per workgroup, strided; four workgroups per compute unit
    b.slots = per_row;
  }
  return b;
}
static size_t slot_bytes(const BwdLaunch& b, int64_t M) {
  return static_cast<size_t>(b.slots) * 2 * static_cast<size_t>(M) * sizeof(float);
}

size_t layernorm_bwd_workspace_bytes(int64_t N, int64_t M, tempo_dtype dt) {
  return slot_bytes(bwd_launch(N, M, dt), M);
}

tempo_status launch_layernorm_bwd(const void* dy, const void* y, const float* gamma,
                                  const float* beta, const float* rstd, void* dx, float* dgamma,
                                  float* dbeta, float* workspace, size_t workspace_bytes,
                                  int64_t N, int64_t M, tempo_dtype dt, hipStream_t st) {
  const BwdLaunch b = bwd_launch(N, M, dt);
  if (workspace_bytes < slot_bytes(b, M)) return TEMPO_ERR_WORKSPACE;
  if (few_rows(N, M, dt)) {
    const int64_t act = N * M * (dt == TEMPO_F32 ? 4 : 2), par = M * 4;
    const bool in_place = overlap(dx, act, dy, act) || overlap(dx, act, y, act);
    // dgamma or dbeta in the place of an input: left to the row kernel, which has read it all before they are written
    bool apart = true;
    auto keep_apart = [&](const void* in, int64_t bytes) {
      apart = apart && !overlap(dgamma, par, in, bytes) && !overlap(dbeta, par, in, bytes);
    };
    keep_apart(dy, act);
    keep_apart(y, act);
    keep_apart(gamma, par);
    keep_apart(beta, par);
    keep_apart(rstd, N * 4);
    if (apart)
      return dt == TEMPO_F32
                 ? ln_bwd_few<float>(is_ragged(M, dt), in_place, st, dy, y, gamma, beta, rstd, dx, dgamma, dbeta, N, M)
                 : ln_bwd_few<bf16_t>(is_ragged(M, dt), in_place, st, dy, y, gamma, beta, rstd, dx, dgamma, dbeta, N, M);
  }
  int grid = b.plan.grid;
  // Ragged rows' slots in whole 16-byte pieces, if the workspace, which is sized in rows of M, has room for that: it
  // nearly always is sized for more slots than the launch has workgroups.  Backward, us, slot rows of M / padded: f32
  // 1000x1001 9.5 / 8.8, 2048x1023 10.8 / 9.5, 8192x1001 24.0 / 23.5; bf16 2048x1001 9.8 / 9.4, 4096x4095 28.6 / 26.9.
  int64_t slot_row = M;
  if (b.fast && grid * lds_row(M) <= b.slots * M) slot_row = lds_row(M);
  if (b.fast) {
    const Shape sh = b.sh;
    const size_t lds_bytes = bwd_lds_bytes(sh, M, dt);
    const BwdPlan plan = b.plan;
#define TEMPO_LAUNCH(L, C)                                                                   \
  do {                                                                                       \
    if (dt == TEMPO_F32) grid = ln_bwd_go<float, L, C>(plan, is_ragged(M, dt), lds_bytes, st, dy, y, gamma, beta, rstd, dx, workspace, N, M, static_cast<int>(slot_row));   \
    else grid = ln_bwd_go<bf16_t, L, C>(plan, is_ragged(M, dt), lds_bytes, st, dy, y, gamma, beta, rstd, dx, workspace, N, M, static_cast<int>(slot_row));                  \
  } while (0)
    TEMPO_LN_DISPATCH(TEMPO_LAUNCH)
#undef TEMPO_LAUNCH
  } else {
    auto go = [&](auto tag, auto kc) {
      using T = decltype(tag);
      hipLaunchKernelGGL((ln_bwd_generic_kernel<T, decltype(kc)::value>), dim3(grid), dim3(256), 0,
                         st, static_cast<const T*>(dy), static_cast<const T*>(y), gamma, beta, rstd,
                         static_cast<T*>(dx), workspace, N, M);
    };
    auto by_length = [&](auto tag) {  // columns per thread held in registers: 1 (short rows) or none
      if (M <= 256) go(tag, std::integral_constant<int, 1>{});
      else go(tag, std::integral_constant<int, 0>{});
    };
    if (dt == TEMPO_F32) by_length(float{});
    else by_length(bf16_t{});
  }
  if (hipGetLastError() != hipSuccess) return TEMPO_ERR_LAUNCH;
  const int fgrid = static_cast<int>((2 * slot_row + kFinCols - 1) / kFinCols);
  auto finalize = slot_row % 2 == 0 ? ln_bwd_finalize_kernel<false> : ln_bwd_finalize_kernel<true>;
  hipLaunchKernelGGL(finalize, dim3(fgrid), dim3(kFinVecLanes * kFinSlices), 0, st, workspace,
                     dgamma, dbeta, grid, M, slot_row);
  return launch_status();
}

// Scratch for callers that cannot allocate: one array per GPU, living in the code object.  Its
// name is only a host-side handle; the address kernels can use is looked up once per device.
static __device__ __align__(256) unsigned char scratch[TEMPO_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

tempo_status static_scratch(void** ptr) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return TEMPO_ERR_LAUNCH;
  }
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (p == nullptr) {  // first call on this device (threads racing here find the same address)
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return TEMPO_ERR_LAUNCH;
    }
    g_scratch_ptr[dev].store(p, std::memory_order_release);
  }
  *ptr = p;
  return TEMPO_OK;
}

}  // namespace tempo
