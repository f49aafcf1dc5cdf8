// Device-side helpers shared by the gfx950 kernels: 128-bit vector access for float32 and
// bfloat16 storage, wave64 reductions, and launch utilities.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/tempo.h"

namespace tempo {

constexpr int kWave = 64;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));  // a 16-byte piece at any element's address
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct bf16_t {
  uint16_t bits;
};

__device__ __forceinline__ float as_f32(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_u32(float f) { return __builtin_bit_cast(uint32_t, f); }

// Round two floats to bfloat16 (nearest even, hardware v_cvt_pk_bf16_f32) and pack lo|hi<<16.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return as_f32(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return as_f32(w & 0xFFFF0000u); }
// Value a float takes after a round trip through bfloat16 storage.
__device__ __forceinline__ float round_bf16(float v) {
  return as_f32(pack_bf16(v, 0.0f) << 16);
}

// Storage traits.  All bulk traffic moves in 16-byte "pieces": 8 consecutive bfloat16 or 4
// consecutive float32 elements.  Kernels are laid out so that the 64 lanes of a wave touch 64
// adjacent pieces with one instruction (1 KiB contiguous): a lane that instead owned 32
// adjacent bytes of float32 (two accesses, each strided by 32 bytes across the wave) was
// measured at 4.0 TB/s where the contiguous form reaches 6.2 TB/s.
// A piece needs a 16-byte aligned address: base pointers are checked on the host and element
// offsets are multiples of the piece length.
template <typename T>
struct Store;

template <>
struct Store<float> {
  static constexpr int kVec = 4;  // elements per piece
  __device__ static __forceinline__ float load1(const float* p) { return *p; }
  __device__ static __forceinline__ void store1(float* p, float v) { *p = v; }
  __device__ static __forceinline__ float round(float v) { return v; }
  __device__ static __forceinline__ void unpack(const u32x4 w, float (&v)[4]) {
    v[0] = as_f32(w.x); v[1] = as_f32(w.y); v[2] = as_f32(w.z); v[3] = as_f32(w.w);
  }
  __device__ static __forceinline__ u32x4 pack(const float (&v)[4]) {
    return u32x4{as_u32(v[0]), as_u32(v[1]), as_u32(v[2]), as_u32(v[3])};
  }
  __device__ static __forceinline__ u32x4 neg_inf_piece() {
    return u32x4{0xFF800000u, 0xFF800000u, 0xFF800000u, 0xFF800000u};
  }
};

template <>
struct Store<bf16_t> {
  static constexpr int kVec = 8;
  __device__ static __forceinline__ float load1(const bf16_t* p) {
    return as_f32(static_cast<uint32_t>(p->bits) << 16);
  }
  __device__ static __forceinline__ void store1(bf16_t* p, float v) {
    p->bits = static_cast<uint16_t>(pack_bf16(v, 0.0f) & 0xFFFFu);
  }
  __device__ static __forceinline__ float round(float v) { return round_bf16(v); }
  __device__ static __forceinline__ void unpack(const u32x4 w, float (&v)[8]) {
    v[0] = bf16_lo(w.x); v[1] = bf16_hi(w.x);
    v[2] = bf16_lo(w.y); v[3] = bf16_hi(w.y);
    v[4] = bf16_lo(w.z); v[5] = bf16_hi(w.z);
    v[6] = bf16_lo(w.w); v[7] = bf16_hi(w.w);
  }
  __device__ static __forceinline__ u32x4 pack(const float (&v)[8]) {
    return u32x4{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]),
                 pack_bf16(v[6], v[7])};
  }
  __device__ static __forceinline__ u32x4 neg_inf_piece() {
    return u32x4{0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u};
  }
};

// Streaming (non-temporal) 16-byte accesses for data that is touched exactly once.  Also for what a backward
// reads again: plain stores leave it in the 256 MiB Infinity Cache for a backward that comes next, but in a
// model those of other layers come first.  8x12x1024x1024 bf16 causal attention on fresh buffers, us, streamed / the
// first 64 MiB / 192 MiB of probs stored plainly: forward + backward 211 / 207 / 196, eight layers' forwards and then their
// backwards 212 / 215 / 213 a layer; bf16 GELU 8192x4096 61.3 / 59.7 / 59.4 and 61.3 / 63.7 / 62.1.
__device__ __forceinline__ u32x4 ldg_stream(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ void stg_stream(void* p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}
// The same at an address that is only a multiple of the element size (rows whose length is no
// multiple of a piece).  The instructions are the same 16-byte ones: global memory takes them at
// any address.  Measured on a plain kernel moving 57 MB per tensor (bfloat16 addresses off by one
// element): loads 4-7 % slower than aligned, stores another 6-12 %; element-wise accesses, the
// alternative, reach a third of the rate.
__device__ __forceinline__ u32x4 ldg_stream_any(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p));
}
__device__ __forceinline__ void stg_stream_any(void* p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any*>(p));
}
template <bool ANY>
__device__ __forceinline__ u32x4 ldg_piece(const void* p) {
  if constexpr (ANY) return ldg_stream_any(p);
  else return ldg_stream(p);
}
template <bool ANY>
__device__ __forceinline__ void stg_piece(void* p, u32x4 v) {
  if constexpr (ANY) stg_stream_any(p, v);
  else stg_stream(p, v);
}
template <typename T>
__device__ __forceinline__ void load_piece(const T* p, float (&v)[Store<T>::kVec]) {
  Store<T>::unpack(ldg_stream(p), v);
}
template <typename T>
__device__ __forceinline__ void store_piece(T* p, const float (&v)[Store<T>::kVec]) {
  stg_stream(p, Store<T>::pack(v));
}
// float32 parameters (gamma, beta, LDS tables): plain cached accesses of kVec floats
template <int V>
__device__ __forceinline__ void load_floats(const float* p, float (&v)[V]) {
  static_assert(V == 4 || V == 8, "piece length");
  const f32x4 a = *reinterpret_cast<const f32x4*>(p);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  if constexpr (V == 8) {
    const f32x4 b = *reinterpret_cast<const f32x4*>(p + 4);
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
}
// The same at any float's address (rows of parameters or column sums whose length is odd).
typedef f32x4 f32x4_any __attribute__((aligned(4)));
template <int V>
__device__ __forceinline__ void load_floats_any(const float* p, float (&v)[V]) {
  static_assert(V == 4 || V == 8, "piece length");
#pragma unroll
  for (int h = 0; h < V; h += 4) {
    const f32x4 a = *reinterpret_cast<const f32x4_any*>(p + h);
    v[h] = a.x; v[h + 1] = a.y; v[h + 2] = a.z; v[h + 3] = a.w;
  }
}
template <int V>
__device__ __forceinline__ void store_floats_any(float* p, const float (&v)[V]) {
  static_assert(V == 4 || V == 8, "piece length");
#pragma unroll
  for (int h = 0; h < V; h += 4)
    *reinterpret_cast<f32x4_any*>(p + h) = f32x4{v[h], v[h + 1], v[h + 2], v[h + 3]};
}
template <int V>
__device__ __forceinline__ void store_floats(float* p, const float (&v)[V]) {
  static_assert(V == 4 || V == 8, "piece length");
  *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
  if constexpr (V == 8) *reinterpret_cast<f32x4*>(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
}

// Rows of any length ("ragged": no multiple of the piece).  A row is owned in pieces counted from
// its own start, at element-aligned addresses; the last piece is moved back to end with the row, so
// that no access leaves the row and none is partial.  The elements it shares with the piece before
// ("dup", at most V - 1, the first ones of the piece) are computed and stored twice with the same
// value and left out of the row sums.  A row shorter than a piece has one piece at column 0 that
// the kernel has to treat on its own.  pc: piece of the row, pieces: how many the row has.
template <bool RAG, int V>
__device__ __forceinline__ int piece_col(int pc, int pieces, int len) {
  return (RAG && pc == pieces - 1) ? max(len - V, 0) : pc * V;
}
template <bool RAG, int V>
__device__ __forceinline__ int piece_dup(int pc, int pieces, int len) {
  return (RAG && pc == pieces - 1 && len >= V) ? pieces * V - len : 0;
}

// Raw (still packed) piece, so rows fetched ahead cost 4 registers per piece.
template <typename T>
struct Raw {
  u32x4 a;
  __device__ __forceinline__ void load(const T* p) { a = ldg_stream(p); }
  __device__ __forceinline__ void unpack(float (&v)[Store<T>::kVec]) const {
    Store<T>::unpack(a, v);
  }
};

// Guarded piece access: elements at or beyond `n_left` (counted from p) are absent.
template <typename T>
__device__ __forceinline__ void load_piece_guarded(const T* p, int64_t n_left,
                                                   float (&v)[Store<T>::kVec], float fill) {
  constexpr int V = Store<T>::kVec;
  if (n_left >= V) {
    load_piece<T>(p, v);
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = (i < n_left) ? Store<T>::load1(p + i) : fill;
  }
}
template <typename T>
__device__ __forceinline__ void store_piece_guarded(T* p, int64_t n_left,
                                                    const float (&v)[Store<T>::kVec]) {
  constexpr int V = Store<T>::kVec;
  if (n_left >= V) {
    store_piece<T>(p, v);
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (i < n_left) Store<T>::store1(p + i, v[i]);
  }
}

// Cross-lane moves inside a row of 16 lanes through DPP (data-parallel primitives: the source
// lane is selected by the instruction itself, no LDS round trip).  The four controls below
// pair every lane with lane^1, lane^2 (quad permutes), then mirror 8 and 16 lanes, which for
// values already equal inside a quad / half row acts like lane^4 and lane^8.
constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // row_half_mirror
constexpr int kDppMirror = 0x140;      // row_mirror
constexpr int kDppRor4 = 0x124;        // row_ror: rotations inside the 16 lanes
constexpr int kDppRor8 = 0x128;
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return as_f32(dpp_u32<CTRL>(as_u32(v)));
}

// The values of the lanes 16 (32) away, added to or compared with the lane's own: v_permlane16_swap
// (v_permlane32_swap) exchanges the odd 16-lane rows of one register with the even rows of another
// (the upper half with the lower half), so that of two copies of v each lane then holds both its own
// and the other's value: a move and a swap on the vector ALU instead of an LDS round trip.
template <int N, typename F>
__device__ __forceinline__ float across_rows(float v, F&& f) {
  static_assert(N == 16 || N == 32, "distance");
  const uint32_t u = as_u32(v);
  if constexpr (N == 16) {
    const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return f(as_f32(p[0]), as_f32(p[1]));
  } else {
    const auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return f(as_f32(p[0]), as_f32(p[1]));
  }
}

// Butterfly reductions over groups of LANES consecutive lanes of a wave (LANES a power of
// two, 4 <= LANES <= 64, groups aligned to LANES); every lane of the group ends with the
// result.  Steps inside a 16-lane row use DPP, the steps across rows v_permlane*_swap.
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(LANES >= 4 && LANES <= 64, "group size");
  v += dpp_f32<kDppXor1>(v);
  v += dpp_f32<kDppXor2>(v);
  if (LANES >= 8) v += dpp_f32<kDppHalfMirror>(v);
  if (LANES >= 16) v += dpp_f32<kDppMirror>(v);
  auto add = [](float a, float b) { return a + b; };
  if (LANES >= 32) v = across_rows<16>(v, add);
  if (LANES >= 64) v = across_rows<32>(v, add);
  return v;
}
template <int LANES>
__device__ __forceinline__ float group_max(float v) {
  static_assert(LANES >= 4 && LANES <= 64, "group size");
  v = fmaxf(v, dpp_f32<kDppXor1>(v));
  v = fmaxf(v, dpp_f32<kDppXor2>(v));
  if (LANES >= 8) v = fmaxf(v, dpp_f32<kDppHalfMirror>(v));
  if (LANES >= 16) v = fmaxf(v, dpp_f32<kDppMirror>(v));
  auto larger = [](float a, float b) { return fmaxf(a, b); };
  if (LANES >= 32) v = across_rows<16>(v, larger);
  if (LANES >= 64) v = across_rows<32>(v, larger);
  return v;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits until the wave's
// outstanding global loads and stores have completed (s_waitcnt vmcnt(0)): behind a batch of
// stores that is microseconds, and in a loop it also waits for the rows fetched ahead.  No
// kernel here passes data between the waves of a workgroup through global memory.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders the LDS traffic of one wave: what its lanes wrote before is what they read after.  (The
// hardware keeps a wave's LDS operations in order; this keeps the compiler from moving them.)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Lanes that reduce by butterflies alone: those of a row inside one wave, a wave of a row over several, the
// largest power of two in rows of 24, 48 or 96 lanes, which lie across waves.
constexpr int butterfly_lanes(int lanes) {
  return lanes >= kWave && lanes % kWave == 0 ? kWave : (lanes & -lanes);
}

// Row reductions for rows owned by LANES consecutive threads of a workgroup.  A row inside
// one wave: butterflies.  Any other: a butterfly per unit (butterfly_lanes), then one
// exchange through `slots` (one entry per unit of the workgroup) behind a workgroup barrier, so
// every thread of the workgroup has to make the call; consecutive calls must alternate between
// two slot arrays (a fast wave may already write its next value while a slow one still reads).
// Every lane of the row ends with the same result.
template <int LANES, bool MAX>
__device__ __forceinline__ float row_reduce(float v, float* slots) {
  constexpr int U = butterfly_lanes(LANES);
  v = MAX ? group_max<U>(v) : group_sum<U>(v);
  if constexpr (U < LANES) {
    if (threadIdx.x % U == 0) slots[threadIdx.x / U] = v;
    lds_barrier();
    constexpr int W = LANES / U;
    const int w0 = (threadIdx.x / LANES) * W;
    v = slots[w0];
#pragma unroll
    for (int k = 1; k < W; ++k) v = MAX ? fmaxf(v, slots[w0 + k]) : v + slots[w0 + k];
  }
  return v;
}

// Two sums at once (one barrier for both); slots holds two floats per wave of the workgroup.
template <int LANES>
__device__ __forceinline__ void row_sum2(float& a, float& b, float2* slots) {
  if constexpr (LANES <= kWave) {
    a = group_sum<LANES>(a);
    b = group_sum<LANES>(b);
  } else {
    a = group_sum<kWave>(a);
    b = group_sum<kWave>(b);
    if ((threadIdx.x & (kWave - 1)) == 0) slots[threadIdx.x / kWave] = make_float2(a, b);
    lds_barrier();
    constexpr int W = LANES / kWave;
    const int w0 = (threadIdx.x / LANES) * W;
    float2 r = slots[w0];
#pragma unroll
    for (int k = 1; k < W; ++k) {
      r.x += slots[w0 + k].x;
      r.y += slots[w0 + k].y;
    }
    a = r.x;
    b = r.y;
  }
}

// Merge the per-piece mask bits of the lanes that share a 32-bit mask word: 4 lanes with 8 bits
// each (bfloat16 pieces) or 8 lanes with 4 bits each (float32 pieces).  `lane` is the index of
// the lane's piece within its row/tile (only its low bits matter).  Every lane of the sharing
// group returns the whole word.
template <int V>
__device__ __forceinline__ uint32_t merge_mask_word(uint32_t bits, int lane) {
  static_assert(V == 4 || V == 8, "piece length");
  constexpr int kLanes = 32 / V;
  uint32_t w = bits << (V * (lane & (kLanes - 1)));
  w |= dpp_u32<kDppXor1>(w);
  w |= dpp_u32<kDppXor2>(w);
  if (V == 4) w |= dpp_u32<kDppHalfMirror>(w);
  return w;
}

// n / d for 32-bit n by a multiplication (Granlund, Montgomery, PLDI'94, the round-up form): a
// division by a run-time value is some 20 dependent instructions before a kernel's first load.
struct FastDiv {
  uint32_t d, m, s1, s2;
  FastDiv() = default;
  explicit FastDiv(uint32_t divisor) : d(divisor) {
    int l = 0;
    while (l < 32 && (uint64_t{1} << l) < d) ++l;
    m = static_cast<uint32_t>(((uint64_t{1} << 32) * ((uint64_t{1} << l) - d)) / d + 1);
    s1 = l < 1 ? l : 1;
    s2 = l > 0 ? l - 1 : 0;
  }
  __host__ __device__ __forceinline__ uint32_t divide(uint32_t n) const {
    const uint32_t t = static_cast<uint32_t>((static_cast<uint64_t>(m) * n) >> 32);
    return (t + ((n - t) >> s1)) >> s2;
  }
};

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace tempo
