// Attention softmax -> dropout sublayer for gfx950 (Sec. 3.3, 3.4; App. E.3, E.4).
//
// Forward keeps only P (the softmax output) and a 1-bit keep mask; the dropout output is a
// transient.  Backward rebuilds the dropout output from (P, mask) by one multiply and derives
// the score gradient from P alone.  A group of LANES lanes owns one row in registers (CH
// 16-byte pieces per lane, piece c of lane t = c*LANES + t so every access of a group is
// contiguous).  The keep bits come from Philox4x32-10, one call per 8 elements, so the mask is
// a pure function of (seed, offset, element index) and does not depend on the launch shape;
// backward can therefore also draw the bits again instead of reading a stored mask.
#include <algorithm>
#include <type_traits>

#include "launch_split.h"
#include "tempo_device.h"
#include "tempo_host.h"

namespace tempo {
namespace {

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

struct RngArgs {
  uint32_t seed_lo, seed_hi, off_lo, off_hi;
  uint32_t t16;  // keep iff 16-bit draw < t16; 65536 keeps everything (generator skipped)
};

// a ^ b ^ c in one VALU op (v_bitop3_b32 with truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32->64 multiplies,
// the key advanced by the two Weyl constants between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&w)[4]) {
  // keeps the 18 round keys out of loops around the call: they would not fit the scalar registers,
  // and adding is cheaper than fetching them back from the lanes of a spilled one
  asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c0;
    const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c2;
    const uint32_t n0 = xor3(static_cast<uint32_t>(p1 >> 32), c1, k0);
    const uint32_t n2 = xor3(static_cast<uint32_t>(p0 >> 32), c3, k1);
    c1 = static_cast<uint32_t>(p1);
    c3 = static_cast<uint32_t>(p0);
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}

// Keep bits of the 8 elements whose draws are w (bit i = element i of the group).  A 16-bit draw r
// is kept iff r < t16, i.e. iff r - t16 is negative: v_alignbit shifts that sign bit into the byte,
// last element first.
__device__ __forceinline__ uint32_t draws_to_byte(const uint32_t (&w)[4], uint32_t t16) {
  uint32_t byte = 0;
#pragma unroll
  for (int i = 3; i >= 0; --i) {
    byte = __builtin_amdgcn_alignbit(byte, (w[i] >> 16) - t16, 31);      // byte << 1 | sign
    byte = __builtin_amdgcn_alignbit(byte, (w[i] & 0xFFFFu) - t16, 31);
  }
  return byte;
}

// Draws of group base + off.
__device__ __forceinline__ void draw_group(uint64_t base, uint32_t off, const RngArgs& a,
                                           uint32_t (&w)[4]) {
  const uint64_t g = base + off;
  philox4x32_10(static_cast<uint32_t>(g), static_cast<uint32_t>(g >> 32), a.off_lo, a.off_hi,
                a.seed_lo, a.seed_hi, w);
}

__device__ __forceinline__ uint32_t keep_byte(uint64_t base, uint32_t off, const RngArgs& a) {
  if (a.t16 >= 65536u) return 0xFFu;
  uint32_t w[4];
  draw_group(base, off, a, w);
  return draws_to_byte(w, a.t16);
}

// The keep decisions of a group in two forms a bfloat16 piece needs, without going through single
// bits: flag words (0 or 1 in each half, one word per two elements) by a saturating subtraction and
// a minimum, both packed 16-bit operations.  Spelled as instructions: from C++ the compiler makes
// compares and selects, twice as many.
__device__ __forceinline__ uint32_t keep_flags(uint32_t draws, uint32_t t16_pair) {
  uint32_t f;
  asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(f) : "s"(t16_pair), "v"(draws));  // 0 iff draw >= t16
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(f) : "v"(f), "s"(0x00010001u));
  return f;
}
__device__ __forceinline__ uint32_t flags_to_mask(uint32_t f) {  // 0 or 0xFFFF in each half
  uint32_t m;
  asm("v_pk_sub_u16 %0, 0, %1" : "=v"(m) : "v"(f));
  return m;
}
__device__ __forceinline__ uint32_t flags_to_byte(const uint32_t (&f)[4]) {
  const uint32_t even = f[0] | (f[1] << 2) | (f[2] << 4) | (f[3] << 6);  // odd elements 16 higher
  return (even | (even >> 15)) & 0xFFu;
}

// All ones if bit K of bits is set, else zero.  Written as the instruction itself: spelled in
// C++ the compiler turns the following AND into test + compare + select, three operations per
// element where two suffice (these kernels run close to the vector-ALU limit).
template <int K>
__device__ __forceinline__ uint32_t bit_mask(uint32_t bits) {
  uint32_t m;
  asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(bits), "n"(K));
  return m;
}

// Zero the dropped elements of a packed piece: keep bit i belongs to element i of the piece.
// bfloat16 words hold two elements: their two masks are merged byte-wise (v_perm_b32).
template <typename T>
__device__ __forceinline__ u32x4 apply_keep(u32x4 w, uint32_t bits) {
  if constexpr (Store<T>::kVec == 4) {
    w.x &= bit_mask<0>(bits);
    w.y &= bit_mask<1>(bits);
    w.z &= bit_mask<2>(bits);
    w.w &= bit_mask<3>(bits);
  } else {
    constexpr uint32_t kLoHalves = 0x05040100u;  // bytes 0,1 of the second source, then of the first
    w.x &= __builtin_amdgcn_perm(bit_mask<1>(bits), bit_mask<0>(bits), kLoHalves);
    w.y &= __builtin_amdgcn_perm(bit_mask<3>(bits), bit_mask<2>(bits), kLoHalves);
    w.z &= __builtin_amdgcn_perm(bit_mask<5>(bits), bit_mask<4>(bits), kLoHalves);
    w.w &= __builtin_amdgcn_perm(bit_mask<7>(bits), bit_mask<6>(bits), kLoHalves);
  }
  return w;
}


// Element `off` of p, p the same for the whole wave: a scalar address and a 32-bit offset.  (The
// offsets stay inside one set of rows: at most 64 rows of a piece per lane, or fewer of up to 8192 elements.)
template <typename T>
__device__ __forceinline__ T* at_offset(T* p, uint32_t off) {
  using Byte = std::conditional_t<std::is_const<T>::value, const char, char>;
  return reinterpret_cast<T*>(reinterpret_cast<Byte*>(p) + off * static_cast<uint32_t>(sizeof(T)));
}

// Element offset of the start of a row: rows are counted in 32 bits on the register-resident
// paths (the host checks), so the product is one 32x32->64 multiply instead of a 64x64 one.
__device__ __forceinline__ int64_t row_offset(uint32_t row, int Sk) {
  return static_cast<int64_t>(static_cast<uint64_t>(row) * static_cast<uint32_t>(Sk));
}

// Number of leading key columns of query row i that take part in the softmax.
__device__ __forceinline__ int row_limit(int i, int key_limit, int causal, int Sq, int Sk) {
  int limit = key_limit;
  if (causal) limit = min(limit, max(i + (Sk - Sq) + 1, 0));
  return limit;
}

// Keep bits of the CH pieces a lane owns in one row.  Piece c of the lane is piece off + c*LANES + t
// counted from group `base`.  bfloat16 pieces (8 elements) are whole Philox groups.  float32 pieces
// (4 elements) are half groups: lanes 2k and 2k+1 hold the two halves of the same group for
// every c, so the pair splits the generator calls (the even lane draws the groups of even c,
// the odd lane those of odd c) and swaps the bytes with one DPP move.
template <typename T, int LANES, int CH>
__device__ __forceinline__ void lane_keep_bits(uint64_t base, uint32_t off, int t,
                                               const RngArgs& rng, uint32_t (&bits)[CH]) {
  if constexpr (Store<T>::kVec == 8) {
#pragma unroll
    for (int c = 0; c < CH; ++c) bits[c] = keep_byte(base, off + c * LANES + t, rng);
  } else {
    const int odd = t & 1;
#pragma unroll
    for (int c = 0; c < CH; c += 2) {
      const int mine = (c + 1 < CH) ? c + odd : c;  // a trailing single piece: both lanes draw
      const uint32_t own = keep_byte(base, (off + mine * LANES + t) >> 1, rng);
      const uint32_t other = dpp_u32<kDppXor1>(own);
      const uint32_t even_c = (c + 1 < CH) ? (odd ? other : own) : own;
      bits[c] = (even_c >> (4 * odd)) & 0xFu;
      if (c + 1 < CH) bits[c + 1] = ((odd ? own : other) >> (4 * odd)) & 0xFu;
    }
  }
}

// Store the mask bits of one piece.  WORDS (Sk % 32 == 0): the lanes sharing a word merge their
// bits and one of them writes the word; otherwise (Sk % 8 == 0) bytes are written: by every
// lane (bf16) or by the even lane of each pair (f32).  All lanes of the sharing group must
// call this together; `valid` says whether the lane's piece exists.
template <typename T, bool WORDS>
__device__ __forceinline__ void store_keep_bits(uint32_t* keep_bits, int64_t base, uint32_t off, int t,
                                                uint32_t bits, bool valid, int64_t total_pieces) {
  constexpr int V = Store<T>::kVec;
  if constexpr (WORDS) {
    const uint32_t word = merge_mask_word<V>(bits, t);
    constexpr int kShare = 32 / V;
    if ((t & (kShare - 1)) == 0 && valid) *at_offset(keep_bits + base / kShare, off / kShare) = word;
  } else {
    uint8_t* kb = reinterpret_cast<uint8_t*>(keep_bits);
    uint32_t byte = bits;
    int64_t bi = base + off;  // byte index
    bool writer = valid;
    if constexpr (V == 4) {
      byte = bits << (4 * (t & 1));
      byte |= dpp_u32<kDppXor1>(byte);
      bi >>= 1;
      writer = valid && (t & 1) == 0;
    }
    if (writer) {
      kb[bi] = static_cast<uint8_t>(byte);
      const int64_t last = (V == 4 ? total_pieces >> 1 : total_pieces) - 1;
      if (bi == last) {
        for (int64_t b = bi + 1; (b & 3) != 0; ++b) kb[b] = 0;  // rest of the last word
      }
    }
  }
}

// Mask bits of piece base + off (base the same for the whole wave) as read by backward.
template <typename T, bool WORDS>
__device__ __forceinline__ uint32_t load_keep_bits(const uint32_t* keep_bits, int64_t base,
                                                   uint32_t off) {
  constexpr int V = Store<T>::kVec;
  if constexpr (WORDS) {  // base is a multiple of the pieces per word
    constexpr int kShare = 32 / V;
    return (*at_offset(keep_bits + base / kShare, off / kShare) >>
            (V * static_cast<int>(off & (kShare - 1)))) &
           ((1u << V) - 1u);
  } else {  // base is a multiple of the pieces per byte
    const uint8_t* kb = reinterpret_cast<const uint8_t*>(keep_bits);
    if constexpr (V == 8) return *at_offset(kb + base, off);
    return (*at_offset(kb + (base >> 1), off >> 1) >> (4 * static_cast<int>(off & 1))) & 0xFu;
  }
}

// ---- rows of any length ("ragged": Sk % 8 != 0) --------------------------------------------
// The pieces of a row (piece_col, piece_dup) do not line up with the generator's groups of 8
// elements, nor rows with mask words: the row's keep bytes, one per group, go through LDS, from
// where a lane takes the 8-bit window that starts at its piece.  One generator call per 8 elements,
// as on the aligned path.
// Measured, forward + backward: bfloat16 16x16x333x333 under a padding mask 198 us element by element,
// 84 us this way (aligned rows of 336 elements: 76); 8x12x1001x1001 557 -> 240 us (regen).
// Rows shorter than a piece (SHORT: only the kernels with the fewest lanes per row take them) are
// read and written element by element; `fill` stands for the rest of the piece.
template <typename T, bool RAG, bool SHORT>
__device__ __forceinline__ u32x4 load_row_piece(const T* p, int Sk, u32x4 fill) {
  constexpr int V = Store<T>::kVec;
  if constexpr (SHORT) {
    if (Sk < V) {
      float v[V];
      Store<T>::unpack(fill, v);
#pragma unroll
      for (int k = 0; k < V; ++k)
        if (k < Sk) v[k] = Store<T>::load1(p + k);
      return Store<T>::pack(v);
    }
  }
  return ldg_piece<RAG>(p);
}
template <typename T, bool RAG, bool SHORT>
__device__ __forceinline__ void store_row_piece(T* p, int Sk, u32x4 w) {
  constexpr int V = Store<T>::kVec;
  if constexpr (SHORT) {
    if (Sk < V) {
      float v[V];
      Store<T>::unpack(w, v);
#pragma unroll
      for (int k = 0; k < V; ++k)
        if (k < Sk) Store<T>::store1(p + k, v[k]);
      return;
    }
  }
  stg_piece<RAG>(p, w);
}
constexpr bool takes_short_rows(bool ragged, int lanes, int vec) { return ragged && lanes * vec == 32; }
// Keep bytes of a row of up to `elements` elements, whatever its alignment, and one more that a
// window may touch.
constexpr int keep_row_bytes(int elements) { return (elements + 7 + 7) / 8 + 2; }

// Draws the keep bytes of the row that starts at element base + off (base the same for the whole
// wave) into `row` (LDS) and, if keep_bits is
// given, stores those of the groups that begin in this row: every byte of the mask has one
// writer.  n: elements of the whole tensor; the last group's bits beyond it are 0, and so is the
// rest of the last word.
template <int LANES>
__device__ __forceinline__ void draw_row_keep(uint8_t* row, int64_t base, uint32_t off, int Sk, int t,
                                              const RngArgs& rng, uint32_t* keep_bits, int64_t n) {
  const int64_t b0 = base >> 3;                                    // the same for the whole wave
  const uint32_t start = static_cast<uint32_t>(base & 7) + off;    // element of the row, from b0
  const uint32_t goff = start >> 3;
  const int64_t g0 = b0 + goff;
  const int h = static_cast<int>(start & 7);
  const int groups = (h + Sk + 7) >> 3;
  for (int b = t; b < groups; b += LANES) {
    const uint32_t byte = keep_byte(static_cast<uint64_t>(b0), goff + b, rng);
    row[b] = static_cast<uint8_t>(byte);
    if (keep_bits && (b > 0 || h == 0)) {
      uint8_t* kb = reinterpret_cast<uint8_t*>(keep_bits) + g0 + b;
      const int64_t left = n - (g0 + b) * 8;
      if (left > 8) {
        *kb = static_cast<uint8_t>(byte);
      } else {  // the last group of the tensor
        *kb = static_cast<uint8_t>(byte & ((1u << left) - 1u));
        for (int64_t i = g0 + b + 1; (i & 3) != 0; ++i) *++kb = 0;
      }
    }
  }
}
// Keep bits of the piece that starts `r` elements after the first group of the row.
template <int V>
__device__ __forceinline__ uint32_t row_keep_window(const uint8_t* row, int r) {
  const int b = r >> 3;
  const uint32_t w = row[b] | (static_cast<uint32_t>(row[b + 1]) << 8);
  return (w >> (r & 7)) & ((1u << V) - 1u);
}
// The same from the stored mask: bits e .. e + V - 1, by one two-byte load that stays inside the
// mask's ceil(n / 32) words.
template <int V>
__device__ __forceinline__ uint32_t mask_window(const uint32_t* keep_bits, int64_t e, int64_t n) {
  typedef uint16_t u16_any __attribute__((aligned(1)));
  const int64_t last = ((n + 31) >> 5) * 4 - 2;
  const int64_t b = min(e >> 3, last);
  const uint32_t w =
      *reinterpret_cast<const u16_any*>(reinterpret_cast<const uint8_t*>(keep_bits) + b);
  return (w >> static_cast<int>(e - b * 8)) & ((1u << V) - 1u);
}

// How the keep bits of a row meet the mask: whole words (Sk % 32 == 0), whole bytes (Sk % 8 == 0),
// or anyhow (ragged rows).
enum MaskLayout { kWords, kBytes, kRagged };

// Work unit = one "row set": kGroups*R consecutive query rows of one [Sq, Sk] slice, where
// kGroups = kThreads/LANES lane groups each own R rows (rows base + r*kGroups + g) and CH
// 16-byte pieces per row (piece c of lane t = c*LANES + t).  All R rows of a group are fetched
// before any arithmetic: short rows would otherwise leave one 16-byte load per lane in
// flight, too little to cover the memory latency at 32 waves per compute unit.  Every row
// set has its own workgroup and the grid sweeps memory front to back (the launch cap splits it into
// several launches): a loop over row sets would keep lane addresses and round keys live across it,
// more registers than there are, and cost a wave that owns a single row more than the row.
// The forward is bound by the vector ALU while rows are short: bfloat16 16x16x336x336 runs at 1300
// cycles per row and SIMD, of which Philox takes a third.  Hence the division by multiplication, scalar
// base addresses with 32-bit lane offsets, packed 16-bit keep decisions and VALU lane swaps.
// LANES = 128 or 256 spreads a long row over 2 or 4 waves: the pieces per lane, and with them
// the registers per lane, stay small enough for many resident waves (a 3072-element bfloat16
// row on one wave needs over 200 registers per lane, which leaves 2 waves per SIMD).
template <typename T, int LANES, int CH, int R, MaskLayout MASK, int THREADS>
__global__ __launch_bounds__(THREADS) void attn_fwd_kernel(
    const T* scores, const int32_t* __restrict__ key_len, int causal, T* probs,
    T* __restrict__ out, uint32_t* __restrict__ keep_bits, int slices, int Sq, int Sk, float scale,
    RngArgs rng, FastDiv sets_per_slice, FastDiv heads, uint32_t first_set) {
  static_assert(THREADS % LANES == 0 && THREADS % kWave == 0, "whole lane groups, whole waves");
  constexpr bool kOneWave = butterfly_lanes(LANES) == LANES;  // a row inside one wave: no barriers
  constexpr int kGroups = THREADS / LANES;
  constexpr int V = Store<T>::kVec;
  int g = threadIdx.x / LANES;
  if constexpr (LANES % kWave == 0) g = __builtin_amdgcn_readfirstlane(g);  // row math stays scalar
  const int t = threadIdx.x % LANES;
  constexpr bool RAG = MASK == kRagged;
  constexpr bool SHORT = takes_short_rows(RAG, LANES, V);
  const int pieces = RAG ? (Sk + V - 1) / V : Sk / V;
  const int64_t total_pieces = static_cast<int64_t>(slices) * Sq * pieces;
  __shared__ float red[2][kOneWave ? 1 : THREADS / butterfly_lanes(LANES)];
  static_assert(kOneWave || R == 1, "rows over several waves: one row per group");
  static_assert(!RAG || R == 1, "ragged rows: one row per group");
  __shared__ uint8_t keep_lds[RAG ? kGroups : 1][RAG ? keep_row_bytes(LANES * CH * V) : 1];

  const uint32_t set = first_set + blockIdx.x;
  const uint32_t slice = sets_per_slice.divide(set);
  const int set0 = static_cast<int>(set - slice * sets_per_slice.d) * (kGroups * R);
  const int key_limit = key_len ? min(max(key_len[heads.divide(slice)], 0), Sk) : Sk;
  // The set's first row is the workgroup's, what a lane adds to it fits 32 bits: addresses are a
  // scalar base and a 32-bit offset.
  const int64_t base = row_offset(slice * static_cast<uint32_t>(Sq) + set0, Sk);
  const T* const s_base = scores + base;
  // limit = number of leading columns of the row that take part in the softmax; -1: no row
  int limit[R];
  Raw<T> raw[R][CH];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = set0 + g + r * kGroups;
    limit[r] = (i < Sq) ? row_limit(i, key_limit, causal, Sq, Sk) : -1;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int col0 = piece_col<RAG, V>(c * LANES + t, pieces, Sk);
      if constexpr (CH == 1) raw[r][c].a = Store<T>::neg_inf_piece();  // see below
      if (col0 < limit[r])
        raw[r][c].a = load_row_piece<T, RAG, SHORT>(
            at_offset(s_base, (g + r * kGroups) * Sk + col0), Sk, Store<T>::neg_inf_piece());
    }
  }
  uint8_t* const keep_row = keep_lds[RAG ? g : 0];
  if constexpr (RAG) {  // while the loads are under way
    if (limit[0] >= 0)
      draw_row_keep<LANES>(keep_row, base, g * Sk, Sk, t, rng, keep_bits,
                           static_cast<int64_t>(slices) * Sq * Sk);
    if constexpr (kOneWave) wave_lds_fence();  // else the reductions' barriers order it
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    // no row: uniform over the lane group; a group of several waves walks on (no loads, no
    // stores) because the reductions below hold workgroup barriers
    const bool live = limit[r] >= 0;
    if (kOneWave && !live) continue;
    const uint32_t row_off = static_cast<uint32_t>(g + r * kGroups) * Sk;  // elements from base
    float v[CH][V];
    float mx = -INFINITY;
    // One piece per lane: the lanes of a masked piece cannot save time by idling (their wave
    // runs on for the others), so a piece that was not loaded holds -inf and goes through the
    // same straight-line code, which gives 0 for it.  Several pieces per lane: a masked piece
    // is skipped, which for a causal mask spares whole waves half of their work.
    constexpr bool kSkip = CH > 1;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int col0 = piece_col<RAG, V>(c * LANES + t, pieces, Sk);
      if (!kSkip || col0 < limit[r]) {
        raw[r][c].unpack(v[c]);
        if (col0 < limit[r] && col0 + V > limit[r]) {  // the piece the limit falls into
#pragma unroll
          for (int k = 0; k < V; ++k) v[c][k] = (col0 + k < limit[r]) ? v[c][k] : -INFINITY;
        }
#pragma unroll
        for (int k = 0; k < V; k += 2) mx = fmaxf(fmaxf(mx, v[c][k]), v[c][k + 1]);  // v_max3
      }
    }
    mx = row_reduce<LANES, true>(mx, red[0]);
    const float shift = (mx == -INFINITY) ? 0.0f : mx * kLog2e;
    float sum = 0.0f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int col0 = piece_col<RAG, V>(c * LANES + t, pieces, Sk);
      const int dup = piece_dup<RAG, V>(c * LANES + t, pieces, Sk);
      if (!kSkip || col0 < limit[r]) {
#pragma unroll
        for (int k = 0; k < V; ++k) {
          const float e = __builtin_amdgcn_exp2f(fmaf(v[c][k], kLog2e, -shift));
          v[c][k] = e;
          sum += (RAG && k < dup) ? 0.0f : e;
        }
      } else {  // masked, or padding beyond the row
#pragma unroll
        for (int k = 0; k < V; ++k) v[c][k] = 0.0f;
      }
    }
    sum = row_reduce<LANES, false>(sum, red[1]);
    // 1 / sum by the hardware estimate; ragged rows add a Newton step, which rounds it like a division
    // (16x16x333x333 bf16 forward + backward: 87.6 us without it, 87.7 with it)
    float est = __builtin_amdgcn_rcpf(sum);
    if constexpr (RAG) est = fmaf(fmaf(-sum, est, 1.0f), est, est);
    const float rinv = (sum > 0.0f) ? est : 0.0f;
    const uint64_t group0 = static_cast<uint64_t>(base) >> 3;  // aligned rows: whole groups
    constexpr bool kFlags = !RAG && V == 8;  // keep decisions as flag words
    uint32_t bits[CH];
    if constexpr (!RAG && !kFlags)
      lane_keep_bits<T, LANES, CH>(group0, row_off / V, t, rng, bits);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int pc = c * LANES + t;
      const bool valid = live && pc < pieces;
      const int col0 = piece_col<RAG, V>(pc, pieces, Sk);
      if constexpr (kFlags) bits[c] = 0xFFu;
      if (valid) {
        if constexpr (RAG)
          bits[c] = row_keep_window<V>(
              keep_row, static_cast<int>((static_cast<uint32_t>(base) + row_off) & 7) + col0);
        float p8[V], o8[V];
#pragma unroll
        for (int k = 0; k < V; ++k) p8[k] = v[c][k] * rinv;
        // round P once, into the words that are stored; Out is computed from the stored P
        const u32x4 pw = Store<T>::pack(p8);
        Store<T>::unpack(pw, p8);
        store_row_piece<T, RAG, SHORT>(at_offset(probs + base, row_off + col0), Sk, pw);
#pragma unroll
        for (int k = 0; k < V; ++k) o8[k] = p8[k] * scale;
        u32x4 ow = Store<T>::pack(o8);
        if constexpr (kFlags) {
          if (rng.t16 < 65536u) {  // else nothing is dropped
            uint32_t w[4], flags[4];
            draw_group(group0, row_off / V + pc, rng, w);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              flags[j] = keep_flags(w[j], rng.t16 * 0x00010001u);
              ow[j] &= flags_to_mask(flags[j]);
            }
            bits[c] = flags_to_byte(flags);
          }
        } else {
          ow = apply_keep<T>(ow, bits[c]);
        }
        if (out) store_row_piece<T, RAG, SHORT>(at_offset(out + base, row_off + col0), Sk, ow);
      }
      if constexpr (!RAG)
        store_keep_bits<T, MASK == kWords>(keep_bits, base / V, row_off / V + pc, t,
                                           valid ? bits[c] : 0u, valid, total_pieces);
    }
  }
}

// Keep bits of one piece from a mask kept the way the paper's implementation keeps it, one
// byte per element (Sec. 3.3; any non-zero byte means kept): one 4-byte (float32 piece) or
// 8-byte (bfloat16 piece) load per lane.  Per 32-bit word: fold each byte's bits onto its bit 0,
// then gather the four bit-0s by one multiply (the partial products land on distinct bits).
__device__ __forceinline__ uint32_t nonzero_bytes_to_bits(uint32_t w) {
  w |= w >> 4;
  w |= w >> 2;
  w |= w >> 1;
  w &= 0x01010101u;
  return (w * 0x01020408u) >> 24;  // byte i -> bit i
}
template <typename T, bool SHORT>
__device__ __forceinline__ uint32_t load_keep_bools(const uint8_t* p, int Sk) {
  if constexpr (SHORT) {
    if (Sk < Store<T>::kVec) {
      uint32_t bits = 0;
      for (int k = 0; k < Sk; ++k) bits |= (p[k] != 0 ? 1u : 0u) << k;
      return bits;
    }
  }
  // at any byte address (ragged rows); aligned ones take the same instructions
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32_any __attribute__((aligned(1)));
  typedef u32x2 u32x2_any __attribute__((aligned(1)));
  if constexpr (Store<T>::kVec == 4) {
    return nonzero_bytes_to_bits(
        __builtin_nontemporal_load(reinterpret_cast<const u32_any*>(p)));
  } else {
    const u32x2 w = __builtin_nontemporal_load(reinterpret_cast<const u32x2_any*>(p));
    return nonzero_bytes_to_bits(w.x) | (nonzero_bytes_to_bits(w.y) << 4);
  }
}

// MASK says where backward takes the keep bits from: the stored bit mask read as whole words
// (Sk % 32 == 0) or as bytes, the generator (no mask is read; Sec. 3.3 weighs storing the
// mask against drawing it again), or a mask of one byte per element (keep_bits then points to
// bytes).
enum MaskSource { kMaskWords, kMaskBytes, kMaskRegen, kMaskBools };

// Work unit = one row per lane group; like the forward, a scalar base address and 32-bit offsets.
template <typename T, int LANES, int CH, MaskSource MASK, bool RAG, int THREADS>
__global__ __launch_bounds__(THREADS) void attn_bwd_kernel(
    const T* dout, const T* __restrict__ probs, const uint32_t* __restrict__ keep_bits,
    T* dscores, T* __restrict__ out_re, uint32_t rows, int Sk, float scale, RngArgs rng,
    uint32_t first_set) {
  static_assert(THREADS % LANES == 0 && THREADS % kWave == 0, "whole lane groups, whole waves");
  static_assert(!RAG || MASK != kMaskWords, "ragged rows: no whole words");
  constexpr bool kOneWave = butterfly_lanes(LANES) == LANES;
  constexpr int kGroups = THREADS / LANES;
  constexpr int V = Store<T>::kVec;
  int g = threadIdx.x / LANES;
  if constexpr (LANES % kWave == 0) g = __builtin_amdgcn_readfirstlane(g);  // row math stays scalar
  const int t = threadIdx.x % LANES;
  constexpr bool SHORT = takes_short_rows(RAG, LANES, V);
  const int pieces = RAG ? (Sk + V - 1) / V : Sk / V;
  __shared__ float red[kOneWave ? 1 : THREADS / butterfly_lanes(LANES)];
  constexpr bool kDraw = RAG && MASK == kMaskRegen;  // the keep bytes of the rows, drawn into LDS
  __shared__ uint8_t keep_lds[kDraw ? kGroups : 1][kDraw ? keep_row_bytes(LANES * CH * V) : 1];

  const uint32_t row = (first_set + blockIdx.x) * kGroups;  // the workgroup's first
  const int64_t base = row_offset(row, Sk);
  const uint32_t row_off = static_cast<uint32_t>(g) * Sk;   // elements from base
  // no row: uniform over the lane group; a group of several waves walks on (the reduction
  // holds a workgroup barrier) with zeros and stores nothing
  const bool live = static_cast<uint32_t>(g) < rows - row;
  Raw<T> rdo[CH], rp[CH];
  uint32_t bits[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int pc = c * LANES + t;
    bits[c] = 0;
    if (live && pc < pieces) {
      const uint32_t off = row_off + piece_col<RAG, V>(pc, pieces, Sk);
      rdo[c].a = load_row_piece<T, RAG, SHORT>(at_offset(dout + base, off), Sk, u32x4{0u, 0u, 0u, 0u});
      rp[c].a = load_row_piece<T, RAG, SHORT>(at_offset(probs + base, off), Sk, u32x4{0u, 0u, 0u, 0u});
      if constexpr (MASK == kMaskBools)
        bits[c] = load_keep_bools<T, SHORT>(
            at_offset(reinterpret_cast<const uint8_t*>(keep_bits) + base, off), Sk);
      else if constexpr (RAG && MASK != kMaskRegen)
        bits[c] = mask_window<V>(keep_bits, base + off, static_cast<int64_t>(rows) * Sk);
      else if constexpr (MASK != kMaskRegen)
        bits[c] = load_keep_bits<T, MASK == kMaskWords>(keep_bits, base / V, row_off / V + pc);
    }
  }
  if constexpr (kDraw) {
    uint8_t* const keep_row = keep_lds[g];
    if (live) draw_row_keep<LANES>(keep_row, base, row_off, Sk, t, rng, nullptr, 0);
    if constexpr (kOneWave) wave_lds_fence();
    else lds_barrier();
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int pc = c * LANES + t;
      if (live && pc < pieces)
        bits[c] = row_keep_window<V>(
            keep_row, static_cast<int>((static_cast<uint32_t>(base) + row_off) & 7) +
                          piece_col<RAG, V>(pc, pieces, Sk));
    }
  } else if constexpr (MASK == kMaskRegen) {  // every lane takes part: lane pairs share draws
    lane_keep_bits<T, LANES, CH>(static_cast<uint64_t>(base) >> 3, row_off / V, t, rng, bits);
  }
  if (kOneWave && !live) return;
  float dp[CH][V], pr[CH][V];
  float dot = 0.0f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int pc = c * LANES + t;
    const int dup = piece_dup<RAG, V>(pc, pieces, Sk);
    if (live && pc < pieces) {
      Store<T>::unpack(apply_keep<T>(rdo[c].a, bits[c]), dp[c]);  // dropped: dP = 0
      rp[c].unpack(pr[c]);
    } else {
#pragma unroll
      for (int k = 0; k < V; ++k) dp[c][k] = pr[c][k] = 0.0f;
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
      dp[c][k] *= scale;
      if (!RAG || k >= dup) dot = fmaf(dp[c][k], pr[c][k], dot);
    }
  }
  dot = row_reduce<LANES, false>(dot, red);
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int pc = c * LANES + t;
    if (live && pc < pieces) {
      const uint32_t off = row_off + piece_col<RAG, V>(pc, pieces, Sk);
      float ds[V];
#pragma unroll
      for (int k = 0; k < V; ++k) ds[k] = pr[c][k] * (dp[c][k] - dot);
      store_row_piece<T, RAG, SHORT>(at_offset(dscores + base, off), Sk, Store<T>::pack(ds));
      if (out_re) {
        float o8[V];
#pragma unroll
        for (int k = 0; k < V; ++k) o8[k] = pr[c][k] * scale;
        store_row_piece<T, RAG, SHORT>(at_offset(out_re + base, off), Sk,
                                       apply_keep<T>(Store<T>::pack(o8), bits[c]));
      }
    }
  }
}

// ---- any Sk: one wave per row, scalar accesses, the row re-read from cache per pass --------

// Keep bits of a block of up to 448 consecutive elements (7 chunks of 64: at most 57 groups of 8
// whatever the block's alignment): each lane draws one group, and the lanes fetch the byte of
// their element's group from the lane that drew it, one generator call per 8 elements instead
// of one per element.  Every lane of the wave has to make both calls.
constexpr int kDrawBlock = 7 * kWave;
struct KeepBlock {
  uint32_t byte;
  int64_t group0;
  __device__ __forceinline__ void draw(int64_t e_block, int lane, const RngArgs& rng) {
    group0 = e_block >> 3;
    byte = keep_byte(static_cast<uint64_t>(group0), lane, rng);
  }
  __device__ __forceinline__ bool kept(int64_t e) const {
    return (__shfl(byte, static_cast<int>((e >> 3) - group0), kWave) >> (e & 7)) & 1u;
  }
};

template <typename T>
__global__ __launch_bounds__(kThreads) void attn_fwd_generic_kernel(
    const T* scores, const int32_t* __restrict__ key_len, int causal, T* probs,
    T* __restrict__ out, int64_t rows, int64_t rows_per_batch, int Sq, int Sk, float scale,
    RngArgs rng) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  constexpr int kWaves = kThreads / kWave;
  for (int64_t row = static_cast<int64_t>(blockIdx.x) * kWaves + wave; row < rows;
       row += static_cast<int64_t>(gridDim.x) * kWaves) {
    const int key_limit = key_len ? min(max(key_len[row / rows_per_batch], 0), Sk) : Sk;
    const int limit = row_limit(static_cast<int>(row % Sq), key_limit, causal, Sq, Sk);
    const T* sr = scores + row * Sk;
    float mx = -INFINITY;
    for (int j = lane; j < limit; j += kWave) mx = fmaxf(mx, Store<T>::load1(sr + j));
    mx = group_max<kWave>(mx);
    const float shift = (mx == -INFINITY) ? 0.0f : mx * kLog2e;
    float sum = 0.0f;
    for (int j = lane; j < limit; j += kWave)
      sum += __builtin_amdgcn_exp2f(fmaf(Store<T>::load1(sr + j), kLog2e, -shift));
    sum = group_sum<kWave>(sum);
    const float rinv = (sum > 0.0f) ? 1.0f / sum : 0.0f;
    for (int b0 = 0; b0 < Sk; b0 += kDrawBlock) {  // uniform over the wave
      KeepBlock keep;
      if (out) keep.draw(row * Sk + b0, lane, rng);
      for (int c0 = b0; c0 < min(b0 + kDrawBlock, Sk); c0 += kWave) {
        const int j = c0 + lane;
        const int64_t e = row * Sk + j;
        const bool kb = out ? keep.kept(e) : false;
        if (j < Sk) {
          float p = 0.0f;
          if (j < limit)
            p = Store<T>::round(
                __builtin_amdgcn_exp2f(fmaf(Store<T>::load1(sr + j), kLog2e, -shift)) * rinv);
          Store<T>::store1(probs + e, p);
          if (out) Store<T>::store1(out + e, kb ? p * scale : 0.0f);
        }
      }
    }
  }
}

// Mask words for shapes whose rows do not end on chunk boundaries: one thread per word.
__global__ __launch_bounds__(kThreads) void keep_words_kernel(uint32_t* __restrict__ keep_bits,
                                                             int64_t n, RngArgs rng) {
  const int64_t words = (n + 31) >> 5;
  for (int64_t w = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; w < words;
       w += static_cast<int64_t>(gridDim.x) * kThreads) {
    uint32_t word = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) word |= keep_byte(static_cast<uint64_t>(w) * 4, b, rng) << (8 * b);
    const int64_t left = n - w * 32;
    if (left < 32) word &= (1u << left) - 1u;
    keep_bits[w] = word;
  }
}

template <typename T, MaskSource MASK>
__global__ __launch_bounds__(kThreads) void attn_bwd_generic_kernel(
    const T* dout, const T* __restrict__ probs, const uint32_t* __restrict__ keep_bits,
    T* dscores, T* __restrict__ out_re, int64_t rows, int Sk, float scale, RngArgs rng) {
  auto stored = [&](int64_t e) -> bool {
    if constexpr (MASK == kMaskBools) return reinterpret_cast<const uint8_t*>(keep_bits)[e] != 0;
    else return (keep_bits[e >> 5] >> (e & 31)) & 1u;
  };
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  constexpr int kWaves = kThreads / kWave;
  for (int64_t row = static_cast<int64_t>(blockIdx.x) * kWaves + wave; row < rows;
       row += static_cast<int64_t>(gridDim.x) * kWaves) {
    float dot = 0.0f;
    for (int b0 = 0; b0 < Sk; b0 += kDrawBlock) {  // uniform over the wave
      KeepBlock keep;
      if constexpr (MASK == kMaskRegen) keep.draw(row * Sk + b0, lane, rng);
      for (int c0 = b0; c0 < min(b0 + kDrawBlock, Sk); c0 += kWave) {
        const int j = c0 + lane;
        const int64_t e = row * Sk + j;
        bool k = false;
        if constexpr (MASK == kMaskRegen) k = keep.kept(e);
        else if (j < Sk) k = stored(e);
        if (j < Sk) {
          const float dp = k ? Store<T>::load1(dout + e) * scale : 0.0f;
          dot = fmaf(dp, Store<T>::load1(probs + e), dot);
        }
      }
    }
    dot = group_sum<kWave>(dot);
    for (int b0 = 0; b0 < Sk; b0 += kDrawBlock) {
      KeepBlock keep;
      if constexpr (MASK == kMaskRegen) keep.draw(row * Sk + b0, lane, rng);
      for (int c0 = b0; c0 < min(b0 + kDrawBlock, Sk); c0 += kWave) {
        const int j = c0 + lane;
        const int64_t e = row * Sk + j;
        bool k = false;
        if constexpr (MASK == kMaskRegen) k = keep.kept(e);
        else if (j < Sk) k = stored(e);
        if (j < Sk) {
          const float p = Store<T>::load1(probs + e);
          const float dp = k ? Store<T>::load1(dout + e) * scale : 0.0f;
          Store<T>::store1(dscores + e, p * (dp - dot));
          if (out_re) Store<T>::store1(out_re + e, k ? p * scale : 0.0f);
        }
      }
    }
  }
}

constexpr int kMaxPieces = 1024;  // 4 per lane of 4 waves

constexpr int kRaggedMaxPieces = 4;  // per lane

// Rows of one piece per lane on a number of lanes that is no power of two (odd_shape()) lie across the waves
// of a workgroup, which takes as many rows as fill whole waves.
constexpr bool is_odd(int lanes) { return (lanes & (lanes - 1)) != 0; }
constexpr int odd_threads(int lanes) {
  const int low = lanes & -lanes;
  return lanes / low * (low > kWave ? low : kWave);
}

// Fewest lanes a workgroup may have: a row's, and two rows' where a forward row takes two waves.  One row /
// two rows per workgroup, us: 32x16x1024x1024 bf16 518-542 / 497-519 by buffers, 16x16x505x505 f32 142 / 135,
// 64x16x512x512 f32 506-545 / 516-528; 12x1024x1024 bf16 causal, on half the chip, 14.3 / 14.7.
constexpr int least_threads(int lanes, bool backward) {
  if (is_odd(lanes)) return odd_threads(lanes);
  return lanes <= kWave ? kWave : (backward ? lanes : 4 * kWave);
}
// Lanes per workgroup of the ragged rows and of those on an odd number of lanes, whatever the knob says.
constexpr int fixed_threads(int lanes, bool backward) {
  return lanes <= kWave && !is_odd(lanes) ? 2 * kWave : least_threads(lanes, backward);
}

struct Shape {
  int lanes;
  int ch;
};

// One piece per lane while the row fits in a wave (every access of a wave is then one
// contiguous run of 16-byte pieces), more pieces per lane for longer rows.  min_lanes: 4 for
// bfloat16, 8 for float32 (the lanes that share a mask word).  ch == 0: row too long.
constexpr Shape pick_shape(int pieces, int min_lanes) {
  int lanes = min_lanes;
  while (lanes < 64 && lanes < pieces) lanes <<= 1;
  const int need = (pieces + lanes - 1) / lanes;
  constexpr int allowed[] = {1, 2, 3, 4, 6, 8, 12, 16};
  for (int a : allowed)
    if (a >= need) return {lanes, lanes == 64 || a == 1 ? a : 0};
  return {0, 0};
}

// A row whose pieces per lane on one wave would exceed max_ch is spread over 2 or 4 waves (at
// most 4 pieces per lane there).
constexpr Shape pick_wide_shape(int pieces, int min_lanes, int max_ch) {
  const Shape one = pick_shape(pieces, min_lanes);
  if (one.lanes == kWave && (one.ch == 0 || one.ch > max_ch)) {
    for (int lanes = 2 * kWave; lanes <= kThreads; lanes *= 2) {
      const int need = (pieces + lanes - 1) / lanes;
      if (need <= max_ch || lanes == kThreads) {
        if (need <= 4) return {lanes, need};
        break;
      }
    }
  }
  return one;
}

// Shape for rows of Sk elements; ch == 0: too long for the register-resident kernels.
// Rows longer than a wave take as many waves as give a lane a single piece, while that leaves few
// lanes idle (an eighth of them at most forward, where the vector ALU counts, a quarter backward);
// longer ones take four waves.  One wave with several pieces per lane against this, us:
// 64x16x512x512 f32 547 -> 520 forward, 706 -> 695 backward; 8x12x1024x1024 bf16 causal backward
// 134 -> 129; 1x16x2048 bf16 forward 72 -> 68; 2x12x3072 bf16 causal forward 206 -> 202; with more idle
// lanes it loses (640 bf16 columns forward: 45 -> 53).  Ragged rows gain more (1001 f32: 363 -> 304
// both ways), but two waves of bfloat16 lose 5 % (901 columns: 143 -> 151).  Several short rows per
// wave with three pieces per lane lose a third wherever rows are not whole 128-byte lines.
// A causal forward (rows of whole groups) takes half the waves with two pieces per lane, since a lane skips
// only pieces of its own that are masked.  One piece / two pieces, us: bf16 2x12x1792x1792 83.5 / 70,
// 12x2048x2048 50 / 47, 5x16x896x896 66 / 61; f32 9x16x448x448 55.6 / 53.4, 2x16x1024x1024 61.3 / 60.6.
// The backward has one shape whatever its mask comes from: the same sums in the same order.
enum RowUse { kForward, kForwardCausal, kBackward };

// Lanes that are no power of two, where those would leave a quarter of the lanes idle or more: the vector ALU, which
// bounds the bfloat16 forward, works for idle lanes too, and the backward keeps fewer loads under way per wave.  The
// price is a workgroup barrier per row sum.  Power of two / this, us:
//  - 12 (bfloat16 only: 8 lanes share a float32 mask word), 24 and 48 lanes for 9..12, 17..24 and 33..48 pieces, both
//    ways: bf16 48x16x80x80 17.5 / 16.4, 32x16x150x150 38.9 / 34.3, 16x16x333x333 padded 84.5 / 75.2, 16x16x384x384 91.7 /
//    88.2; f32 32x16x96x96 26.7 / 25.8, 32x16x150x150 67.9 / 60.8;
//  - backward on 96 lanes for 65..96 pieces, bf16 8x16x520x520 55.3 / 49.4, 8x16x765x765 117 / 106, 8x16x768x768 99.6 /
//    99.0, f32 16x16x333x333 86.9 / 80.3; 160 for 129..160, bf16 2x16x1101x1101 63.2 / 55.1, 1280 70.9 / 69.0; 224
//    for 193..224 of bf16 ragged, 1701 148 / 131, not aligned, 1792 133.1 / 133.1, nor f32, 800 107 / 108.5; 320 for 257..320,
//    bf16 2x8x2100x2100 105 / 96, 2560 140.0 / 138.7; 384 for 321..352 of ragged rows, bf16 2700 166 / 159, f32
//    2x16x1401x1401 174 / 168;
//  - the bfloat16 forward without a causal mask, whose pieces a lane skips, on 96 lanes from 89 pieces, 8x16x744x744
//    89.8 / 79.1 (704 columns the same, 520 4 % slower).
// The same as a mean of the ratio over two dozen sizes of 0.3 to 38 M elements each, below 3 M / above, since every size
// at which the workgroups just exceed what is resident loses up to 17 % and others gain as much:
//  - taken: 12..48 lanes forward 0.83-1.00 / 0.87-0.94, backward 0.89-1.00 / 0.91-0.99; backward on 96 0.87-0.98 /
//    0.90-0.97, 160 0.81-1.00 / 0.89-0.98, 320 0.89-1.00 / 0.92-1.00, 224 0.94 / 0.92 with the mask stored, 1.00 / 1.02 drawn
//    again, 384 ragged 0.92 / 0.94 and 0.99 / 0.99; forward on 96 0.87-0.91 / 0.96-1.02;
//  - not taken: forward on 192 0.94 / 1.06-1.09 (2x4x1360x1360 1.26-1.29), 224 0.92-0.99 / 0.97-1.04 (2x1728x1728 1.20-1.23),
//    160, 320 and 384 (1200 padded 47.6 / 56.1 us) and of float32 from 96 up (4x16x600x600 47.4 / 51.1); backward on 192,
//    float32 0.96 / 0.97 stored, 1.05-1.09 / 0.98 drawn again (up to 1.26), bf16 aligned 0.97 / 0.98 and 1.02 / 1.01 (up to 1.16),
//    ragged 1501 106 / 115 us; aligned backward on 384 1.01 and 1.03 (3072, full, 195.5 / 200.5 us).
constexpr Shape odd_shape(int p, bool ragged, int vec, RowUse use) {
  const bool bf16 = vec == 8;
  if (p > 8 && p <= 12 && bf16) return {12, 1};
  if (p > 16 && p <= 24) return {24, 1};
  if (p > 32 && p <= 48) return {48, 1};
  if (use == kBackward) {
    if (p > 64 && p <= 96) return {96, 1};
    if (p > 128 && p <= 160) return {160, 1};
    if (p > 192 && p <= 224 && bf16 && ragged) return {224, 1};
    if (p > 256 && p <= 320) return {320, 1};
    if (p > 320 && p <= 352 && ragged) return {384, 1};
  } else if (use == kForward && bf16) {
    if (p > 88 && p <= 96) return {96, 1};
  }
  return {0, 0};
}
constexpr Shape shape_of(int p, bool ragged, int vec, int max_ch, RowUse use) {
  const bool backward = use == kBackward;
  if (ragged || max_ch <= kRaggedMaxPieces) {
    const Shape odd = odd_shape(p, ragged, vec, use);
    if (odd.ch != 0) return odd;
    const int wide = p <= 2 * kWave ? 2 * kWave : kThreads;
    const bool two_ragged_bf16 = ragged && vec == 8 && wide == 2 * kWave;
    if (p > kWave && p <= kThreads && p * 8 >= wide * (backward ? 6 : 7) && !two_ragged_bf16)
      return use == kForwardCausal && !ragged && max_ch >= 2 ? Shape{wide / 2, 2} : Shape{wide, 1};
    if (p > kThreads) return {kThreads, (p + kThreads - 1) / kThreads};
  }
  return pick_wide_shape(p, 32 / vec, ragged ? kRaggedMaxPieces : max_ch);
}
Shape row_shape(int64_t Sk, int vec, int max_ch, RowUse use) {
  const int64_t pieces = (Sk + vec - 1) / vec;
  if (pieces > kMaxPieces) return {0, 0};
  return shape_of(static_cast<int>(pieces), Sk % 8 != 0, vec, max_ch, use);
}
// Whether rows come to a shape: all that there are kernels for.  (Aligned rows on a power of two come to any from 32
// elements, by the knobs.)
constexpr bool has_kernel(int lanes, int ch, int vec, bool ragged, bool backward) {
  if (!ragged && !is_odd(lanes)) return lanes * vec >= 32;
  for (int p = 1; p <= kMaxPieces; ++p) {
    for (RowUse use : {kForward, kForwardCausal, kBackward}) {
      const Shape sh = shape_of(p, ragged, vec, 1, use);
      if (sh.lanes == lanes && sh.ch == ch && (use == kBackward) == backward) return true;
    }
  }
  return false;
}
constexpr bool ragged_shapes_exist(int vec) {
  for (int p = 1; p <= kMaxPieces; ++p) {
    for (RowUse use : {kForward, kForwardCausal, kBackward}) {
      if (shape_of(p, true, vec, 1, use).ch == 0) return false;
    }
  }
  return true;
}
static_assert(ragged_shapes_exist(4) && ragged_shapes_exist(8), "float32 and bfloat16");

// Dynamic LDS that no kernel reads: it keeps the waves that are resident on a compute unit to `waves`
// (rounded up to whole workgroups; 0 and 26 or more: as many as fit, which is as good).
constexpr int kLdsPerCu = 160 * 1024;
size_t residency_lds_bytes(int waves, int threads) {
  const int groups = (waves + threads / kWave - 1) / (threads / kWave);
  if (waves == 0 || waves >= 26 || groups > 12) return 0;
  return kLdsPerCu / groups / 256 * 256 - 1280;  // less the static LDS; one more would not fit
}
int pieces_per_wave(const Shape& sh, int pieces) { return std::max(1, pieces * kWave / sh.lanes); }

// Resident waves of the backward.  It streams two tensors in and two out, and the more waves have loads
// under way, the worse the memory system does, until they are too few.  All waves / this, us:
//  - one piece per lane, 18 waves where the lanes are full: 8x12x1024x1024 bf16 causal 130 / 126, 16x16x512x512
//    bf16 88 / 85, 64x16x256x256 f32 175 / 173 (64x16x512x512 f32: as much faster as slower, by buffers), and
//    20 or 24 at three quarters or five eighths: 25x16x384x384 bf16 80.5 / 76.7, 36x16x320x320 79.5 / 77.5;
//  - several pieces, 12 waves: 16x4096x4096 bf16 373 / 350, 16x2048x2048 f32 causal 188 / 172, 8x3072x3072 f32
//    210 / 196.  More on four waves with idle lanes.  Two pieces: 16, or 20 with a stored mask, 2x12 causal
//    slices of 2304, 2816 and 3072 bf16 columns 169, 250, 304 / 166, 246, 294 (12: 194, 271, 310), with the bits
//    drawn again 168, 250, 299 / 162, 242, 289 (the last at 12).  Three pieces: 16, 4x5120x5120 bf16 141.5 / 137 (12: 140.5),
//    and with the bits drawn again all, 4x6144x6144 bf16 199 (12: 207);
//  - ragged rows of one piece pay at 23 waves what aligned ones gain: 23x16x333x333 bf16 62.3 / 63.7.
int bwd_waves(const Shape& sh, int pieces, bool regen, bool ragged) {
  const int per_wave = pieces_per_wave(sh, pieces);
  if (!ragged) {
    if (sh.ch == 1) return std::max(18, (15 * kWave + per_wave - 1) / per_wave);
    if (sh.lanes == kThreads && sh.ch == 2)
      return per_wave <= 88 && !regen ? 20 : (per_wave < 96 || (per_wave == 96 && !regen) ? 16 : 12);
    if (sh.lanes == kThreads && sh.ch == 3) return regen ? 0 : (per_wave <= 160 ? 16 : 12);
  }
  return std::max(12, (18 * kWave + per_wave - 1) / per_wave);
}

// Dynamic LDS of the float32 forward (one tensor in, two out), whose vector work leaves room for the
// same.  All waves / this, us: one piece per lane of one wave at 28 waves, 64x16x256x256 132 / 129; one wave of
// three pieces at 20, 5x16x640x640 causal 59 / 59.5 and padded 64.7 / 64.4 (12: 62.8, 66.4), of four at 12, 4x16x800x800
// 86 / 85, padded 82.3 / 80, causal 75 / 74 (8: 87.6, 87.3, 83.8).  Four waves: rows of which much is masked
// keep fewer loads under way per wave and want more of them.  Three pieces: 12 waves, 8x3072x3072 159 / 150;
// causal 20, 8x3072x3072 145 / 133, 12x2560x2560 136 / 138 (12: 134, 150).  Four pieces: 8 waves where the
// lanes are full, 8x4096x4096 284 / 268; 12 where they are not, 4x3200x3200 91 / 83 (8: 87), and causal,
// 4x4096x4096 135 / 122 (8: 125).
// The bfloat16 forward is bound by the vector ALU and wants all waves (3072 columns, causal: 201 us, 255
// at 16 waves).
size_t fwd_f32_lds_bytes(const Shape& sh, int pieces, int threads, bool causal, bool padded) {
  const bool one_wave = sh.lanes <= kWave;
  const int per_wave = pieces_per_wave(sh, pieces);
  if (sh.ch == 1 && one_wave && threads == 2 * kWave && pieces * 8 >= sh.lanes * 7)
    return 11 * 1024;  // 28 waves
  if (sh.ch == 3) return residency_lds_bytes(one_wave || causal ? 20 : 12, threads);
  if (sh.ch == 4)
    return residency_lds_bytes(one_wave || causal || per_wave <= (padded ? 240 : 224) ? 12 : 8, threads);
  return 0;
}

// Rows a lane group of the forward kernel fetches at once: 2 (if the knob allows) when a
// bfloat16 row is exactly one piece per lane of a whole wave, else 1.  Measured in steady state
// on rows of 128..1024 elements: 2 rows gain 5-7 % there (512 columns) and lose 3-9 % for
// shorter rows (several rows per wave already), for two pieces per lane and for float32;
// backward always takes 1.
int attn_rows(int ch, int lanes, int vec, int tuned) {
  return (vec == 8 && ch == 1 && lanes == kWave && tuned >= 2) ? 2 : 1;
}

// Lanes per workgroup of the register-resident kernels.  Small workgroups come and go
// independently, which the memory system rewards: against workgroups of four waves, two waves
// gain 2-8 % (forward at every size, backward on tensors from 2 GB up, never a loss); single
// waves do no better than two and lose 1-2 % in places.  So: two waves, and never fewer lanes
// than a row takes.
int group_threads(int lanes, bool backward) {
  if (is_odd(lanes)) return odd_threads(lanes);
  const int least = least_threads(lanes, backward);  // 64, 128 or 256
  int want = tune_get(kTuneAttnThreads);
  want = want >= 256 ? 256 : (want >= 128 ? 128 : kWave);
  return want > least ? want : least;
}

// Workgroups of the any-length kernels: one wave per row, rows beyond the cap in a loop.
int row_grid(int64_t rows, int blocks_per_cu) {
  const int64_t want = (rows + kThreads / kWave - 1) / (kThreads / kWave);
  const int64_t cap = most_groups(static_cast<int64_t>(compute_units()) * blocks_per_cu, kThreads);
  return static_cast<int>(std::max<int64_t>(1, std::min(want, cap)));
}

}  // namespace

// LAUNCH(lanes, pieces per lane); the rows per lane group come from attn_rows().
#define TEMPO_ATTN_DISPATCH(LAUNCH)                                                        \
  switch (sh.lanes * 100 + sh.ch) {                                                        \
    case 401: LAUNCH(4, 1); break;                                                         \
    case 801: LAUNCH(8, 1); break;                                                         \
    case 1201: LAUNCH(12, 1); break;                                                       \
    case 1601: LAUNCH(16, 1); break;                                                       \
    case 2401: LAUNCH(24, 1); break;                                                       \
    case 3201: LAUNCH(32, 1); break;                                                       \
    case 4801: LAUNCH(48, 1); break;                                                       \
    case 6401: LAUNCH(64, 1); break;                                                       \
    case 6402: LAUNCH(64, 2); break;                                                       \
    case 6403: LAUNCH(64, 3); break;                                                       \
    case 6404: LAUNCH(64, 4); break;                                                       \
    case 6406: LAUNCH(64, 6); break;                                                       \
    case 6408: LAUNCH(64, 8); break;                                                       \
    case 6412: LAUNCH(64, 12); break;                                                      \
    case 6416: LAUNCH(64, 16); break;                                                      \
    default: return TEMPO_ERR_UNSUPPORTED;                                                 \
  }

#define TEMPO_ATTN_WIDE_DISPATCH(LAUNCH)                                                   \
  switch (sh.lanes * 100 + sh.ch) {                                                        \
    case 9601: LAUNCH(96, 1); break;                                                       \
    case 12801: LAUNCH(128, 1); break;                                                     \
    case 12802: LAUNCH(128, 2); break;                                                     \
    case 12803: LAUNCH(128, 3); break;                                                     \
    case 12804: LAUNCH(128, 4); break;                                                     \
    case 16001: LAUNCH(160, 1); break;                                                     \
    case 22401: LAUNCH(224, 1); break;                                                     \
    case 25601: LAUNCH(256, 1); break;                                                     \
    case 25602: LAUNCH(256, 2); break;                                                     \
    case 25603: LAUNCH(256, 3); break;                                                     \
    case 25604: LAUNCH(256, 4); break;                                                     \
    case 32001: LAUNCH(320, 1); break;                                                     \
    case 38401: LAUNCH(384, 1); break;                                                     \
    default: return TEMPO_ERR_UNSUPPORTED;                                                 \
  }

// Calls f with the workgroup size as a compile-time constant: 64, 128 or 256, at least
// least_threads; with FIXED and for odd numbers of lanes the only size.
template <int L, bool BACKWARD, bool FIXED, typename F>
static void with_threads(int threads, F&& f) {
  using std::integral_constant;
  if constexpr (FIXED || is_odd(L)) {
    return f(integral_constant<int, fixed_threads(L, BACKWARD)>{});
  } else {
    constexpr int least = least_threads(L, BACKWARD);
    if constexpr (least <= 64) {
      if (threads == 64) return f(integral_constant<int, 64>{});
    }
    if constexpr (least <= 128) {
      if (threads == 128) return f(integral_constant<int, 128>{});
    }
    f(integral_constant<int, 256>{});
  }
}

template <typename T, int L, int C>
static void attn_fwd_go(int rr, MaskLayout layout, int threads, size_t lds, uint32_t first_set, uint32_t sets, hipStream_t st,
                        const void* scores, const int32_t* key_len, int causal, void* probs,
                        void* out, uint32_t* keep_bits, int slices, const FastDiv& heads,
                        const FastDiv& sets_per_slice, int64_t Sq, int64_t Sk, float scale,
                        const RngArgs& rng) {
  auto go = [&](auto rows, auto w) {
    with_threads<L, false, decltype(w)::value == kRagged>(threads, [&](auto th) {
      constexpr int TH = decltype(th)::value;
      hipLaunchKernelGGL(
          (attn_fwd_kernel<T, L, C, decltype(rows)::value, decltype(w)::value, TH>), dim3(sets),
          dim3(TH), lds, st, static_cast<const T*>(scores), key_len, causal, static_cast<T*>(probs),
          static_cast<T*>(out), keep_bits, slices, static_cast<int>(Sq), static_cast<int>(Sk), scale,
          rng, sets_per_slice, heads, first_set);
    });
  };
  using std::integral_constant;
  const integral_constant<MaskLayout, kWords> words{};
  const integral_constant<MaskLayout, kBytes> bytes{};
  if constexpr (std::is_same<T, bf16_t>::value && C == 1 && L == kWave) {  // attn_rows()
    if (rr == 2) {
      if (layout == kWords) return go(integral_constant<int, 2>{}, words);
      return go(integral_constant<int, 2>{}, bytes);
    }
  }
  if constexpr (has_kernel(L, C, Store<T>::kVec, true, false)) {
    if (layout == kRagged) return go(integral_constant<int, 1>{}, integral_constant<MaskLayout, kRagged>{});
  }
  if constexpr (has_kernel(L, C, Store<T>::kVec, false, false)) {
    if (layout == kWords) return go(integral_constant<int, 1>{}, words);
    go(integral_constant<int, 1>{}, bytes);
  }
}

template <typename T, int L, int C>
static void attn_bwd_go(MaskSource mask, bool ragged, int threads, size_t lds, uint32_t first_set, uint32_t sets, hipStream_t st, const void* dout,
                        const void* probs, const uint32_t* keep_bits, void* dscores, void* out_re,
                        int64_t rows, int64_t Sk, float scale, const RngArgs& rng) {
  auto go = [&](auto m, auto rag) {
    with_threads<L, true, decltype(rag)::value>(threads, [&](auto th) {
      constexpr int TH = decltype(th)::value;
      hipLaunchKernelGGL((attn_bwd_kernel<T, L, C, decltype(m)::value, decltype(rag)::value, TH>), dim3(sets), dim3(TH),
                         lds, st, static_cast<const T*>(dout), static_cast<const T*>(probs), keep_bits,
                         static_cast<T*>(dscores), static_cast<T*>(out_re),
                         static_cast<uint32_t>(rows), static_cast<int>(Sk), scale, rng, first_set);
    });
  };
  using std::integral_constant;
  const integral_constant<MaskSource, kMaskBytes> bytes{};
  const integral_constant<MaskSource, kMaskBools> bools{};
  const integral_constant<MaskSource, kMaskRegen> regen{};
  if constexpr (has_kernel(L, C, Store<T>::kVec, true, true)) {
    if (ragged) {
      if (mask == kMaskBytes) return go(bytes, std::true_type{});
      if (mask == kMaskBools) return go(bools, std::true_type{});
      return go(regen, std::true_type{});
    }
  }
  if constexpr (has_kernel(L, C, Store<T>::kVec, false, true)) {
    if (mask == kMaskWords) return go(integral_constant<MaskSource, kMaskWords>{}, std::false_type{});
    if (mask == kMaskBytes) return go(bytes, std::false_type{});
    if (mask == kMaskBools) return go(bools, std::false_type{});
    go(regen, std::false_type{});
  }
}

static RngArgs make_rng(float p, uint64_t seed, uint64_t offset) {
  RngArgs rng;
  rng.seed_lo = static_cast<uint32_t>(seed);
  rng.seed_hi = static_cast<uint32_t>(seed >> 32);
  rng.off_lo = static_cast<uint32_t>(offset);
  rng.off_hi = static_cast<uint32_t>(offset >> 32);
  double t = (1.0 - static_cast<double>(p)) * 65536.0 + 0.5;
  t = t < 0.0 ? 0.0 : (t > 65536.0 ? 65536.0 : t);
  rng.t16 = (p == 0.0f) ? 65536u : static_cast<uint32_t>(t);  // floor for t >= 0
  return rng;
}

tempo_status launch_attn_fwd(const void* scores, const int32_t* key_len, int causal, void* probs,
                             void* out, uint32_t* keep_bits, int64_t B, int64_t A, int64_t Sq,
                             int64_t Sk, float p, uint64_t seed, uint64_t offset, tempo_dtype dt,
                             hipStream_t st) {
  // A workgroup's rows are of one slice.  Where no causal mask tells the rows of a slice apart, those of a
  // batch (of the call, without key_len) count as one: few rows per slice would leave most of the workgroup
  // idle (2^24 slices of one row of one bf16 element: 8.5 ms, 0.41 this way; 1024x16x1x333 17.4 us, 13.8).
  if (Sq == 1) causal = 0;  // the only row sees every key
  const int64_t alike = key_len ? A * Sq : B * A * Sq;
  if (!causal && alike <= int64_t{1} << 30) {
    if (!key_len) B = 1;
    A = 1;
    Sq = alike;
  }
  const int64_t rows = B * A * Sq;
  const int64_t rows_per_batch = A * Sq;
  const float scale = 1.0f / (1.0f - p);
  const RngArgs rng = make_rng(p, seed, offset);
  const int bpc = tune_get(kTuneAttnFwdBlocksPerCu);
  const int vec = dt == TEMPO_F32 ? 4 : 8;
  const bool ragged = Sk % 8 != 0;
  const Shape sh = row_shape(Sk, vec, tune_get(kTuneAttnFwdMaxPieces), causal ? kForwardCausal : kForward);
  if (sh.ch != 0 && rows <= UINT32_MAX) {  // rows counted in 32 bits
    const int slices = static_cast<int>(B * A);
    const int rr = sh.lanes > kWave || ragged
                       ? 1 : attn_rows(sh.ch, sh.lanes, vec, tune_get(kTuneAttnFwdRows));
    const int threads =
        ragged ? fixed_threads(sh.lanes, false) : group_threads(sh.lanes, false);
    const int rows_per_set = (threads / sh.lanes) * rr;
    const FastDiv sets_per_slice(static_cast<uint32_t>((Sq + rows_per_set - 1) / rows_per_set));
    const FastDiv heads(static_cast<uint32_t>(A));
    const int64_t total_sets = static_cast<int64_t>(slices) * sets_per_slice.d;
    const int pieces = static_cast<int>((Sk + vec - 1) / vec);
    const size_t lds = dt == TEMPO_F32 ? fwd_f32_lds_bytes(sh, pieces, threads, causal != 0, key_len != nullptr) : 0;
    const MaskLayout layout = ragged ? kRagged : (Sk % 32 == 0 ? kWords : kBytes);
#define TEMPO_LAUNCH(L, C)                                                                   \
  do {                                                                                       \
    if (dt == TEMPO_F32) attn_fwd_go<float, L, C>(rr, layout, threads, lds, first, sets, st, scores, key_len, causal, probs, out, keep_bits, slices, heads, sets_per_slice, Sq, Sk, scale, rng);   \
    else attn_fwd_go<bf16_t, L, C>(rr, layout, threads, lds, first, sets, st, scores, key_len, causal, probs, out, keep_bits, slices, heads, sets_per_slice, Sq, Sk, scale, rng);                  \
  } while (0)
    const int64_t cap = most_groups(static_cast<int64_t>(compute_units()) * bpc, threads);
    tempo_status status = TEMPO_OK;
    split_launch(total_sets, cap, [&](uint32_t first, uint32_t sets) {
      status = [&]() -> tempo_status {
        if (sh.lanes > kWave) {
          TEMPO_ATTN_WIDE_DISPATCH(TEMPO_LAUNCH)
        } else {
          TEMPO_ATTN_DISPATCH(TEMPO_LAUNCH)
        }
        return launch_status();
      }();
      return status == TEMPO_OK;
    });
#undef TEMPO_LAUNCH
    return status;
  }
  const int grid = row_grid(rows, bpc);
  if (dt == TEMPO_F32)
    hipLaunchKernelGGL((attn_fwd_generic_kernel<float>), dim3(grid), dim3(kThreads), 0, st,
                       static_cast<const float*>(scores), key_len, causal,
                       static_cast<float*>(probs), static_cast<float*>(out), rows, rows_per_batch,
                       static_cast<int>(Sq), static_cast<int>(Sk), scale, rng);
  else
    hipLaunchKernelGGL((attn_fwd_generic_kernel<bf16_t>), dim3(grid), dim3(kThreads), 0, st,
                       static_cast<const bf16_t*>(scores), key_len, causal,
                       static_cast<bf16_t*>(probs), static_cast<bf16_t*>(out), rows,
                       rows_per_batch, static_cast<int>(Sq), static_cast<int>(Sk), scale, rng);
  if (hipGetLastError() != hipSuccess) return TEMPO_ERR_LAUNCH;
  const int64_t n = rows * Sk;
  const int64_t words = (n + 31) / 32;
  const int64_t wgrid = (words + kThreads - 1) / kThreads;
  const int64_t cap = static_cast<int64_t>(compute_units()) * 8;
  hipLaunchKernelGGL(keep_words_kernel, dim3(static_cast<int>(wgrid < cap ? wgrid : cap)),
                     dim3(kThreads), 0, st, keep_bits, n, rng);
  return launch_status();
}

// keep_bits == nullptr: no stored mask, the bits are drawn again from (seed, offset).
// bools: keep_bits points to one byte per element instead of packed bits.
static tempo_status attn_bwd_any(const void* dout, const void* probs, const uint32_t* keep_bits,
                                 bool bools, void* dscores, void* out_re, int64_t B, int64_t A,
                                 int64_t Sq, int64_t Sk, float p, const RngArgs& rng,
                                 tempo_dtype dt, hipStream_t st) {
  const int64_t rows = B * A * Sq;
  const float scale = 1.0f / (1.0f - p);
  const bool regen = keep_bits == nullptr;
  const int bpc = tune_get(kTuneAttnBwdBlocksPerCu);
  const int vec = dt == TEMPO_F32 ? 4 : 8;
  const bool ragged = Sk % 8 != 0;
  const Shape sh = row_shape(Sk, vec, tune_get(kTuneAttnBwdMaxPieces), kBackward);
  if (sh.ch != 0 && rows <= UINT32_MAX) {  // rows counted in 32 bits
    const int threads =
        ragged ? fixed_threads(sh.lanes, true) : group_threads(sh.lanes, true);
    const int64_t total_sets = (rows + threads / sh.lanes - 1) / (threads / sh.lanes);
    const int pieces = static_cast<int>((Sk + vec - 1) / vec);
    const size_t lds = residency_lds_bytes(bwd_waves(sh, pieces, regen, ragged), threads);
    const MaskSource mask =
        regen ? kMaskRegen : (bools ? kMaskBools : (Sk % 32 == 0 ? kMaskWords : kMaskBytes));
#define TEMPO_LAUNCH(L, C)                                                                   \
  do {                                                                                       \
    if (dt == TEMPO_F32) attn_bwd_go<float, L, C>(mask, ragged, threads, lds, first, sets, st, dout, probs, keep_bits, dscores, out_re, rows, Sk, scale, rng);   \
    else attn_bwd_go<bf16_t, L, C>(mask, ragged, threads, lds, first, sets, st, dout, probs, keep_bits, dscores, out_re, rows, Sk, scale, rng);                  \
  } while (0)
    const int64_t cap = most_groups(static_cast<int64_t>(compute_units()) * bpc, threads);
    tempo_status status = TEMPO_OK;
    split_launch(total_sets, cap, [&](uint32_t first, uint32_t sets) {
      status = [&]() -> tempo_status {
        if (sh.lanes > kWave) {
          TEMPO_ATTN_WIDE_DISPATCH(TEMPO_LAUNCH)
        } else {
          TEMPO_ATTN_DISPATCH(TEMPO_LAUNCH)
        }
        return launch_status();
      }();
      return status == TEMPO_OK;
    });
#undef TEMPO_LAUNCH
    return status;
  }
  const int grid = row_grid(rows, bpc);
  auto go = [&](auto tag, auto m) {
    using T = decltype(tag);
    hipLaunchKernelGGL((attn_bwd_generic_kernel<T, decltype(m)::value>), dim3(grid),
                       dim3(kThreads), 0, st, static_cast<const T*>(dout),
                       static_cast<const T*>(probs), keep_bits, static_cast<T*>(dscores),
                       static_cast<T*>(out_re), rows, static_cast<int>(Sk), scale, rng);
  };
  using std::integral_constant;
  auto with_mask = [&](auto tag) {
    if (regen) go(tag, integral_constant<MaskSource, kMaskRegen>{});
    else if (bools) go(tag, integral_constant<MaskSource, kMaskBools>{});
    else go(tag, integral_constant<MaskSource, kMaskWords>{});
  };
  if (dt == TEMPO_F32) with_mask(float{});
  else with_mask(bf16_t{});
  return launch_status();
}

tempo_status launch_attn_bwd(const void* dout, const void* probs, const uint32_t* keep_bits,
                             void* dscores, void* out_re, int64_t B, int64_t A, int64_t Sq,
                             int64_t Sk, float p, tempo_dtype dt, hipStream_t st) {
  return attn_bwd_any(dout, probs, keep_bits, false, dscores, out_re, B, A, Sq, Sk, p,
                      make_rng(0.0f, 0, 0), dt, st);
}

tempo_status launch_attn_bwd_bytemask(const void* dout, const void* probs,
                                      const uint8_t* keep_bytes, void* dscores, void* out_re,
                                      int64_t B, int64_t A, int64_t Sq, int64_t Sk, float p,
                                      tempo_dtype dt, hipStream_t st) {
  return attn_bwd_any(dout, probs, reinterpret_cast<const uint32_t*>(keep_bytes), true, dscores,
                      out_re, B, A, Sq, Sk, p, make_rng(0.0f, 0, 0), dt, st);
}

tempo_status launch_attn_bwd_regen(const void* dout, const void* probs, void* dscores,
                                   void* out_re, int64_t B, int64_t A, int64_t Sq, int64_t Sk,
                                   float p, uint64_t seed, uint64_t offset, tempo_dtype dt,
                                   hipStream_t st) {
  return attn_bwd_any(dout, probs, nullptr, false, dscores, out_re, B, A, Sq, Sk, p,
                      make_rng(p, seed, offset), dt, st);
}

}  // namespace tempo
