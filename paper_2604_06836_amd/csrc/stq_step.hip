// gfx950 kernel of the quantized Adam step: the per-layer loop body of Algorithm 1 of the paper
// (moment update, Quantize(m,'linear'), Quantize(v,'log'), bias correction of the quantized
// moments, decoupled-weight-decay update) with the block quantizers of Section 3.5 and the
// per-layer statistics of Section 3.3, fused into one pass over HBM.
//
// Arithmetic contract: IEEE binary32, every operation rounded on its own (build with
// -ffp-contract=off); division and square root are the correctly rounded ones.
//
// Work decomposition: one wavefront works on one part of a 2048-element tile at a time, a half (4 rows) or, in small
// launches, a quarter (2 rows).  A half's working set fits the 128 registers of four waves per SIMD (107 to 124 in use), a
// quarter's the 80 of six, with nothing spilled to scratch memory, so the kernel's HBM traffic is the algorithmic traffic.
// In row i lane j holds the 4 elements 256*i + 4*j + e, so
// every parameter and gradient access is a coalesced 16-byte (8-byte for bf16) per-lane access,
// and a block of K = 64/128/256 consecutive elements is 16/32/64 neighbouring lanes of one row.
// The lane's 32 codes of a state are exactly b 32-bit words; word p of all lanes is one contiguous
// 256-byte row of the code buffer.  A part reads the words that hold its codes and writes the words, or the bytes of
// words that it shares with its neighbours, that are its own: a part's codes start and end on a byte.
//
// Only the bit-stream unpack and pack are specialised per width (small switch arms); all
// arithmetic is width-generic and takes the width through table offsets and constants.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cstdint>
#include <utility>

#include "stq_device.h"
#include "stq_round.h"
#include "stq_tables.h"
#include "stq_wave.h"

#pragma clang fp contract(off)

namespace stq {
namespace {

constexpr int XS = 68;  // row stride (words) of the transpose scratch: keeps 16-byte alignment, shifts banks
// The part of a tile that a wave works on at a time: ROWS rows of 256 elements, 4*ROWS elements per lane.
template <int ROWS>
struct Part {
  static constexpr int kLgRows = ROWS == 2 ? 1 : 2;
  static constexpr int kElems = 4 * ROWS;          // per lane
  static constexpr int kPairs = 2 * ROWS;          // (state, row) pairs; a pair's block scales belong to 64/kPairs lanes
  static constexpr int kLgPairs = kLgRows + 1;
  // per-wave LDS scratch: XR[kPairs][XS] partial maxima (later the den or root table), old scales, new scales, reciprocals
  static constexpr int kTableWords = kPairs * XS;
  static constexpr int kScratch = kTableWords + 3 * 64;
  static constexpr uint32_t kDenEntries = 64u * ROWS;  // capacity of the per-wave den table (8 bytes per entry, inside XR)
  static_assert(ROWS == 2 || ROWS == 4, "quarters and halves of a tile");
  static_assert(kDenEntries * 2 <= kTableWords, "the den table lies inside XR");
  static_assert((4 * ROWS) << (kMaxBits - 3) <= kTableWords, "and so do the roots of the widest code at the smallest block");
};
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// value at byte offset `off` of an LDS float table
__device__ __forceinline__ float lds_at(const float* base, uint32_t off) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off);
}

__device__ __forceinline__ void wave_lds_sync() {
  // LDS operations of one wavefront execute in order; this only stops the compiler from moving
  // accesses of other lanes' data across the point.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- bit streams
// Within a part, code n of width B sits at bits [n*B, n*B+B) of the part's local stream.
// Bits [SH, SH+B) of x in one instruction.  Written as the instruction itself: from the plain expression
// the compiler makes a shift and a mask, and then cannot fold the table offset that follows into either.
template <int SH, int B>
__device__ __forceinline__ uint32_t bit_field(uint32_t x) {
  uint32_t r;
  asm("v_bfe_u32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "n"(SH), "n"(B));
  return r;
}

template <int B, int N, int W>
__device__ __forceinline__ uint32_t extract(const uint32_t (&w)[W]) {
  constexpr int off = N * B, p = off >> 5, sh = off & 31;
  if constexpr (sh + B <= 32) return bit_field<sh, B>(w[p]);
  // a code that straddles two words: align it first
  else return bit_field<0, B>(__builtin_amdgcn_alignbit(w[p + 1], w[p], static_cast<uint32_t>(sh)));
}

// Byte N of x, times 4; byte N of x masked: one instruction each (the byte is selected by the operand).
template <int N>
__device__ __forceinline__ uint32_t byte_times4(uint32_t x, uint32_t two) {
  uint32_t r;
  if (N == 0) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(two), "v"(x));
  if (N == 1) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(two), "v"(x));
  if (N == 2) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(two), "v"(x));
  if (N == 3) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(two), "v"(x));
  return r;
}
template <int N>
__device__ __forceinline__ uint32_t byte_and(uint32_t x, uint32_t mask) {
  uint32_t r;
  if (N == 0) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "s"(mask), "v"(x));
  if (N == 1) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "s"(mask), "v"(x));
  if (N == 2) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "s"(mask), "v"(x));
  if (N == 3) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "s"(mask), "v"(x));
  return r;
}

template <int B, int W, int... N>
__device__ __forceinline__ void extract_offsets(const uint32_t (&w)[W], uint32_t* off, std::integer_sequence<int, N...>) {
  ((off[N] = extract<B, N>(w) << 2), ...);
}

// The codes of a part, times 4: byte offsets into the width's value table.
// lw holds the lane's words from the one that contains the part's first bit; s0 is the position of that bit in lw[0]
// (0, 8, 16 or 24 for a quarter, 0 or 16 for a half; always 0 where kWordAligned).
template <int ROWS, int B>
constexpr bool kWordAligned = (4 * ROWS * B) % 32 == 0;
template <int ROWS, int B, int W>
__device__ __forceinline__ void unpack_offsets(const uint32_t (&lw)[W], uint32_t s0, uint32_t (&off)[4 * ROWS]) {
  if constexpr (B == 8) {
    uint32_t two = 2u;
    asm("" : "+v"(two));
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      off[4 * k + 0] = byte_times4<0>(lw[k], two); off[4 * k + 1] = byte_times4<1>(lw[k], two);
      off[4 * k + 2] = byte_times4<2>(lw[k], two); off[4 * k + 3] = byte_times4<3>(lw[k], two);
    }
  } else if constexpr (B == 4) {
#pragma unroll
    for (int k = 0; k < ROWS / 2; ++k) {
      const uint32_t even = lw[k] << 2, odd = lw[k] >> 2;  // code 2i / 2i+1 at bits 2..5 of byte i
      off[8 * k + 0] = byte_and<0>(even, 0x3Cu); off[8 * k + 1] = byte_and<0>(odd, 0x3Cu);
      off[8 * k + 2] = byte_and<1>(even, 0x3Cu); off[8 * k + 3] = byte_and<1>(odd, 0x3Cu);
      off[8 * k + 4] = byte_and<2>(even, 0x3Cu); off[8 * k + 5] = byte_and<2>(odd, 0x3Cu);
      off[8 * k + 6] = byte_and<3>(even, 0x3Cu); off[8 * k + 7] = byte_and<3>(odd, 0x3Cu);
    }
  } else {
    constexpr int kWords = (4 * ROWS * B + 31) / 32;
    uint32_t w[kWords + 1];
#pragma unroll
    for (int k = 0; k < kWords; ++k) w[k] = kWordAligned<ROWS, B> ? lw[k] : __builtin_amdgcn_alignbit(k + 1 < W ? lw[k + 1] : 0u, lw[k], s0);
    w[kWords] = 0u;
    extract_offsets<B>(w, off, std::make_integer_sequence<int, 4 * ROWS>{});
  }
}

// Stores of a launch that writes through (see launch_table): to memory at once instead of when the L2 makes room.  (Only both
// the parameters and the words of codes together gain; the bytes of words that two parts share are left to the L2, which
// has them from both.  The words of 16- and 32-bit states are plain stores in every variant.)
__device__ __forceinline__ void store_through(STQ_GLOBAL uint32_t* p, uint32_t x) {
  __hip_atomic_store((uint32_t*)p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// 16 bytes to byte `off` of the `bytes` at base (the same in all lanes), with the non-temporal hint
__device__ __forceinline__ void store_through(STQ_GLOBAL float* base, int bytes, uint32_t off, f32x4 x) {
  constexpr int kNt = 2, kSc1 = 16;
  const auto where = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);  // (a raw buffer)
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), where, off, 0, kNt | kSc1);
}
// a whole word of codes
template <bool THROUGH>
__device__ __forceinline__ void store_word(STQ_GLOBAL uint32_t* p, uint32_t x) {
  if constexpr (THROUGH) store_through(p, x);
  else *p = x;
}

// Bytes [FIRST, END) of x to the same bytes of the word at p.
template <int FIRST, int END>
__device__ __forceinline__ void store_bytes(STQ_GLOBAL uint32_t* p, uint32_t x) {
  STQ_GLOBAL uint8_t* b = reinterpret_cast<STQ_GLOBAL uint8_t*>(p);
  STQ_GLOBAL uint16_t* h = reinterpret_cast<STQ_GLOBAL uint16_t*>(p);
  if constexpr (FIRST == 0 && END == 4) *p = x;
  else if constexpr (FIRST == 0 && END >= 2) h[0] = static_cast<uint16_t>(x);
  else if constexpr (FIRST <= 2 && END == 4) h[1] = static_cast<uint16_t>(x >> 16);
  if constexpr (FIRST == 0 && END == 1) b[0] = static_cast<uint8_t>(x);
  if constexpr (FIRST == 1) b[1] = static_cast<uint8_t>(x >> 8);
  if constexpr (FIRST == 0 && END == 3) b[2] = static_cast<uint8_t>(x >> 16);
  if constexpr (FIRST == 3) b[3] = static_cast<uint8_t>(x >> 24);
  static_assert((FIRST == 0 && END >= 1) || (FIRST >= 1 && END == 4), "a part starts or ends with its word");
}

// Pack the low B bits of the codes of a part and store them from bit s0 of the word at C on (word stride 64).
// Each code enters its word from the top with one v_alignbit, which needs no masking of what lies above the code; MINUS1:
// the codes given are all one too large (and at least 1), which one subtraction per word undoes (and one per code that
// straddles two words).
// Other waves have the parts before and after this one: of the words that it shares with them it writes its own bytes (a
// part starts and ends on a byte; their waves read these words as a whole, but use no byte that is not theirs).
template <int ROWS, int B, bool MINUS1, bool THROUGH>
__device__ __forceinline__ void pack_store(const uint32_t (&code)[4 * ROWS], STQ_GLOBAL uint32_t* C, uint32_t s0, uint32_t lane) {
  constexpr int N = 4 * ROWS, kBits = N * B, kWhole = kBits / 32, kWords = (kBits + 31) / 32;
  uint32_t w[kWords], ones[kWords];  // the part's bits, and a 1 for each of its codes that lies in one word
#pragma unroll
  for (int k = 0; k < kWords; ++k) ones[k] = 0u;
  {
    uint32_t x = 0u;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int p = (n * B) >> 5, at = (n * B) & 31, in_word = 32 - at;  // bits left in word p
      if (B <= in_word) {
        ones[p] |= 1u << at;
        x = at == 0 ? code[n] << (32 - B) : __builtin_amdgcn_alignbit(code[n], x, B);
        if (B == in_word) w[p] = x;
      } else {
        const uint32_t c = MINUS1 ? code[n] - 1u : code[n];
        w[p] = __builtin_amdgcn_alignbit(c, x, in_word);
        x = c << (32 - B);  // (its lowest bits, which are in w[p], leave the word at the bottom again)
      }
    }
    if (kBits % 32 != 0) w[kWords - 1] = x >> (32 - kBits % 32);
  }
  if (MINUS1) {
#pragma unroll
    for (int k = 0; k < kWords; ++k) w[k] -= ones[k];
  }
  C += lane;
  if (kWordAligned<ROWS, B> || s0 == 0) {
#pragma unroll
    for (int k = 0; k < kWhole; ++k) store_word<THROUGH>(C + 64u * k, w[k]);
    if constexpr (kWhole < kWords) store_bytes<0, kBits % 32 / 8>(C + 64 * kWhole, w[kWhole]);
    return;
  }
  if constexpr (!kWordAligned<ROWS, B>) {
    const uint32_t m0 = w[0] << s0;
    if constexpr (ROWS == 4) {  // the second half of a tile, from the middle of a word to the end of one
      store_bytes<2, 4>(C, m0);
#pragma unroll
      for (int k = 1; k < kWords; ++k) store_word<THROUGH>(C + 64u * k, __builtin_amdgcn_alignbit(w[k], w[k - 1], 16u));
    } else {  // a quarter in the middle or at the end of a tile: of three words at most
      const uint32_t hi = kWords == 2 ? w[kWords - 1] : 0u;
      const uint32_t m1 = __builtin_amdgcn_alignbit(hi, w[0], 32u - s0), m2 = hi >> (32u - s0);
      const uint32_t end = s0 + kBits, done = end >> 5;  // words that end within the part: 1 or 2
      if (s0 == 8) store_bytes<1, 4>(C, m0);
      else if (s0 == 16) store_bytes<2, 4>(C, m0);
      else store_bytes<3, 4>(C, m0);
      if (done == 2) C[64] = m1;
      const uint32_t rest = done == 2 ? m2 : m1;
      STQ_GLOBAL uint32_t* last = C + 64u * done;
      switch (end & 31u) {
        case 8: store_bytes<0, 1>(last, rest); break;
        case 16: store_bytes<0, 2>(last, rest); break;
        case 24: store_bytes<0, 3>(last, rest); break;
        default: break;
      }
    }
  }
}

#define STQ_SWITCH_BITS(bits, CALL)               \
  switch (bits) {                                 \
    case 2: { constexpr int B = 2; CALL; } break; \
    case 3: { constexpr int B = 3; CALL; } break; \
    case 4: { constexpr int B = 4; CALL; } break; \
    case 5: { constexpr int B = 5; CALL; } break; \
    case 6: { constexpr int B = 6; CALL; } break; \
    case 7: { constexpr int B = 7; CALL; } break; \
    default: { constexpr int B = 8; CALL; } break; \
  }

// element n of this lane in part q is real (not pad) in a tile with n_valid elements
template <int ROWS>
__device__ __forceinline__ bool is_valid(int n, uint32_t q, int lane, uint32_t n_valid) {
  return (256u * ROWS * q + static_cast<uint32_t>(256 * (n >> 2) + 4 * lane + (n & 3))) < n_valid;
}

// -------------------------------------------------------------------- statistics
// (The sums of squares use fused multiply-adds: the fixed operation order binds the Adam
// arithmetic, not the statistics, which are compared within a tolerance.)
// Running statistics of one wave, kept in its LDS slice so that they cost no registers between the places
// that add to them.  A contribution is first combined over a few neighbouring lanes with DPP steps, then one
// lane of the group adds it to the group's word with an LDS atomic that returns nothing: the wave does not
// wait for it, where a read-modify-write would put an LDS round trip into every part's dependency chain
// (that latency, not the arithmetic, was most of the statistics' cost: it showed when fewer waves were
// resident to hide it).  The atomics are issued from 8 or 16 lanes: from all 64 they are several times slower.
//  * The gradient's three sums (all that the bit-width decision reads, Eq. 2, 3, 8) are taken in fp64 from the
//    first addition on: fp64 vector additions issue at the rate of fp32 ones here, and a decision that compares a
//    score with a threshold should not hinge on the rounding of a sum (the variance in Eq. 3 is a difference of
//    two such sums).  Groups of four lanes, 16-word slots; the gradient's maximum likewise in a 16-word slot of
//    bit patterns (all maxima are non-negative, so they order like their bit patterns).
//  * S = 1 adds the moments' six sums (groups of eight lanes, 8-word slots): that of the first moments, whose terms cancel, in
//    fp64 like the gradient's, the others, of terms that are not negative, in fp32 over the eight elements that a lane has in
//    two rows and in fp64 from there on; and two maxima (the owner lanes of the block scales hold them: lanes 0..31 the first
//    moment's, 32..63 the second's, so a group of four is of one kind).
// S = 2: the gradient's statistics only.
enum GradSlot { kLGSum = 0, kLGAbs, kLGSq };
enum MomentSlot { kLMSum = 0, kLMSq, kLMErr, kLVSum, kLVSq, kLVErr };

// Layout of a wave's slice (32-bit words), S = 2 | S = 1:
//   gradient sums  3 slots of G doubles, G = 16 | 8 (one word per group of 64/G lanes)
//   maxima         16 | 32 words: [0, G) max|g|; S = 1: [16, 24) max|m| (lanes 0..31 own the first moment's
//                  block scales), [24, 32) max v (lanes 32..63); words [8, 16) stay 0
//   S = 1 only     moment sums: 6 slots of 8 doubles
template <int S>
struct LaneStats {
  static constexpr int kGShift = S == 1 ? 3 : 2;  // log2 of the lanes that share a gradient word
  static constexpr int kG = 64 >> kGShift;        // words per gradient slot
  static constexpr int kMaxWords = S == 1 ? 32 : 16;
  static constexpr int kMaxOff = 3 * 2 * kG, kMomentOff = kMaxOff + kMaxWords;
  static constexpr int kWords = S == 0 ? 0 : (S == 1 ? kMomentOff + 6 * 8 * 2 : kMomentOff);
  float* acc;      // this wave's slice, null in the plain kernel
  __device__ __forceinline__ double* grad_sums() const { return reinterpret_cast<double*>(acc); }
  __device__ __forceinline__ uint32_t* maxima() const { return reinterpret_cast<uint32_t*>(acc) + kMaxOff; }
  __device__ __forceinline__ double* moment_sums() const { return reinterpret_cast<double*>(acc + kMomentOff); }

  __device__ __forceinline__ void add_grad(int k, int lane, double x) {
    x = S == 1 ? octet_sum(x) : quad_sum(x);
    if ((lane & ((1 << kGShift) - 1)) == 0)
      __hip_atomic_fetch_add(&grad_sums()[k * kG + (lane >> kGShift)], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  __device__ __forceinline__ void max_grad(int lane, float x) {
    const uint32_t xb = S == 1 ? octet_max(f2u(x)) : quad_max(f2u(x));
    if ((lane & ((1 << kGShift) - 1)) == 0)
      __hip_atomic_fetch_max(maxima() + (lane >> kGShift), xb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  // parts: the fp32 sums of two rows each
  template <int PAIRS>
  __device__ __forceinline__ void add(int slot, int lane, const float (&parts)[PAIRS]) {
    double x = static_cast<double>(parts[0]);
    if (PAIRS == 2) x += static_cast<double>(parts[PAIRS - 1]);
    add(slot, lane, x);
  }
  __device__ __forceinline__ void add(int slot, int lane, double x) {
    x = octet_sum(x);
    if ((lane & 7) == 0)
      __hip_atomic_fetch_add(&moment_sums()[slot * 8 + (lane >> 3)], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  // the maximum of a block of a moment, from its owner lanes (a quad is of one kind: see the layout)
  __device__ __forceinline__ void max_moment(int lane, float x) {
    const uint32_t xb = quad_max(f2u(x));
    if ((lane & 3) == 0)
      __hip_atomic_fetch_max(maxima() + 16 + (lane >> 2), xb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  __device__ __forceinline__ void clear(int lane) {
    if (lane < 3 * kG) grad_sums()[lane] = 0.0;
    if (lane < kMaxWords) maxima()[lane] = 0u;
    if (S == 1 && lane < 48) moment_sums()[lane] = 0.0;
  }
  // The reductions of a slice, for the flushes below (call wave_lds_sync() first).
  // Gradient sum k (0..2), complete, in the lanes [k*kG, (k+1)*kG); zero in the lanes from 3*kG on.
  __device__ __forceinline__ double reduced_grad(int lane) const {
    const double x = lane < 3 * kG ? grad_sums()[lane] : 0.0;
    return S == 1 ? octet_sum(x) : row_sum(x);
  }
  // Moment sum k (0..5) in the lanes [8k, 8k+8); zero from lane 48 on.
  __device__ __forceinline__ double reduced_moment(int lane) const { return octet_sum(lane < 48 ? moment_sums()[lane] : 0.0); }
  // max|g| in lane 0; S = 1: max|m| in lane 16, max v in lane 24.
  __device__ __forceinline__ uint32_t reduced_max(int lane) const {
    const uint32_t x = lane < kMaxWords ? maxima()[lane] : 0u;
    return S == 1 ? octet_max(x) : row_max(x);
  }
  // lane holds gradient sum `k` / moment sum `k` / maximum `k` (0 g, 1 m, 2 v) of the reductions above
  __device__ __forceinline__ static bool grad_lead(int lane, int& k) { k = lane >> (6 - kGShift); return lane < 3 * kG && (lane & (kG - 1)) == 0; }
  __device__ __forceinline__ static bool moment_lead(int lane, int& k) { k = lane >> 3; return S == 1 && lane < 48 && (lane & 7) == 0; }
  __device__ __forceinline__ static bool max_lead(int lane, int& k) {
    k = lane == 0 ? 0 : (lane == 16 ? 1 : 2);
    return lane == 0 || (S == 1 && (lane == 16 || lane == 24));
  }
};

// the wave's statistics -> the tensor's global slots; the slice is cleared
template <int S>
__device__ __forceinline__ void flush_stats(LaneStats<S>& s, double* slot, int lane) {
  asm volatile("" : "+v"(lane));
  wave_lds_sync();
  const double g = s.reduced_grad(lane);
  const uint32_t mx = s.reduced_max(lane);
  uint32_t* out = reinterpret_cast<uint32_t*>(&slot[kMaxGM]);  // max |g|, max |m|, max v: consecutive words
  int k;
  if (LaneStats<S>::grad_lead(lane, k)) atomicAdd(&slot[kGSum + k], g);
  if (LaneStats<S>::max_lead(lane, k)) atomicMax(&out[k], mx);
  if (S == 1) {
    const double mo = s.reduced_moment(lane);
    if (LaneStats<S>::moment_lead(lane, k)) atomicAdd(&slot[kMSum + k], mo);
  }
  s.clear(lane);
}

// ---- the workgroup's statistics ----
// The waves of a workgroup keep their sums while the workgroup's units stay in one tensor (that of the first unit of each
// ticket).  When it goes on to another, each wave reduces its values over its lanes into its record, and after a barrier
// wave 0 adds up the records and adds the result to the tensor's global slots: one set of global atomics per workgroup
// and tensor.  A wave whose unit lies in a later tensor than the first unit of its ticket adds to the global slots itself.
template <int S>
struct StatRecord {
  double sum[S == 1 ? 9 : 3];           // in the order of the global slots from kGSum on
  uint32_t max_bits[S == 1 ? 4 : 2];    // max|g|, (max|m|, max v,) pad
};

// the wave's statistics -> its record; the slice is cleared
template <int S>
__device__ __forceinline__ void record_stats(LaneStats<S>& s, StatRecord<S>* rec, int lane) {
  asm volatile("" : "+v"(lane));
  wave_lds_sync();
  const double g = s.reduced_grad(lane), mo = S == 1 ? s.reduced_moment(lane) : 0.0;
  const uint32_t mx = s.reduced_max(lane);
  int k;
  if (LaneStats<S>::grad_lead(lane, k)) rec->sum[k] = g;
  if (LaneStats<S>::moment_lead(lane, k)) rec->sum[3 + k] = mo;
  if (LaneStats<S>::max_lead(lane, k)) rec->max_bits[k] = mx;
  s.clear(lane);
}

// wave 0, after a barrier: the records of the workgroup's waves -> the tensor's global slots
template <int S>
__device__ __forceinline__ void flush_records(const StatRecord<S>* recs, double* slot, int lane) {
  static_assert(kWavesPerGroup == 8, "lane 8 k + w takes value k of wave w's record");
  asm volatile("" : "+v"(lane));
  constexpr int kSums = S == 1 ? 9 : 3, kMaxima = S == 1 ? 3 : 1;
  const StatRecord<S>& r = recs[lane & 7];
  const int k = lane >> 3;
  const bool lead = (lane & 7) == 0;
  const double x = octet_sum(k < kSums ? r.sum[k] : 0.0);
  if (lead && k < kSums) atomicAdd(&slot[kGSum + k], x);
  if (kSums > 8) {
    const double y = octet_sum(lane < 8 ? r.sum[kSums - 1] : 0.0);  // the ninth
    if (lane == 0) atomicAdd(&slot[kGSum + 8], y);
  }
  const uint32_t mx = octet_max(k < kMaxima ? r.max_bits[k] : 0u);
  if (lead && k < kMaxima) atomicMax(reinterpret_cast<uint32_t*>(&slot[kMaxGM]) + k, mx);
}

// Whether every number added is +0 or has its magnitude between two given ones (as bit patterns).  -0 does not pass: the
// short quotient makes +0 of it, the IEEE one -0, which shows in a parameter that is itself -0.  (A quantized moment is
// never -0.)
struct SafeRange {
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  __device__ __forceinline__ void add(float x) {
    const uint32_t u = __builtin_rotateleft32(f2u(x), 1);  // the magnitude, below it the sign: +0 is 0 and -0 is 1
    lo = min(lo, u - 1u);  // +0 passes
    hi = max(hi, u);
  }
  __device__ __forceinline__ bool within(uint32_t least, uint32_t most) const { return lo >= 2u * least - 1u && hi <= 2u * most + 1u; }
};
// 2^-40 <= x <= 2^40, for x >= 0: positive floats order like their bit patterns
__device__ __forceinline__ bool in_safe_range(float x) { return f2u(x) - 0x2B800000u <= 0x53800000u - 0x2B800000u; }

// ------------------------------------------------------------------ update
struct UpdateArgs {
  float ibc1, ibc2, eps, lr, decay;
};

// theta' = theta*decay - lr * ratio
__device__ __forceinline__ float updated_param(float theta, float ratio, const UpdateArgs& u) {
  const float upd = u.lr * ratio;
  const float dec = theta * u.decay;
  return dec - upd;
}

// Codes of the second moment: the number of thresholds at or below rho = v/blockmax, as one subtraction and one shift
// of rho's bit pattern (see stq_tables.h).  The subtrahend is the same for every mantissa at widths up to 4; wider
// codes look it up by the top five mantissa bits (32 words: a wave's reads never meet in a bank).
template <int ROWS, bool TAIL>
__device__ __forceinline__ void quantize_v(const float (&v)[4 * ROWS], uint32_t (&code)[4 * ROWS], const float (&inv)[ROWS], uint32_t b,
                                           const uint32_t* vq, uint32_t q, int lane, uint32_t n_valid) {
  constexpr int N = 4 * ROWS;
  const uint32_t sh = 27u - b;
  if (b <= 4) {
    const uint32_t D = b == 4 ? kVqConst4 : (b == 3 ? kVqConst3 : kVqConst2);
#pragma unroll
    for (int n = 0; n < N; ++n) code[n] = __builtin_elementwise_sub_sat(f2u(v[n] * inv[n >> 2]), D) >> sh;
  } else {
    const char* D = reinterpret_cast<const char*>(vq + (b - kMinBits) * kVqBuckets);
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const uint32_t bits = f2u(v[n] * inv[n >> 2]);
      const uint32_t d = *reinterpret_cast<const uint32_t*>(D + ((bits >> (kVqShift - 2)) & (4u * (kVqBuckets - 1))));
      code[n] = __builtin_elementwise_sub_sat(bits, d) >> sh;
    }
  }
  if (TAIL) {
#pragma unroll
    for (int n = 0; n < N; ++n)
      if (!is_valid<ROWS>(n, q, lane, n_valid)) code[n] = 0u;
  }
}

// The parameter update from the quantized moments (mq: values of the first, code: codes of the second moment).  It needs
// den = sqrt(vq*ibc2) + eps of the quantized value vq, which takes only 2^b values per block:
//  kDenTable: den and 1/den come from the wave's table TAB of (den, 1/den), indexed by (row, block, code) (without FAST
//          1/den is not there);
//  kRoots: two octaves of v further down the root is half as large, so a table of the roots of the lowest two octaves'
//          levels holds them all; TAB keeps, per (row, block, code mod P), the root's bits less (code mod P) << (26-b),
//          and the root of code c is that plus c << (26-b): its exponent counts the whole multiples of P;
//  kDirect: from the level itself with the IEEE routines, when a scale is out of the range the short forms need and there
//          is no table of den.
// FAST: the short form of the quotient, else the IEEE division.
// (Vector instructions per parameter on a 3.5 G-parameter launch at widths 4..8 and 3..6, K = 64: 51.5.  What these forms and
// quantize_v gave was measured when a wave took whole tiles: 58.8 instructions, with IEEE-shaped expansions and a 514-entry
// search table 67.3; 2.4 M parameters, which stay in the caches, 8.7 us instead of 9.4, and the large launch, which the memory
// system bounds, as before.  A den table of twice the entries, for levels that serve two elements, changed nothing then.)
enum UpdateKind { kDenTable, kRoots, kDirect };
template <int KIND, bool FAST, int ROWS>
__device__ __forceinline__ void update_params(const float (&mq)[4 * ROWS], const uint32_t (&code)[4 * ROWS], float (&theta)[4 * ROWS],
                                              const uint32_t* TAB, const uint32_t (&row)[ROWS], uint32_t b, const float (&sn)[ROWS],
                                              const float* Lreg, const UpdateArgs& u) {
  const uint32_t below = b > 3 ? (1u << (b - 3)) - 1u : 0u;  // P - 1 (kRoots)
#pragma unroll
  for (int n = 0; n < 4 * ROWS; ++n) {
    const int i = n >> 2;
    const float mt = mq[n] * u.ibc1;
    float den, rden = 0.0f;
    if (KIND == kDenTable) {
      const float2 dr = reinterpret_cast<const float2*>(TAB)[row[i] + code[n]];
      den = dr.x;
      rden = dr.y;
    } else if (KIND == kRoots) {
      den = u2f((code[n] << (26u - b)) + TAB[row[i] + (code[n] & below)]) + u.eps;
      if (FAST) rden = rcp_rn_safe(den);
    } else {
      const float vq = sn[i] * lds_at(Lreg, (code[n] << 2) | (4u << b));
      den = __builtin_sqrtf(vq * u.ibc2) + u.eps;
    }
    theta[n] = updated_param(theta[n], FAST ? div_rn_safe(mt, den, rden) : mt / den, u);
  }
}

// ------------------------------------------------------------------ one part of a tile
// ROWS rows, a quarter (2) or a half (4) of the tile.  The 2*ROWS (state, row) pairs belong to 64/(2*ROWS) lanes each:
// lane L owns a block scale of pair vL, state = vL / ROWS, row = ROWS*q + vL % ROWS, as the qL-th of the pair's lanes; it
// stands for 2*ROWS lanes of the row, 8*ROWS elements.  A block's owners are K/(8*ROWS), i.e. 2 to 16, neighbouring lanes
// of one 16-lane row, so their maxima combine by DPP lane swaps.
// bfloat16 rounding (to nearest, ties to even) of a finite float, kept as a float
__device__ __forceinline__ float bf16_rne(float x) {
  uint32_t u = f2u(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u2f(u & 0xFFFF0000u);
}

// MODE 0: widths stay as they are; 1: the launch changes widths (other destination buffers);
// 2: as 1, and states may have the wide formats: 32 bits = the fp32 value, 16 bits = its bfloat16
// rounding, stored in the same tile format with 32- or 16-bit codes and without scales.
template <bool BF16, int STATS, bool TAIL, int MODE, int ROWS, bool THROUGH>
__device__ __forceinline__ void process_part(const TensorDesc& d, uint32_t tile, uint32_t q, uint32_t n_valid,
                                             const StepArgs& a, const uint32_t* lds, uint32_t* ws, int lane,
                                             LaneStats<STATS>& st) {
  // Everything derived from the lane index and the block size is cheap to recompute.  Hide the two
  // from loop-invariant code motion, which would otherwise keep dozens of such values live across
  // the whole tile loop and spill them.
  asm volatile("" : "+v"(lane));
  uint32_t lgK = a.lgK;
  asm volatile("" : "+s"(lgK), "+s"(q));
  constexpr bool XW = MODE >= 1, WIDE = MODE == 2;
  typedef Part<ROWS> P_;
  constexpr int N = P_::kElems;
  const uint32_t bm = d.bm, bv = d.bv;              // widths of the stored codes
  // widths this step writes: the same, unless the launch changes widths (XW)
  const uint32_t bmo = XW ? d.bm_out : bm, bvo = XW ? d.bv_out : bv;
  const size_t e0 = static_cast<size_t>(tile) * kTile + 256u * ROWS * q;
  STQ_GLOBAL float* P = as_global(d.param + e0);
  // the part's first bit: bit s0 of word first_word of the lane's b words
  auto first_bit = [&](uint32_t b) { return (4u * ROWS * q * b) & 31u; };
  auto first_word = [&](uint32_t b) { return ((4u * ROWS * q * b) >> 5) * 64u; };
  const uint32_t s0m = first_bit(bm), s0v = first_bit(bv);
  STQ_GLOBAL uint32_t* CM = as_global(d.m_codes + static_cast<size_t>(tile) * 64u * bm) + first_word(bm);
  STQ_GLOBAL uint32_t* CV = as_global(d.v_codes + static_cast<size_t>(tile) * 64u * bv) + first_word(bv);
  // where the new codes go: the same buffers at the same widths, or other buffers at the new widths
  const uint32_t s0mo = first_bit(bmo), s0vo = first_bit(bvo);
  STQ_GLOBAL uint32_t* CMO = XW ? as_global(d.m_out + static_cast<size_t>(tile) * 64u * bmo) + first_word(bmo) : CM;
  STQ_GLOBAL uint32_t* CVO = XW ? as_global(d.v_out + static_cast<size_t>(tile) * 64u * bvo) + first_word(bvo) : CV;
  const size_t sbase = static_cast<size_t>(tile) << (11 - lgK);  // scales per tile = 2048/K
  // the lane index as a 6-bit unsigned offset: global addresses become uniform base + 32-bit offset
  const uint32_t ul = static_cast<uint32_t>(lane) & 63u;
  constexpr int kLgOwners = 6 - P_::kLgPairs, kLgSpan = P_::kLgPairs + 2;  // lanes of a pair; elements an owner stands for
  const int vL = lane >> kLgOwners, qL = lane & ((1 << kLgOwners) - 1);
  const uint32_t sidx = ((ROWS * q + static_cast<uint32_t>(vL & (ROWS - 1))) << (8 - lgK)) + (static_cast<uint32_t>(qL) >> (lgK - kLgSpan));
  STQ_GLOBAL float* SC = as_global((vL >> P_::kLgRows) ? d.v_scales : d.m_scales);

  // ---- loads for the moment phase --------------------------------------------
  const float sc_old = SC[sbase + sidx];
  // (a quarter of 7-bit codes may touch three words, a half four; a part of a wide state is N/2 or N whole words)
  constexpr int kMaxWords = WIDE ? N : (ROWS == 2 ? 3 : 4);
  uint32_t lwm[kMaxWords], lwv[kMaxWords];
  {
    const uint32_t nwm = (s0m + N * bm + 31u) >> 5, nwv = (s0v + N * bv + 31u) >> 5;
#pragma unroll
    for (int k = 0; k < kMaxWords; ++k) lwm[k] = (static_cast<uint32_t>(k) < nwm) ? CM[k * 64u + ul] : 0u;
#pragma unroll
    for (int k = 0; k < kMaxWords; ++k) lwv[k] = (static_cast<uint32_t>(k) < nwv) ? CV[k * 64u + ul] : 0u;
  }
  float g[N];
  {
    STQ_GLOBAL const float* G32 = as_global(static_cast<const float*>(d.grad) + e0);
    STQ_GLOBAL const uint16_t* G16 = as_global(static_cast<const uint16_t*>(d.grad) + e0);
    if (!TAIL) {
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        if (BF16) {
          const u32x2 r = __builtin_nontemporal_load(&reinterpret_cast<STQ_GLOBAL const u32x2*>(G16 + 256 * i)[ul]);
          g[4 * i + 0] = u2f(r.x << 16); g[4 * i + 1] = u2f(r.x & 0xFFFF0000u);
          g[4 * i + 2] = u2f(r.y << 16); g[4 * i + 3] = u2f(r.y & 0xFFFF0000u);
        } else {
          const f32x4 r = __builtin_nontemporal_load(&reinterpret_cast<STQ_GLOBAL const f32x4*>(G32 + 256 * i)[ul]);
          g[4 * i + 0] = r.x; g[4 * i + 1] = r.y; g[4 * i + 2] = r.z; g[4 * i + 3] = r.w;
        }
      }
    } else {
#pragma unroll
      for (int n = 0; n < N; ++n) {
        float x = 0.0f;
        if (is_valid<ROWS>(n, q, lane, n_valid)) {
          const uint32_t idx = 256u * (n >> 2) + 4u * ul + (n & 3);
          x = BF16 ? u2f(static_cast<uint32_t>(G16[idx]) << 16) : G32[idx];
        }
        g[n] = x;
      }
    }
  }

  // old scales to every lane that needs them: lane j reads the values of its lane group
  float* wsf = reinterpret_cast<float*>(ws);
  float* XR = wsf;                          // [kPairs][XS]
  float* SO = wsf + P_::kTableWords;        // [64] old scales at [lane group * kPairs + pair]
  float* SN = SO + 64;                      // [64] new scales
  float* SI = SN + 64;                      // [64] reciprocals of the new scales
  SO[qL * P_::kPairs + vL] = sc_old;
  wave_lds_sync();
  // the values of state `state` (0 first, 1 second moment) at the lane's blocks, from one of these arrays
  auto of_rows = [&](const float* S, int state, float (&x)[ROWS]) {
    const float* at = S + (lane >> P_::kLgPairs) * P_::kPairs + state * ROWS;
    if (ROWS == 2) {
      const float2 y = *reinterpret_cast<const float2*>(at);
      x[0] = y.x; x[1] = y.y;
    } else {
      const float4 y = *reinterpret_cast<const float4*>(at);
      x[0] = y.x; x[1] = y.y; x[ROWS - 2] = y.z; x[ROWS - 1] = y.w;
    }
  };
  float som[ROWS], sov[ROWS];
  of_rows(SO, 0, som);
  of_rows(SO, 1, sov);

  if (STATS) {
    double sg_sum = 0.0, sg_abs = 0.0, sg_sq = 0.0;  // fp64 from the first addition (pads are zeros)
    float sg_max = 0.0f;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const double gd = static_cast<double>(g[n]);
      sg_sum += gd;
      sg_abs += __builtin_fabs(gd);
      sg_sq = __builtin_fma(gd, gd, sg_sq);
      sg_max = fmaxf(sg_max, fabsf(g[n]));
    }
    st.add_grad(kLGSum, lane, sg_sum);
    st.add_grad(kLGAbs, lane, sg_abs);
    st.add_grad(kLGSq, lane, sg_sq);
    st.max_grad(lane, sg_max);
  }

  // ---- moments: m_t = beta1*m_{t-1} + (1-beta1)*g ; v_t = beta2*v_{t-1} + (1-beta2)*g^2 ----
  const float* Rreg = reinterpret_cast<const float*>(lds) + kTabROff;  // value tables, see stq_tables.h
  const float* Lreg = reinterpret_cast<const float*>(lds) + kTabLOff;
  float m[N], v[N];
  {
    uint32_t off[N];
    float old[N];  // the stored moments m_{t-1}, then v_{t-1}
    if (WIDE && bm >= 16) {
#pragma unroll
      for (int n = 0; n < N; ++n)
        old[n] = bm == 32 ? u2f(lwm[n]) : u2f((n & 1) ? (lwm[n >> 1] & 0xFFFF0000u) : (lwm[n >> 1] << 16));
    } else {
      const float* R = Rreg + (1u << bm);
      STQ_SWITCH_BITS(bm, (unpack_offsets<ROWS, B>(lwm, s0m, off)));
#pragma unroll
      for (int n = 0; n < N; ++n) old[n] = som[n >> 2] * lds_at(R, off[n]);
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const float x = a.beta1 * old[n], y = a.omb1 * g[n];
      m[n] = x + y;
    }
    if (WIDE && bv >= 16) {
#pragma unroll
      for (int n = 0; n < N; ++n)
        old[n] = bv == 32 ? u2f(lwv[n]) : u2f((n & 1) ? (lwv[n >> 1] & 0xFFFF0000u) : (lwv[n >> 1] << 16));
    } else {
      const float* L = Lreg + (1u << bv);
      STQ_SWITCH_BITS(bv, (unpack_offsets<ROWS, B>(lwv, s0v, off)));
#pragma unroll
      for (int n = 0; n < N; ++n) old[n] = sov[n >> 2] * lds_at(L, off[n]);
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const float gg = g[n] * g[n];
      const float x = a.beta2 * old[n], y = a.omb2 * gg;
      v[n] = x + y;
    }
  }
  if (TAIL) {
#pragma unroll
    for (int n = 0; n < N; ++n)
      if (!is_valid<ROWS>(n, q, lane, n_valid)) { m[n] = 0.0f; v[n] = 0.0f; }
  }

  if (STATS == 1) {
    // the moments' sums and sums of squares, taken here where few other values are live (their quantization
    // errors follow in the quantizer loops)
    double sm_sum = 0.0;
    float sm_sq[ROWS / 2] = {}, sv_sum[ROWS / 2] = {}, sv_sq[ROWS / 2] = {};
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int p = n >> 3;
      sm_sum += static_cast<double>(m[n]);
      sm_sq[p] = __builtin_fmaf(m[n], m[n], sm_sq[p]);
      sv_sum[p] += v[n];
      sv_sq[p] = __builtin_fmaf(v[n], v[n], sv_sq[p]);
    }
    st.add(kLMSum, lane, sm_sum);
    st.add(kLMSq, lane, sm_sq);
    st.add(kLVSum, lane, sv_sum);
    st.add(kLVSq, lane, sv_sq);
  }

  // ---- parameters: issued here so that they arrive while the block maxima are reduced ----
  // Parameters and gradients are touched once per step: non-temporal accesses keep them from
  // displacing the code and scale lines in the caches (measured: both the load and the store of
  // the parameters must carry the hint; on the code and scale streams it loses).
  float theta[N];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    if (!TAIL) {
      const f32x4 t = __builtin_nontemporal_load(&reinterpret_cast<STQ_GLOBAL const f32x4*>(P + 256 * i)[ul]);
      theta[4 * i] = t.x; theta[4 * i + 1] = t.y; theta[4 * i + 2] = t.z; theta[4 * i + 3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        theta[4 * i + e] = is_valid<ROWS>(4 * i + e, q, lane, n_valid) ? P[256u * i + 4u * ul + e] : 0.0f;
    }
  }

  // ---- block maxima: lane partials -> LDS transpose -> one owner lane per (state,row,block)
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const float pm = fmaxf(fmaxf(fabsf(m[4 * i]), fabsf(m[4 * i + 1])), fmaxf(fabsf(m[4 * i + 2]), fabsf(m[4 * i + 3])));
    const float pv = fmaxf(fmaxf(v[4 * i], v[4 * i + 1]), fmaxf(v[4 * i + 2], v[4 * i + 3]));
    XR[i * XS + lane] = pm;
    XR[(ROWS + i) * XS + lane] = pv;
  }
  wave_lds_sync();
  // the maxima are non-negative, so they order like their bit patterns: integer max, no NaN handling
  float r;
  {
    uint32_t rb = 0u;
#pragma unroll
    for (int k = 0; k < P_::kPairs; k += 4) {
      const uint4 t0 = *reinterpret_cast<const uint4*>(XR + vL * XS + qL * P_::kPairs + k);
      rb = max(max(max(rb, t0.x), max(t0.y, t0.z)), t0.w);
    }
    if (ROWS == 2) {
      rb = max(rb, dpp_u32<kDppXor1>(rb));
      rb = max(rb, dpp_u32<kDppXor2>(rb));
      if (lgK >= 7) rb = max(rb, dpp_u32<kDppHalfMirror>(rb));
      if (lgK == 8) rb = max(rb, dpp_u32<kDppMirror>(rb));
    } else {
      rb = max(rb, dpp_u32<kDppXor1>(rb));
      if (lgK >= 7) rb = max(rb, dpp_u32<kDppXor2>(rb));
      if (lgK == 8) rb = max(rb, dpp_u32<kDppHalfMirror>(rb));
    }
    r = u2f(rb);
  }
  if (STATS == 1) {
    st.max_moment(lane, r);
  }
  // a block whose maximum is below the smallest normal number is stored as all-zero
  const float sc_new = (r < FLT_MIN) ? 0.0f : r;
  float sc_inv;
  if (__all(static_cast<int>(sc_new == 0.0f) | static_cast<int>(in_safe_range(sc_new)))) {
    sc_inv = (sc_new > 0.0f) ? rcp_rn_safe(sc_new) : 0.0f;
  } else {
    sc_inv = (sc_new > 0.0f) ? 1.0f / sc_new : 0.0f;
  }
  SN[qL * P_::kPairs + vL] = sc_new;
  SI[qL * P_::kPairs + vL] = sc_inv;
  {
    // a wide state has no scales: its owners store nothing
    const bool has_scale = !WIDE || (vL < ROWS ? bmo : bvo) < 16;
    if (has_scale && (static_cast<uint32_t>(qL) & ((1u << (lgK - kLgSpan)) - 1u)) == 0u) SC[sbase + sidx] = sc_new;
  }
  wave_lds_sync();

  // ---- table of den = sqrt(vq*ibc2) + eps and 1/den, or of the roots (see update_params) ----
  // Levels P codes apart (P = 2^(b-3), 1 below b = 4) lie a whole number of octaves pairs apart, so their roots differ by
  // a power of two: one root per (row, block, code mod P), roots = (256*ROWS/K)*P.  When a level serves at least four
  // elements, entries = (256*ROWS/K) << bv_out <= 64*ROWS, the lanes go on to den and its reciprocal; 64/roots lanes share the
  // multiples of a root.  The table takes the place of XR, whose last readers have finished.
  const UpdateArgs ua = {a.ibc1, a.ibc2, a.eps, a.lr, a.decay};
  const bool wide_m = WIDE && bmo >= 16, wide_v = WIDE && bvo >= 16;
  const uint32_t bq = wide_v ? 8u : bvo;
  const bool use_table = !wide_v && ((256u * ROWS >> lgK) << bq) <= P_::kDenEntries;
  const uint32_t lgP = bq > 3 ? bq - 3 : 0, lg_roots = 8u + P_::kLgRows - lgK + lgP;
  // The short forms need every operand in a range where no intermediate underflows or overflows.  The owner lanes
  // check their scales: m~ = (s_m*R)*ibc1 is 0 or at least s_m*ibc1/127, in [2^-85, 2^40] when s_m*ibc1 lies in
  // [2^-78, 2^40]; v~ = (s_v*L)*ibc2 is 0 or at least s_v*ibc2*2^-16, in [2^-96, 2^78] when s_v*ibc2 lies in
  // [2^-80, 2^78], and a root is then at most 2^39.
  int bad_m = 0, bad_v = 0;
  if (vL < ROWS) {
    bad_m = (static_cast<int>(sc_new == 0.0f) | static_cast<int>(f2u(sc_new * a.ibc1) - 0x18800000u <= 0x53800000u - 0x18800000u)) ^ 1;
  } else {
    bad_v = (static_cast<int>(sc_new == 0.0f) | static_cast<int>(f2u(sc_new * a.ibc2) - 0x17800000u <= 0x66800000u - 0x17800000u)) ^ 1;
  }
  // den = root + eps then lies in [2^-70, 2^40]
  const bool eps_ok = f2u(a.eps) - 0x1C800000u <= 0x53000000u - 0x1C800000u;  // (eps > 0)
  bool fast_root = eps_ok && !__any(bad_v);                // the roots (and den) by the short form
  bool fast_m = !__any(bad_m);                             // and, with it, the quotient
  if (__builtin_expect(fast_root && !wide_v, 1)) {
    for (uint32_t e = lane; e < (1u << lg_roots) || (use_table && e < 64u); e += 64) {
      const uint32_t root = e & ((1u << lg_roots) - 1u), i = root & ((1u << lgP) - 1u), rg = root >> lgP;
      const uint32_t rw = rg >> (8 - lgK), blk = rg & ((1u << (8 - lgK)) - 1u);
      const float sv = SN[((blk << (lgK - kLgSpan)) << P_::kLgPairs) + ROWS + rw];
      const float vq = sv * lds_at(Lreg, (i << 2) | (4u << bq));
      const uint32_t s_bits = f2u(sqrt_rn_safe(vq * a.ibc2));
      if (use_table) {
        for (uint32_t h = e >> lg_roots; h < (1u << (bq - lgP)); h += 64u >> lg_roots) {
          // (a root of 0 becomes a number of at most 2^-96 here, which eps >= 2^-70 absorbs)
          const float den = u2f(s_bits + (((h << lgP) << (26u - bq)))) + a.eps;
          reinterpret_cast<float2*>(XR)[(rg << bq) + (h << lgP) + i] = make_float2(den, rcp_rn_safe(den));
        }
      } else {
        reinterpret_cast<uint32_t*>(XR)[root] = s_bits - (i << (26u - bq));
      }
    }
    wave_lds_sync();
  } else if (__builtin_expect(use_table, 0)) {
    // A scale or eps out of the short forms' range (small gradients, an eps such as 1e-30): den by the IEEE routines, still
    // once per level; the quotients take the IEEE division.  (1.5 G parameters, K = 128, 5 bits, bf16 gradients: 3270 us,
    // in range 3116; with a root per element it was 4 % more when a wave took whole tiles.  Where a level serves fewer elements
    // the root is taken per element.)
    for (uint32_t e = lane; e < (256u * ROWS >> lgK) << bq; e += 64) {
      const uint32_t c = e & ((1u << bq) - 1u), rg = e >> bq;
      const uint32_t rw = rg >> (8 - lgK), blk = rg & ((1u << (8 - lgK)) - 1u);
      const float vq = SN[((blk << (lgK - kLgSpan)) << P_::kLgPairs) + ROWS + rw] * lds_at(Lreg, (c << 2) | (4u << bq));
      reinterpret_cast<float2*>(XR)[e] = make_float2(__builtin_sqrtf(vq * a.ibc2) + a.eps, 0.0f);
    }
    wave_lds_sync();
  }

  // ---- linear symmetric quantization of m; m is replaced by its quantized value ----
  if (wide_m) {
    float sm_err[ROWS / 2] = {};
    uint32_t kept[N];
    SafeRange range;  // the elements are not multiples of a block scale: look at each
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const float mq = bmo == 32 ? m[n] : bf16_rne(m[n]);  // pads are 0 and stay 0
      range.add(mq * ua.ibc1);
      if (STATS == 1) {
        const float dd = m[n] - mq;
        sm_err[n >> 3] = __builtin_fmaf(dd, dd, sm_err[n >> 3]);
      }
      m[n] = mq;
      kept[n] = f2u(mq);
    }
    fast_m = __all(range.within(0x15000000u, 0x53800000u));  // 2^-85, 2^40
    if (STATS == 1) st.add(kLMErr, lane, sm_err);
    if (bmo == 32) {
#pragma unroll
      for (int n = 0; n < N; ++n) CMO[n * 64u + ul] = kept[n];
    } else {
#pragma unroll
      for (int k = 0; k < N / 2; ++k) CMO[k * 64u + ul] = (kept[2 * k] >> 16) | (kept[2 * k + 1] & 0xFFFF0000u);
    }
  } else {
    float sn[ROWS], inv[ROWS];
    of_rows(SN, 0, sn);
    of_rows(SI, 0, inv);
    const int qmax = (1 << (bmo - 1)) - 1;
    const float qmaxf = static_cast<float>(qmax);
    // Round half to even by adding 1.5*2^23, which leaves the integer q in the low mantissa bits (|t| <= 127.5); with
    // 2^(b-1) = qmax + 1 added as well (an even number, so the same rounding), they hold code + 1.
    // |m| <= s and 1/s is within half an ulp, so |t| <= qmax*(1 + 2^-22) rounds to at most qmax:
    // the clamp of the quantizer's definition can never act and is left out.
    const float magic = 12582912.0f + static_cast<float>(qmax + 1);
    const uint32_t magic_code = 0x4B400001u;  // bits of (magic + q), less the code
    const uint32_t r_base = (4u << bmo) - 4u * magic_code;
    uint32_t code[N];  // low bits: code + 1
    float sm_err[ROWS / 2] = {};  // sums of squared quantization errors of two rows each
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int i = n >> 2;
      const float t = (m[n] * inv[i]) * qmaxf;
      uint32_t u = f2u(t + magic);
      if (TAIL && !is_valid<ROWS>(n, q, lane, n_valid)) u = magic_code;
      code[n] = u;
      float mq = sn[i] * lds_at(Rreg, (u << 2) + r_base);
      if (STATS == 1) {
        if (TAIL && !is_valid<ROWS>(n, q, lane, n_valid)) mq = 0.0f;
        const float dd = m[n] - mq;
        sm_err[n >> 3] = __builtin_fmaf(dd, dd, sm_err[n >> 3]);
      }
      m[n] = mq;
    }
    if (STATS == 1) st.add(kLMErr, lane, sm_err);
    STQ_SWITCH_BITS(bmo, (pack_store<ROWS, B, true, THROUGH>(code, CMO, s0mo, ul)));
  }

  // ---- logarithmic quantization of v and the parameter update ----
  if (wide_v) {
    float sv_err[ROWS / 2] = {};
    uint32_t kept[N];
    SafeRange range;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const float vq = bvo == 32 ? v[n] : bf16_rne(v[n]);
      if (STATS == 1) {
        const float dd = v[n] - vq;
        sv_err[n >> 3] = __builtin_fmaf(dd, dd, sv_err[n >> 3]);
      }
      kept[n] = f2u(vq);
      v[n] = vq * ua.ibc2;
      range.add(v[n]);
    }
    // The short forms where every element of the wave's part allows them (124 M parameters at widths drawn from
    // {4, 8, 16, 32}: 390 us; 406 with an eps out of range, for which all states take the IEEE routines)
    if (eps_ok && __all(range.within(0x0F800000u, 0x66800000u)) && fast_m) {  // 2^-96, 2^78
#pragma unroll
      for (int n = 0; n < N; ++n) {
        const float den = sqrt_rn_safe(v[n]) + ua.eps;
        theta[n] = updated_param(theta[n], div_rn_safe(m[n] * ua.ibc1, den, rcp_rn_safe(den)), ua);
      }
    } else {
#pragma unroll
      for (int n = 0; n < N; ++n) {
        const float den = __builtin_sqrtf(v[n]) + ua.eps;
        theta[n] = updated_param(theta[n], (m[n] * ua.ibc1) / den, ua);
      }
    }
    if (STATS == 1) st.add(kLVErr, lane, sv_err);
    if (bvo == 32) {
#pragma unroll
      for (int n = 0; n < N; ++n) CVO[n * 64u + ul] = kept[n];
    } else {
#pragma unroll
      for (int k = 0; k < N / 2; ++k) CVO[k * 64u + ul] = (kept[2 * k] >> 16) | (kept[2 * k + 1] & 0xFFFF0000u);
    }
  } else {
    float sn[ROWS], inv[ROWS];
    of_rows(SN, 1, sn);
    of_rows(SI, 1, inv);
    uint32_t code[N];
    quantize_v<ROWS, TAIL>(v, code, inv, bvo, lds + kTabVqOff, q, lane, n_valid);
    if (STATS == 1) {
      float sv_err[ROWS / 2] = {};  // sums of squared quantization errors of two rows each
#pragma unroll
      for (int n = 0; n < N; ++n) {
        float vq = sn[n >> 2] * lds_at(Lreg, (code[n] << 2) | (4u << bvo));
        if (TAIL && !is_valid<ROWS>(n, q, lane, n_valid)) vq = 0.0f;
        const float dd = v[n] - vq;
        sv_err[n >> 3] = __builtin_fmaf(dd, dd, sv_err[n >> 3]);
      }
      st.add(kLVErr, lane, sv_err);
    }
    STQ_SWITCH_BITS(bvo, (pack_store<ROWS, B, false, THROUGH>(code, CVO, s0vo, ul)));
    // first table entry of the lane's two blocks: ((row*G + block) << bv_out, or << lgP for the roots), G = 256/K blocks per row
    const uint32_t lg_row = use_table ? bvo : lgP;
    uint32_t row[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
      row[i] = ((static_cast<uint32_t>(i) << (8 - lgK)) + (static_cast<uint32_t>(lane) >> (lgK - 2))) << lg_row;
    const uint32_t* TAB = ws;
    if (__builtin_expect(!fast_root && !use_table, 0)) update_params<kDirect, false, ROWS>(m, code, theta, TAB, row, bvo, sn, Lreg, ua);
    else if (use_table && fast_root && fast_m) update_params<kDenTable, true, ROWS>(m, code, theta, TAB, row, bvo, sn, Lreg, ua);
    else if (use_table) update_params<kDenTable, false, ROWS>(m, code, theta, TAB, row, bvo, sn, Lreg, ua);
    else if (fast_m) update_params<kRoots, true, ROWS>(m, code, theta, TAB, row, bvo, sn, Lreg, ua);
    else update_params<kRoots, false, ROWS>(m, code, theta, TAB, row, bvo, sn, Lreg, ua);
  }

#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    if (!TAIL) {
      const f32x4 t = {theta[4 * i], theta[4 * i + 1], theta[4 * i + 2], theta[4 * i + 3]};
      if constexpr (THROUGH) store_through(P, 1024 * ROWS, 16u * ul + 1024u * i, t);
      else __builtin_nontemporal_store(t, &reinterpret_cast<STQ_GLOBAL f32x4*>(P + 256 * i)[ul]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (is_valid<ROWS>(4 * i + e, q, lane, n_valid)) P[256u * i + 4u * ul + e] = theta[4 * i + e];
    }
  }
}

// -------------------------------------------------------------- step kernel
// Order of the work.  A unit is a part of a tile: a half (ROWS = 4), or a quarter (ROWS = 2) in launches that halves would
// not fill.  Ticket k stands for the kWaves consecutive units k*kWaves .. k*kWaves + kWaves-1, one per wave of a workgroup.
//  * Drawn (a.sched set): the workgroups draw tickets from counters in device memory and their waves meet at a barrier
//    before they go on to the next one, which was drawn while they worked.  The chip as a whole then sweeps the arrays in
//    order, and the narrower the window in which it works at one time, the more the memory system gives: 1.56 G parameters
//    (bf16 gradients) 3.09 ms with half tiles in one order, 3.36 with whole tiles (tickets twice as long), 3.39 with two
//    half tiles one after the other per draw, 3.82 with every workgroup walking its own tickets.  (Without writing
//    through, which makes 3.05 of the 3.09.)
//    One counter alone is drawn from at most every 12 ns or so, which 512 workgroups starting together feel (9 M
//    parameters: 26.9 us, with eight counters 22.5; 130 M: 268.8 and 266.9; 1.56 G: 3092 and 3120).  The workgroups of a
//    counter have to be spread over the XCDs: with a counter for each XCD, which do not run at the same pace, the classes
//    drift apart (1.56 G: 3590 us).
//  * Else workgroup g takes the tickets g, g + G, ...: launches below 8.4 M parameters (with bf16 gradients or wide states
//    12.6 M; see launch_table), where there is nothing to keep in order.
// With statistics a workgroup's waves keep their sums as long as its tickets start in the same tensor (see StatRecord).
// Counters that start anew by themselves leave nothing to clear: every launch -- also a replayed one -- finds them at zero.
// (A count of the workgroups that have left, with acquire and release, cost 20 us: each one writes back its L2.)
// Why halves: what a part needs besides its elements (addresses, scales, the exchange of maxima, the table of roots, the
// sums of the statistics over the lanes) is a third of a quarter's vector instructions, and one chain of latencies; with
// four rows it is shared by twice the elements, and the waves that 128 registers leave, 16 per CU, keep as many bytes in
// flight.  bf16 gradients, static order: 30 M parameters 73.8 us with quarters, 61.1 with halves; 12.5 M 33.3 and 27.7.
// What bounds it: large launches the memory system (3.5 G parameters, 44.65 GB in 6.98 ms = 6.4 TB/s, where an in-place
// addition of one array reaches 5.9), as do launches of 0.1 G (1.81 GB in 291 us); launches that leave the chip partly
// idle one pass of latencies (tables, descriptor, loads, three LDS exchanges, stores): 6 us for 0.2 M parameters.
// the class of ticket counter that a workgroup belongs to
__device__ __forceinline__ uint32_t class_of(uint32_t group, uint32_t lg_classes) { return (group >> 3) & ((1u << lg_classes) - 1u); }

// What a workgroup needs first comes as arguments of its own, which are in registers when it starts (the build has them
// preloaded; a struct's members would be read from memory first: 25 ragged tensors of 0.2 M elements 6.0 us, now 5.6).
template <bool BF16, int STATS, int MODE, int ROWS, bool THROUGH>
__global__ __launch_bounds__(64 * kWavesPerGroup, ROWS == 4 || MODE == 2 ? 4 : 6) void step_kernel(
    const TensorDesc* desc, const uint32_t* tables, uint32_t* sched, uint32_t n_tensors, uint32_t total_tiles, uint32_t lg_classes,
    const StepArgs a) {
  constexpr int kWaves = kWavesPerGroup;
  constexpr int kWaveScratch = Part<ROWS>::kScratch, kLdsWords = kTabWords + kWaves * kWaveScratch;
  constexpr uint32_t kLgParts = 3u - Part<ROWS>::kLgRows, kParts = 1u << kLgParts;  // of a tile
  __shared__ __attribute__((aligned(16))) uint32_t lds[kLdsWords + kWaves * LaneStats<STATS>::kWords];
  __shared__ uint32_t drawn[2];  // the ticket being worked on and the next one, alternating
  __shared__ StatRecord<STATS> records[kWaves];
  __shared__ uint32_t group_end[2];  // statistics: where the tensor ends that the first unit of the ticket lies in, alternating
  constexpr int kTabLoads = (kTabWords + 64 * kWaves - 1) / (64 * kWaves);  // the tables: 5 KB
  uint32_t tab[kTabLoads];
#pragma unroll
  for (int k = 0; k < kTabLoads; ++k) tab[k] = tables[min(k * 64 * kWaves + static_cast<int>(threadIdx.x), kTabWords - 1)];

  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* ws = lds + kTabWords + wave * kWaveScratch;
  const bool draws = sched != nullptr;
  const uint64_t total_units = static_cast<uint64_t>(total_tiles) << kLgParts;
  const uint32_t n_tickets = static_cast<uint32_t>((total_units + kWaves - 1) / kWaves);
  uint32_t turn = 0;  // which of drawn[] is current
  // Ticket k belongs to class k mod C, each with a counter; so does a workgroup, to one class with its seven neighbours,
  // which are on the other XCDs (C > 1 only if this gives every class as many).  Its first ticket is the one of its own index
  // within the class; the counter hands out those that follow and starts anew after as many draws as the class has
  // tickets: every workgroup draws until it gets a number past the end, one draw for each ticket that it works on.
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  uint32_t cur = blockIdx.x;
  if (draws) cur = ((((blockIdx.x >> 3) >> lg_classes) << 3) + (blockIdx.x & 7u)) << lg_classes | class_of(blockIdx.x, lg_classes);

  // tensor holding the wave's first unit: the table's loads, the search and the first descriptor are in flight together
  uint32_t l = 0, held_l = kNone;  // held_l, with statistics: the tensor that the wave's sums belong to, if it has any
  TensorDesc d;
  if (static_cast<uint64_t>(cur) * kWaves + wave < total_units) {
    l = find_begin(desc, n_tensors, static_cast<uint32_t>((static_cast<uint64_t>(cur) * kWaves + wave) >> kLgParts), lane);
    d = load_desc(desc, l);
  }
#pragma unroll
  for (int k = 0; k < kTabLoads; ++k) {
    const int i = k * 64 * kWaves + static_cast<int>(threadIdx.x);
    if (i < kTabWords) lds[i] = tab[k];
  }
  __syncthreads();

  LaneStats<STATS> st;
  st.acc = STATS ? reinterpret_cast<float*>(lds + kLdsWords + wave * LaneStats<STATS>::kWords) : nullptr;
  if (STATS) {
    st.clear(lane);
  }
  auto slots_of = [&](uint32_t tensor) { return a.stats + static_cast<size_t>(tensor) * kStatSlots; };
  while (cur < n_tickets) {  // the same for every wave of the workgroup
    uint32_t next_ticket = 0;
    if (draws && threadIdx.x == 0) {
      uint32_t group = blockIdx.x;
      asm volatile("" : "+s"(group));  // nothing of this is worth a register throughout the loop
      const uint32_t cls = class_of(group, lg_classes), tickets = (n_tickets + (1u << lg_classes) - 1u - cls) >> lg_classes;
      next_ticket = atomicInc(sched + cls * kSchedStride, tickets - 1u);
    }
    const uint64_t u = static_cast<uint64_t>(cur) * kWaves + wave;
    if (u < total_units) {
      const uint32_t t = static_cast<uint32_t>(u >> kLgParts), q = static_cast<uint32_t>(u) & (kParts - 1u);
      if (t >= d.tile_begin + d.n_tiles) {  // t < total_tiles, so a later tensor holds it
        if (__builtin_expect(a.look_ahead != 0u, 0)) {
          int hidden = lane;
          asm volatile("" : "+v"(hidden));  // no address of the search is worth a register throughout the loop
          uint32_t window, ahead;
          do {  // (on to the next window from the last entry of one; the last of all is a window of one)
            window = min(a.look_ahead, n_tensors - l);
            ahead = find_begin(desc + l, window, t, hidden);
            l += ahead;
          } while (ahead == window - 1u && window > 1u);
          d = load_desc(desc, l);
        } else {
          do {
            ++l;
            d = load_desc(desc, l);
          } while (t >= d.tile_begin + d.n_tiles);
        }
      }
      bool in_group = true;  // the unit lies in the tensor of the ticket's first unit (it cannot lie behind it)
      if (STATS) {
        in_group = static_cast<uint32_t>((u - wave) >> kLgParts) >= d.tile_begin;
        if (!in_group && held_l != kNone) flush_stats(st, slots_of(held_l), lane);
        held_l = in_group ? l : kNone;
      }
      const uint32_t tile = t - d.tile_begin;
      const uint64_t left = d.numel - static_cast<uint64_t>(tile) * kTile;
      if (left >= 256u * ROWS * (q + 1u))
        process_part<BF16, STATS, false, MODE, ROWS, THROUGH>(d, tile, q, kTile, a, lds, ws, lane, st);
      else
        process_part<BF16, STATS, true, MODE, ROWS, THROUGH>(d, tile, q, static_cast<uint32_t>(left), a, lds, ws, lane, st);
      if (STATS) {
        if (!in_group) flush_stats(st, slots_of(l), lane);
        if (wave == 0 && lane == 0) group_end[turn] = d.tile_begin + d.n_tiles;
      }
    }
    if (draws && threadIdx.x == 0) {
      uint32_t group = blockIdx.x;
      asm volatile("" : "+s"(group));
      drawn[turn] = ((gridDim.x >> lg_classes) + next_ticket) << lg_classes | class_of(group, lg_classes);
    }
    if (STATS || draws) __syncthreads();  // the workgroup goes on together
    cur = draws ? __builtin_amdgcn_readfirstlane(drawn[turn]) : cur + gridDim.x;
    if constexpr (STATS != 0) {
      const uint32_t end = __builtin_amdgcn_readfirstlane(group_end[turn]);
      if (cur >= n_tickets || static_cast<uint32_t>(static_cast<uint64_t>(cur) * kWaves >> kLgParts) >= end) {
        record_stats(st, &records[wave], lane);
        held_l = kNone;
        __syncthreads();
        if (wave == 0) flush_records(records, slots_of(l), lane);  // (wave 0 has the first unit of every ticket)
      }
    }
    turn ^= 1u;  // (what the next round leaves goes into the other half: a wave is at most one barrier ahead)
  }
}

}  // namespace

template <int MODE, int STATS, int ROWS, bool THROUGH>
static void launch_grads(const StepWork& w, const StepArgs& a, bool grad_bf16, dim3 grid, dim3 block, hipStream_t s) {
  const auto kernel = grad_bf16 ? step_kernel<true, STATS, MODE, ROWS, THROUGH> : step_kernel<false, STATS, MODE, ROWS, THROUGH>;
  hipLaunchKernelGGL(kernel, grid, block, 0, s, w.desc, w.tables, w.sched, w.n_tensors, w.total_tiles, w.lg_classes, a);
}

template <int MODE, int STATS>
static void launch_variant(const StepWork& w, const StepArgs& a, bool grad_bf16, dim3 grid, dim3 block, hipStream_t s) {
  if (w.unit_rows == 2) {
    launch_grads<MODE, STATS, 2, false>(w, a, grad_bf16, grid, block, s);
  } else {
    if constexpr (STATS != 1) {
      if (w.write_through) {
        launch_grads<MODE, STATS, 4, true>(w, a, grad_bf16, grid, block, s);
        return;
      }
    }
    launch_grads<MODE, STATS, 4, false>(w, a, grad_bf16, grid, block, s);
  }
}

template <int MODE>
static void launch_mode(const StepWork& w, const StepArgs& a, bool grad_bf16, int stats, dim3 grid, dim3 block, hipStream_t s) {
  if (stats == 1) launch_variant<MODE, 1>(w, a, grad_bf16, grid, block, s);
  else if (stats == 2) launch_variant<MODE, 2>(w, a, grad_bf16, grid, block, s);
  else launch_variant<MODE, 0>(w, a, grad_bf16, grid, block, s);
}

// mode: 0 in place at unchanged widths, 1 widths change, 2 as 1 with 16- or 32-bit states
// stats: 0 none, 1 every statistic, 2 the gradient's only
int launch_step(const StepWork& w, const StepArgs& a, bool grad_bf16, int stats, int mode, uint32_t groups, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  const dim3 grid(groups), block(64 * kWavesPerGroup);
  if (mode == 2) launch_mode<2>(w, a, grad_bf16, stats, grid, block, s);
  else if (mode == 1) launch_mode<1>(w, a, grad_bf16, stats, grid, block, s);
  else launch_mode<0>(w, a, grad_bf16, stats, grid, block, s);
  return static_cast<int>(hipGetLastError());
}

}  // namespace stq
