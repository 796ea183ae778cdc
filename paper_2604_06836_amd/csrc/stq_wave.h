// Device code that the kernels of this library share: global and constant pointers, lane exchange and small reductions
// by DPP, the tensor table.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "stq_device.h"

namespace stq {
namespace {

// Pointers that arrive through the tensor table are loaded from memory, so the compiler cannot
// see that they are global; say so, to get global_load/global_store instead of flat accesses.
#define STQ_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ STQ_GLOBAL T* as_global(T* p) { return (STQ_GLOBAL T*)p; }

__device__ __forceinline__ uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }


// x from the lane that a DPP control word names (all lanes of the wave active)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7-i inside each 8 lanes
constexpr int kDppMirror = 0x140;      // lane i <-> 15-i inside each row of 16 lanes

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint64_t lo = dpp_u32<CTRL>(static_cast<uint32_t>(u)), hi = dpp_u32<CTRL>(static_cast<uint32_t>(u >> 32));
  return __builtin_bit_cast(double, (hi << 32) | lo);
}
// Sums and maxima over groups of 4, 8 or 16 neighbouring lanes, left in every lane of the group.  DPP steps
// only: a shuffle through LDS needs a lane-dependent address register, and the compiler keeps those
// alive across the whole tile loop.
__device__ __forceinline__ double quad_sum(double x) {
  x += dpp_f64<kDppXor1>(x);
  x += dpp_f64<kDppXor2>(x);
  return x;
}
__device__ __forceinline__ double octet_sum(double x) {
  x = quad_sum(x);
  x += dpp_f64<kDppHalfMirror>(x);
  return x;
}
__device__ __forceinline__ double row_sum(double x) {
  x = octet_sum(x);
  x += dpp_f64<kDppMirror>(x);
  return x;
}
__device__ __forceinline__ uint32_t quad_max(uint32_t x) {
  x = max(x, dpp_u32<kDppXor1>(x));
  x = max(x, dpp_u32<kDppXor2>(x));
  return x;
}
__device__ __forceinline__ uint32_t octet_max(uint32_t x) {
  x = quad_max(x);
  return max(x, dpp_u32<kDppHalfMirror>(x));
}
__device__ __forceinline__ uint32_t row_max(uint32_t x) {
  x = octet_max(x);
  return max(x, dpp_u32<kDppMirror>(x));
}

// The descriptor table is never written while a step runs: reading it through the constant
// address space gives scalar loads, so everything derived from a descriptor (all base addresses)
// lives in scalar registers.
#define STQ_CONSTANT __attribute__((address_space(4)))
__device__ __forceinline__ TensorDesc load_desc(const TensorDesc* table, uint32_t l) {
  const STQ_CONSTANT uint64_t* p = (const STQ_CONSTANT uint64_t*)(table + l);
  static_assert(sizeof(TensorDesc) == 96, "descriptor layout");
  uint64_t w[sizeof(TensorDesc) / 8];
#pragma unroll
  for (size_t i = 0; i < sizeof(TensorDesc) / 8; ++i) w[i] = p[i];
  TensorDesc d;
  __builtin_memcpy(&d, w, sizeof(TensorDesc));
  return d;
}
// The entry (tensor or job) that holds tile t: the last l with tile_begin <= t (tile_begin ascends from 0, t < total_tiles).
// The wave looks at 64 entries at a time, so a table of up to 4096 entries takes two loads one after the other.
template <class T>
__device__ __forceinline__ uint32_t find_begin(const T* table, uint32_t n, uint32_t t, uint32_t lane) {
  uint32_t lo = 0;
  for (uint32_t left = n; left > 1;) {
    const uint32_t step = (left + 63u) >> 6, i = lane * step;
    const uint32_t begin = i < left ? as_global(&table[lo + i].tile_begin)[0] : 0xFFFFFFFFu;
    const uint32_t at = static_cast<uint32_t>(__popcll(__ballot(i < left && begin <= t))) - 1u;
    lo += at * step;
    left = min(step, left - at * step);
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

}  // namespace
}  // namespace stq
