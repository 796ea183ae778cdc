// The short root, reciprocal and quotient of the step kernel against 64-bit arithmetic, for tests/test_short_forms.py.
// (A root or quotient of floats rounded to double and then to float is the correctly rounded float: 53 >= 2*24 + 2 bits.)
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>

#include "stq_round.h"

namespace {

struct Result {
  unsigned long long bad;  // how many are wrong
  unsigned int first;      // the least bit pattern (or index) among them
};

__device__ void compare(float got, double want, uint32_t at, Result* r) {
  if (__builtin_bit_cast(uint32_t, got) != __builtin_bit_cast(uint32_t, static_cast<float>(want))) {
    atomicAdd(&r->bad, 1ull);
    atomicMin(&r->first, at);
  }
}

// every bit pattern from lo to hi
template <bool ROOT>
__global__ __launch_bounds__(256) void unary_kernel(uint32_t lo, uint32_t hi, Result* r) {
  const uint64_t step = static_cast<uint64_t>(gridDim.x) * 256;
  for (uint64_t u = lo + static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x; u <= hi; u += step) {
    const float x = __builtin_bit_cast(float, static_cast<uint32_t>(u));
    if (ROOT) compare(stq::sqrt_rn_safe(x), sqrt(static_cast<double>(x)), static_cast<uint32_t>(u), r);
    else compare(stq::rcp_rn_safe(x), 1.0 / static_cast<double>(x), static_cast<uint32_t>(u), r);
  }
}

// `count` pairs from a hash of their index: |n| from 2^-85 to 2^40, either sign, d from 2^-70 to 2^40
__global__ __launch_bounds__(256) void quotient_kernel(uint32_t count, Result* r) {
  const uint64_t step = static_cast<uint64_t>(gridDim.x) * 256;
  for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x; i < count; i += step) {
    uint64_t h = (i + 1) * 0x9E3779B97F4A7C15ull;  // (splitmix64)
    h = (h ^ (h >> 30)) * 0xBF58476D1CE4E5B9ull;
    h = (h ^ (h >> 27)) * 0x94D049BB133111EBull;
    h ^= h >> 31;
    const uint32_t n_bits = 0x15000000u + static_cast<uint32_t>((h & 0xFFFFFFFFu) * (0x53800000u - 0x15000000u + 1ull) >> 32);
    const uint32_t d_bits = 0x1C800000u + static_cast<uint32_t>((h >> 32) * (0x53800000u - 0x1C800000u + 1ull) >> 32);
    const float n = __builtin_bit_cast(float, n_bits | (static_cast<uint32_t>(i & 1u) << 31)), d = __builtin_bit_cast(float, d_bits);
    compare(stq::div_rn_safe(n, d, stq::rcp_rn_safe(d)), static_cast<double>(n) / static_cast<double>(d), static_cast<uint32_t>(i), r);
  }
}

}  // namespace

// which 0: roots of the bit patterns a..b, 1: their reciprocals, 2: b pairs of the quotient.  0 or a HIP error.
extern "C" int short_forms_check(int which, uint32_t a, uint32_t b, uint64_t* bad, uint32_t* first) {
  Result h = {0ull, 0xFFFFFFFFu}, *d = nullptr;
  hipError_t e = hipMalloc(&d, sizeof(Result));
  if (e != hipSuccess) return static_cast<int>(e);
  e = hipMemcpy(d, &h, sizeof(Result), hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    if (which == 0) hipLaunchKernelGGL(unary_kernel<true>, dim3(4096), dim3(256), 0, nullptr, a, b, d);
    else if (which == 1) hipLaunchKernelGGL(unary_kernel<false>, dim3(4096), dim3(256), 0, nullptr, a, b, d);
    else hipLaunchKernelGGL(quotient_kernel, dim3(4096), dim3(256), 0, nullptr, b, d);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpy(&h, d, sizeof(Result), hipMemcpyDeviceToHost);
  (void)hipFree(d);
  *bad = h.bad;
  *first = h.first;
  return static_cast<int>(e);
}

// On the host, over the divisor mantissas D from d_begin to d_end (of [2^23, 2^24)): every quotient of 24-bit numbers N/D
// within max_r / (2 D) units in the last place of the middle between two floats.  With Q the odd number of half units there,
// N 2^s = D Q + R (s = 24 for N >= D, 25 below), and Q = -R D^-1 mod 2^s as far as D is odd.  N and D are scaled by
// 2^en and 2^ed.  Returns the number of wrong quotients, *pairs the number looked at.
extern "C" uint64_t short_forms_quotients(uint32_t d_begin, uint32_t d_end, int max_r, int en, int ed, uint64_t* pairs) {
  uint64_t bad = 0, seen = 0;
  const float sn = ldexpf(1.0f, en - 23), sd = ldexpf(1.0f, ed - 23);
  for (uint32_t D = d_begin; D < d_end; ++D) {
    const int k = __builtin_ctz(D);
    const uint64_t odd = D >> k;
    uint64_t inv = odd;  // of D / 2^k modulo 2^64: correct bits double, from three
    for (int i = 0; i < 5; ++i) inv *= 2 - odd * inv;
    const float d = static_cast<float>(D) * sd, y = 1.0f / d;
    for (int s = 24; s <= 25; ++s) {
      for (int64_t R = -max_r; R <= max_r; ++R) {
        // D Q + R is a multiple of 2^s for an odd Q: 2^k divides R, and an odd number of times
        if (R == 0 || k > 24 || (R & ((int64_t{1} << k) - 1)) != 0 || ((R >> k) & 1) == 0) continue;
        const uint64_t mod = uint64_t{1} << (s - k);
        for (uint64_t Q = (0 - static_cast<uint64_t>(R >> k) * inv) & (mod - 1); Q < (uint64_t{1} << 25); Q += mod) {
          if (Q < (uint64_t{1} << 24)) continue;
          const uint64_t N = (D * Q + static_cast<uint64_t>(R)) >> s;
          if (N < (1u << 23) || N >= (1u << 24) || (N >= D) != (s == 24)) continue;
          const float n = static_cast<float>(N) * sn;
          ++seen;
          if (stq::div_rn_safe(n, d, y) != n / d) ++bad;
        }
      }
    }
  }
  *pairs = seen;
  return bad;
}
