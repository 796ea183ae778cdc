// Host-side table construction for the quantizers of Section 3.5 (see stq_tables.h).
#include "stq_tables.h"

#include <cmath>
#include <cstring>

namespace stq {

static inline uint32_t f2u(float f) { uint32_t u; std::memcpy(&u, &f, 4); return u; }

// One table serves every width: level k of width b is 2^(-k * 2^(4-b)) = G[k << (9-b)] and the
// decision threshold between levels k and k+1 (their geometric mean) is G[(2k+1) << (8-b)].
float table_G(int j) { return static_cast<float>(std::exp2(-static_cast<double>(j) / 32.0)); }

float table_R(int b, int u) {
  const int qmax = (1 << (b - 1)) - 1;
  // quotient of two small integers: the double quotient rounds to the same fp32 as the exact one
  return static_cast<float>(static_cast<double>(u - qmax) / static_cast<double>(qmax));
}

float table_L(int b, int c) { return table_G((((1 << b) - 1) - c) << (9 - b)); }

float table_T(int b, int k) { return table_G((2 * k + 1) << (8 - b)); }

// the code the kernel computes for the bit pattern of rho
static uint32_t vq_code(const std::vector<uint32_t>& img, int b, uint32_t rho_bits) {
  const uint32_t D = img[kTabVqOff + (b - 2) * kVqBuckets + ((rho_bits >> kVqShift) & (kVqBuckets - 1))];
  return rho_bits > D ? (rho_bits - D) >> (27 - b) : 0u;
}

bool build_table_image(std::vector<uint32_t>& img) {
  img.assign(kTabWords, 0u);
  const uint32_t one = f2u(1.0f);
  for (int b = kMinBits; b <= kMaxBits; ++b) {
    const int qmax = (1 << (b - 1)) - 1, kmax = (1 << b) - 1;
    for (int u = 0; u <= 2 * qmax; ++u) img[kTabROff + (1 << b) + u] = f2u(table_R(b, u));
    for (int c = 0; c <= kmax; ++c) img[kTabLOff + (1 << b) + c] = f2u(table_L(b, c));
    std::vector<uint32_t> thr(kmax);  // bit patterns, descending in k; positive floats order like theirs
    for (int k = 0; k < kmax; ++k) thr[k] = f2u(table_T(b, k));
    auto at_or_below = [&](uint32_t x) {  // thresholds at or below x: the code the definition gives
      uint32_t n = 0;
      for (uint32_t t : thr) n += t <= x ? 1u : 0u;
      return n;
    };
    uint32_t* D = &img[kTabVqOff + (b - 2) * kVqBuckets];
    for (int i = 0; i < kVqBuckets; ++i) {
      if (b <= 4) {
        D[i] = b == 4 ? kVqConst4 : (b == 3 ? kVqConst3 : kVqConst2);
        continue;
      }
      // The octave below 1 (threshold k is the lower end of code kmax - k; k grows downwards).  A bucket with a
      // threshold: D puts that threshold on the multiple of its code; one without: its first pattern on its code's.
      const uint32_t lo = one - (1u << 23) + (static_cast<uint32_t>(i) << kVqShift), hi = lo + (1u << kVqShift);
      uint32_t at = lo;
      for (uint32_t t : thr)
        if (t >= lo && t < hi) at = t;
      D[i] = at - (at_or_below(at) << (27 - b));
    }
    // the decisions on both sides of every threshold, at both ends of the range, and at the bucket edges
    for (uint32_t t : thr)
      if (vq_code(img, b, t) != at_or_below(t) || vq_code(img, b, t - 1) != at_or_below(t - 1)) return false;
    if (vq_code(img, b, one) != static_cast<uint32_t>(kmax) || vq_code(img, b, one + 1) != static_cast<uint32_t>(kmax) ||
        vq_code(img, b, 0u) != 0u)
      return false;
    for (uint32_t x = one; x > one - (20u << 23); x -= 1u << kVqShift)
      if (vq_code(img, b, x) != at_or_below(x) || vq_code(img, b, x - 1) != at_or_below(x - 1)) return false;
  }
  return true;
}

void build_repack_lut(int state, int b_old, int b_new, uint8_t* out) {
  std::memset(out, 0, 256);
  if (state == 0) {
    const int qo = (1 << (b_old - 1)) - 1, qn = (1 << (b_new - 1)) - 1;
    for (int u = 0; u <= 2 * qo; ++u) {
      const float t = table_R(b_old, u) * static_cast<float>(qn);
      float r = std::nearbyintf(t);  // half to even in the default rounding mode
      if (r > static_cast<float>(qn)) r = static_cast<float>(qn);
      if (r < -static_cast<float>(qn)) r = -static_cast<float>(qn);
      out[u] = static_cast<uint8_t>(static_cast<int>(r) + qn);
    }
  } else {
    const int ko = (1 << b_old) - 1, kn = (1 << b_new) - 1;
    for (int c = 0; c <= ko; ++c) {
      const float rho = table_L(b_old, c);
      int code = 0;  // number of new thresholds at or below the old level's value
      for (int k = 0; k < kn; ++k) if (rho >= table_T(b_new, k)) ++code;
      out[c] = static_cast<uint8_t>(code);
    }
  }
}

}  // namespace stq
