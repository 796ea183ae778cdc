// Host-side tables of the two block quantizers (Section 3.5 of the paper: linear
// symmetric codes for the first moment, logarithmic codes for the second) in the
// form the gfx950 kernels consume.  Pure host code, no HIP.
#pragma once
#include <cstdint>
#include <vector>

namespace stq {

constexpr int kGLen = 511;    // G[j] = fl32(2^(-j/32)), j = 0..510
constexpr int kMinBits = 2;
constexpr int kMaxBits = 8;

// Second-moment quantizer without a search: the thresholds of width b lie 2^(4-b) octaves apart, so the bit
// patterns of the thresholds repeat with every octave (every 2 or 4 octaves for b = 3, 2), 2^(b-4) of them per
// octave.  With D[i] for the mantissa bucket i = bits 18..22 of rho = v / blockmax in (0, 1],
//   code = max(bits(rho) - D[i], 0) >> (27 - b),
// where D places the one threshold of the bucket (if it has one) on a multiple of 2^(27-b); a bucket is 2^18 ulps
// wide, no wider than half a step of the widest code.  For b <= 4 one constant serves every bucket.
constexpr int kVqShift = 18;
constexpr int kVqBuckets = 32;
constexpr uint32_t kVqConst4 = 0x37B504F3u;  // bits of fl32(2^-14.5) less one step of 2^23
constexpr uint32_t kVqConst3 = 0x38000000u;  // bits of 2^-13 less one step of 2^24
constexpr uint32_t kVqConst2 = 0x38800000u;  // bits of 2^-10 less one step of 2^25

// Offsets (in 32-bit words) inside the table image that stq_init uploads and every
// workgroup copies to LDS.
// R_b and L_b start at word (1<<b) of their 512-word regions, so that a code index can be OR-ed
// onto the table's base.
constexpr int kTabROff = 0;     // R_b[u] at kTabROff + (1<<b) + u
constexpr int kTabLOff = 512;   // L_b[c] at kTabLOff + (1<<b) + c
constexpr int kTabVqOff = 1024; // D of width b at kTabVqOff + (b-2)*kVqBuckets
constexpr int kTabWords = kTabVqOff + 7 * kVqBuckets;

float table_G(int j);
float table_R(int b, int u);  // value of first-moment code u at scale 1
float table_L(int b, int c);  // value of second-moment code c at scale 1
float table_T(int b, int k);  // threshold between second-moment levels k and k+1 at scale 1

// Fills `img` (kTabWords words).  Returns false if the form above does not reproduce the thresholds exactly.
bool build_table_image(std::vector<uint32_t>& img);

// Code-domain conversion tables for a width change (scale of the block unchanged).
// state 0: first moment, 1: second moment.  out has 256 entries.
void build_repack_lut(int state, int b_old, int b_new, uint8_t* out);

}  // namespace stq
