// Small gfx950 kernels around the quantized Adam step: the initial state m_0 = v_0 = 0 of
// Algorithm 1, the conversion of stored codes when a layer's bit-width changes, the statistics of the
// gradients alone, uploads of small tables, and a fill.
// The step kernel itself is in stq_step.hip.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <utility>

#include "stq_device.h"
#include "stq_tables.h"
#include "stq_wave.h"

#pragma clang fp contract(off)

namespace stq {
namespace {

// ------------------------------------------------------- initial state kernel
// m_0 = v_0 = 0: first-moment codes hold the zero code qmax (pad elements 0), second-moment
// codes and all scales are 0.  One thread per (tile, lane).
__global__ __launch_bounds__(256) void zero_kernel(const ZeroArgs a) {
  const uint64_t gid = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x;
  const uint64_t tile = gid >> 6;
  const uint32_t lane = gid & 63;
  if (tile >= a.n_tiles) return;
  const uint32_t qmax = a.bm >= 16 ? 0u : (1u << (a.bm - 1)) - 1u;  // a 16- or 32-bit state stores +0.0
  for (uint32_t p = 0; p < a.bm; ++p) {
    uint32_t word = 0;
    for (uint32_t n = 0; n < 32; ++n) {
      const uint64_t idx = tile * kTile + 256 * (n >> 2) + 4 * lane + (n & 3);
      const uint32_t code = idx < a.numel ? qmax : 0u;
      const uint32_t bit = n * a.bm;               // stream position of the code
      const int rel = static_cast<int>(bit) - static_cast<int>(32 * p);
      if (rel >= 32 || rel + static_cast<int>(a.bm) <= 0) continue;
      word |= rel >= 0 ? (code << rel) : (code >> (-rel));
    }
    a.m_codes[tile * 64 * a.bm + p * 64 + lane] = word;
  }
  for (uint32_t p = 0; p < a.bv; ++p) a.v_codes[tile * 64 * a.bv + p * 64 + lane] = 0u;
  if (lane < a.scales_per_tile) {
    a.m_scales[tile * a.scales_per_tile + lane] = 0.0f;
    a.v_scales[tile * a.scales_per_tile + lane] = 0.0f;
  }
}

// --------------------------------------------------------------- re-pack kernel
// Width change of stored states: every code goes through a 256-entry table; pad codes stay 0.
// The lane's 32 codes of width B out of / into its B stream words; all shifts are compile-time.
// Bits [SH, SH+B) of x in one instruction (from the plain expression the compiler makes a shift and a mask).
template <int SH, int B>
__device__ __forceinline__ uint32_t bit_field(uint32_t x) {
  uint32_t r;
  asm("v_bfe_u32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "n"(SH), "n"(B));
  return r;
}
// code N of a lane's stream words
template <int B, int N>
__device__ __forceinline__ uint32_t extract(const uint32_t (&w)[8]) {
  constexpr int off = N * B, p = off >> 5, sh = off & 31;
  if constexpr (sh + B <= 32) {
    return bit_field<sh, B>(w[p]);
  } else {  // a code that straddles two words: align it first
    return bit_field<0, B>(__builtin_amdgcn_alignbit(w[p + 1], w[p], static_cast<uint32_t>(sh)));
  }
}
template <int B, int... N>
__device__ __forceinline__ void extract_all(const uint32_t (&w)[8], uint32_t (&code)[32], std::integer_sequence<int, N...>) {
  ((code[N] = extract<B, N>(w)), ...);
}
template <int B, bool ONCE>
__device__ __forceinline__ void load_words(const STQ_GLOBAL uint32_t* src, uint32_t (&w)[8]) {
#pragma unroll
  for (int p = 0; p < B; ++p) w[p] = ONCE ? __builtin_nontemporal_load(src + 64 * p) : src[64 * p];
}
template <int B>
__device__ __forceinline__ void unpack32(const uint32_t (&w)[8], uint32_t (&code)[32]) {
  extract_all<B>(w, code, std::make_integer_sequence<int, 32>{});
}

template <int B>
__device__ __forceinline__ void pack32(const uint32_t (&code)[32], STQ_GLOBAL uint32_t* dst) {
  uint32_t w[B];
#pragma unroll
  for (int p = 0; p < B; ++p) w[p] = 0u;
#pragma unroll
  for (int n = 0; n < 32; ++n) {
    const int off = n * B, p = off >> 5, sh = off & 31;
    if (sh == 0) w[p] = code[n]; else w[p] |= code[n] << sh;
    if (sh + B > 32) w[p + 1] = code[n] >> (32 - sh);  // first bits of the next word
  }
#pragma unroll
  for (int p = 0; p < B; ++p) __builtin_nontemporal_store(w[p], dst + 64 * p);
}

#define STQ_SWITCH_WIDTH(bits, CALL)       \
  switch (bits) {                          \
    case 2: { constexpr int B = 2; CALL; } break; \
    case 3: { constexpr int B = 3; CALL; } break; \
    case 4: { constexpr int B = 4; CALL; } break; \
    case 5: { constexpr int B = 5; CALL; } break; \
    case 6: { constexpr int B = 6; CALL; } break; \
    case 7: { constexpr int B = 7; CALL; } break; \
    default: { constexpr int B = 8; CALL; } break; \
  }

// The job table is not written while the kernel runs: reading it through the constant address
// space gives scalar loads.
__device__ __forceinline__ RepackJob load_job(const RepackJob* table, uint32_t j) {
  const STQ_CONSTANT uint64_t* p = (const STQ_CONSTANT uint64_t*)(table + j);
  static_assert(sizeof(RepackJob) == 48, "job layout");
  uint64_t w[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) w[i] = p[i];
  RepackJob r;
  __builtin_memcpy(&r, w, sizeof(RepackJob));
  return r;
}
// Many width changes in one launch.  One wave per workgroup and `chunk` consecutive tiles of the launch-wide tile order
// per wave: handed out by the hardware in order, the waves at work at one time stay closer together than persistent ones.
// When a wave enters a job with another conversion table it reloads its table.  The table sits at LDS address 0 as 256 bytes (new codes have at most 8 bits), so
// an old code is the address of its new code as it comes out of the bit-field extraction: one vector
// instruction per code to unpack, none to look up, one to pack -- the kernel moves (b_old + b_new)/8 bytes per
// element and is bound by the memory system: the writes, which nothing here touches again, carry the non-temporal hint,
// so do the reads of a launch too large for the caches (ONCE, see launch_repack_many), and the loads of two tiles are in
// flight before the first of them is converted.
// (2.85 GB of codes of 1.56 G parameters: 523 us with chunks of 4 tiles, 541 with 2, 540 with 8, 772 with 1; 580 with
// persistent waves that took a tile at a time without the hint.)
template <bool ONCE>
__global__ __launch_bounds__(64) void repack_many_kernel(const RepackManyArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lut[256];  // the kernel's only LDS variable: address 0
  const uint32_t lane = threadIdx.x;
  const uint64_t n_waves = gridDim.x;
  uint64_t base = static_cast<uint64_t>(blockIdx.x) * a.chunk;
  if (base >= a.total_tiles) return;
  uint32_t j = find_begin(a.jobs, a.n_jobs, static_cast<uint32_t>(base), lane), loaded = 0xFFFFFFFFu;
  RepackJob job = load_job(a.jobs, j);
  // one tile of `job` from its words to its destination
  auto convert = [&](const uint32_t (&w)[8], uint32_t tile) {
    uint32_t code[32];
    STQ_SWITCH_WIDTH(job.b_old, (unpack32<B>(w, code)));
#pragma unroll
    for (int n = 0; n < 32; ++n) code[n] = lut[code[n]];
    const uint64_t left = job.numel - static_cast<uint64_t>(tile) * kTile;
    if (left < static_cast<uint64_t>(kTile)) {  // ragged last tile: pad codes are 0
      const uint32_t n_valid = static_cast<uint32_t>(left);
      // (the element offsets are computed here, where they are needed: derived from the plain lane index
      // they would be hoisted out of the loops and occupy two dozen registers throughout)
      uint32_t first = 4u * lane;
      asm volatile("" : "+v"(first));
#pragma unroll
      for (int n = 0; n < 32; ++n)
        if (256u * (n >> 2) + first + (n & 3) >= n_valid) code[n] = 0u;
    }
    STQ_GLOBAL uint32_t* dst = (STQ_GLOBAL uint32_t*)(job.dst + static_cast<size_t>(tile) * 64 * job.b_new + lane);
    STQ_SWITCH_WIDTH(job.b_new, (pack32<B>(code, dst)));
  };
  for (; base < a.total_tiles; base += n_waves * a.chunk) {
    const uint32_t c_end = static_cast<uint32_t>(min(base + a.chunk, static_cast<uint64_t>(a.total_tiles)));
    for (uint32_t t = static_cast<uint32_t>(base); t < c_end;) {
      while (t >= job.tile_begin + job.n_tiles) job = load_job(a.jobs, ++j);  // t < total_tiles: a later job holds it
      const uint32_t which = job.lut;
      const uint32_t tile = t - job.tile_begin;
      const bool two = t + 1u < c_end && tile + 1u < job.n_tiles;
      const STQ_GLOBAL uint32_t* src = (const STQ_GLOBAL uint32_t*)(job.src + static_cast<size_t>(tile) * 64 * job.b_old + lane);
      uint32_t w0[8], w1[8];
      if (two) STQ_SWITCH_WIDTH(job.b_old, (load_words<B, ONCE>(src, w0), load_words<B, ONCE>(src + 64 * B, w1)))
      else STQ_SWITCH_WIDTH(job.b_old, (load_words<B, ONCE>(src, w0)))
      if (loaded != which) {
        __builtin_amdgcn_wave_barrier();  // the previous tile's table reads are done (same wave, in order)
        // lane k packs entries 4k .. 4k+3 of the word table in device memory into one LDS word
        const uint4 e = *reinterpret_cast<const uint4*>(a.luts + which * 256 + 4 * lane);
        reinterpret_cast<uint32_t*>(lut)[lane] = e.x | (e.y << 8) | (e.z << 16) | (e.w << 24);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        loaded = which;
      }
      convert(w0, tile);
      if (two) convert(w1, tile + 1u);
      t += two ? 2u : 1u;
    }
  }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t* p, uint64_t words) {
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < words) p[i] = 0u;
}

// A table from pinned host memory to the device.  A kernel: a copy goes to another engine and back, between two kernels of
// the stream (re-packs of 7 M elements 13.2 us, now 10.0; of 1.56 G, 0.5 ms, no more than two runs differ).
__global__ __launch_bounds__(256) void upload_kernel(uint4* dst, const uint4* pinned, uint64_t n) {
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) dst[i] = pinned[i];
}

// The same with the table in the launch's own arguments, for a launch that is recorded into a graph: a replay finds them
// unchanged, where a staging slot would by then hold a later call's table.
struct UploadChunk {
  uint4 part[240];  // (3840 bytes: a launch takes 4096 bytes of arguments)
};
constexpr uint64_t kChunkParts = sizeof(UploadChunk) / sizeof(uint4);
static_assert(kChunkParts <= 256, "a thread for each");
__global__ __launch_bounds__(256) void upload_by_value_kernel(uint4* dst, uint32_t n, const UploadChunk chunk) {
  if (threadIdx.x < n) dst[threadIdx.x] = chunk.part[threadIdx.x];
}

// --------------------------------------------------- gradient statistics kernel
// The per-layer sums the bit-width decision reads (Eq. 2, 3, 8: sum g, sum |g|, sum g^2) and max |g|,
// from the gradients alone: for the order in which Algorithm 1 is written, where the decision of step t
// precedes that step's layer loop.  One read of the gradients, and bound by it as long as the sums do not wait for each
// other: a workgroup takes one contiguous range of tiles, its eight waves in turn, with the next tile's loads in flight
// while a tile is added up; a lane keeps fp64 totals; what the waves hold at the end goes to the layer's accumulators
// by one set of atomics per workgroup.
// With read-back and decision, us: 0.12 G bf16 gradients in 148 tensors 78.5 before, now 75.5, 30 M fp32 in one tensor 42.5 and
// 38.8, 400 ragged tensors of up to 0.4 M 98 and 93.5, for three changes together: the atomics of a workgroup's three sums were
// an instruction each (see add_grad_sums), one lane added up the waves' sums, and a ragged tile was read element by element.  (Two tiles in
// flight, with 16-byte loads: the same there, but 1.5 G bf16 gradients 482 where this takes 462; one set of atomics per
// wave, 8192 of them on the same words, 127 for 0.12 G.)
struct GradSums {
  double sum, abs, sq;
  float top;
};

// over the wave; complete in every lane
__device__ __forceinline__ GradSums wave_sums(GradSums s) {
  s.sum = row_sum(s.sum);
  s.abs = row_sum(s.abs);
  s.sq = row_sum(s.sq);
  uint32_t top = row_max(f2u(s.top));  // non-negative floats order like their bit patterns
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    s.sum += __shfl_xor(s.sum, o, 64);
    s.abs += __shfl_xor(s.abs, o, 64);
    s.sq += __shfl_xor(s.sq, o, 64);
    top = max(top, static_cast<uint32_t>(__shfl_xor(static_cast<int>(top), o, 64)));
  }
  s.top = u2f(top);
  return s;
}

// Sums that every lane holds -> the tensor's accumulators, by one instruction for the three sums: what adds to the same
// cache line at the same time is taken in turn, whatever the number of an instruction's lanes.  256 workgroups, us above an empty
// launch: one instruction each 1.9, these two 2.0, one lane adding four values one after the other 11.1.
__device__ __forceinline__ void add_grad_sums(double* slot, const GradSums& s, int lane) {
  static_assert(kGAbsSum == kGSum + 1 && kGSqSum == kGSum + 2, "neighbours");
  const double x = lane == 0 ? s.sum : (lane == 1 ? s.abs : s.sq);
  if (lane < 3) atomicAdd(&slot[kGSum + lane], x);
  if (lane == 3) atomicMax(reinterpret_cast<uint32_t*>(&slot[kMaxGM]), f2u(s.top));
}

typedef uint32_t gs_u32x2 __attribute__((ext_vector_type(2)));
typedef float gs_f32x4 __attribute__((ext_vector_type(4)));
template <bool BF16>
struct GradRow {  // four neighbouring gradients
  typedef gs_f32x4 type;
};
template <>
struct GradRow<true> {
  typedef gs_u32x2 type;
};

__device__ __forceinline__ void add_grad(GradSums& s, float g) {
  // fp64 from the first addition: the decision compares scores with thresholds, and the variance of Eq. 3
  // is a difference of two of these sums
  const double gd = static_cast<double>(g);
  s.sum += gd;
  s.abs += __builtin_fabs(gd);
  s.sq = __builtin_fma(gd, gd, s.sq);
  s.top = fmaxf(s.top, fabsf(g));
}
__device__ __forceinline__ void add_row(GradSums& s, gs_f32x4 r) {
  add_grad(s, r.x); add_grad(s, r.y); add_grad(s, r.z); add_grad(s, r.w);
}
__device__ __forceinline__ void add_row(GradSums& s, gs_u32x2 r) {
  add_grad(s, u2f(r.x << 16)); add_grad(s, u2f(r.x & 0xFFFF0000u));
  add_grad(s, u2f(r.y << 16)); add_grad(s, u2f(r.y & 0xFFFF0000u));
}

template <bool BF16>
__global__ __launch_bounds__(64 * kGradWaves) void grad_stats_kernel(const TensorDesc* desc, uint32_t n_tensors,
                                                                     uint32_t total_tiles, uint32_t per_group, double* stats) {
  typedef typename GradRow<BF16>::type Row;
  __shared__ GradSums held[kGradWaves];
  __shared__ uint32_t ended_in[kGradWaves];  // the tensor a wave ended in, plus one
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t begin = static_cast<uint64_t>(blockIdx.x) * per_group;
  const uint32_t end = static_cast<uint32_t>(min(begin + per_group, static_cast<uint64_t>(total_tiles)));
  GradSums s = {0.0, 0.0, 0.0, 0.0f};
  uint32_t sum_of = 0;  // the tensor that s belongs to, plus one
  if (begin + wave < end) {
    uint32_t t = static_cast<uint32_t>(begin) + wave;
    uint32_t l = find_begin(desc, n_tensors, t, lane);
    TensorDesc d = load_desc(desc, l);
    Row row[8];
    auto whole = [&]() { return d.numel - static_cast<uint64_t>(t - d.tile_begin) * kTile >= static_cast<uint64_t>(kTile); };
    auto load = [&]() {  // a whole tile: eight loads in flight
      const STQ_GLOBAL Row* p = (const STQ_GLOBAL Row*)(d.grad) + static_cast<size_t>(t - d.tile_begin) * (kTile / 4) + lane;
#pragma unroll
      for (int i = 0; i < 8; ++i) row[i] = __builtin_nontemporal_load(p + 64 * i);
    };
    bool loaded = whole();
    if (loaded) load();
    for (;;) {
      // this tile's values out of the registers that the next tile's loads go into
      Row cur[8];
      const bool cur_whole = loaded;
      const uint64_t base = static_cast<uint64_t>(t - d.tile_begin) * kTile, left = d.numel - base;
      const void* const grad = d.grad;
      sum_of = l + 1u;
#pragma unroll
      for (int i = 0; i < 8; ++i) cur[i] = row[i];
      t += kGradWaves;
      const bool more = t < end;
      if (more) {
        while (t >= d.tile_begin + d.n_tiles) d = load_desc(desc, ++l);  // t < total_tiles: a later tensor holds it
        loaded = whole();
        if (loaded) load();
      }
      if (cur_whole) {
#pragma unroll
        for (int i = 0; i < 8; ++i) add_row(s, cur[i]);
      } else {  // the ragged last tile of a tensor: whole rows of four at once, the up to three elements behind them by a lane each
        const STQ_GLOBAL Row* p = (const STQ_GLOBAL Row*)(grad) + base / 4 + lane;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          cur[i] = Row{};
          if (4u * (64u * i + lane) + 4u <= left) cur[i] = p[64 * i];
        }
        const uint32_t rest = static_cast<uint32_t>(left) & 3u;
        uint32_t last = 0u;
        if (static_cast<uint32_t>(lane) < rest) {
          const uint64_t at = base + left - rest + lane;
          last = BF16 ? as_global(static_cast<const uint16_t*>(grad))[at] : as_global(static_cast<const uint32_t*>(grad))[at];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) add_row(s, cur[i]);
        add_grad(s, u2f(BF16 ? last << 16 : last));
        asm volatile("");  // (keeps these additions apart from a whole tile's, which must not wait for all loads)
      }
      if (!more) break;
      if (l + 1u != sum_of) {
        add_grad_sums(stats + static_cast<size_t>(sum_of - 1u) * kStatSlots, wave_sums(s), lane);
        s = {0.0, 0.0, 0.0, 0.0f};
      }
    }
  }
  // the waves that ended in the workgroup's last tensor together, a wave that ended in an earlier one by itself
  const GradSums w = wave_sums(s);
  if (lane == 0) {
    held[wave] = w;
    ended_in[wave] = sum_of;
  }
  __syncthreads();
  static_assert(kGradWaves == 8, "a lane of an octet for each wave");
  const uint32_t mine = ended_in[lane & 7], last = octet_max(mine);
  if (wave == 0) {
    const GradSums& h = held[lane & 7];
    const bool in = mine == last;
    const GradSums sum = {octet_sum(in ? h.sum : 0.0), octet_sum(in ? h.abs : 0.0), octet_sum(in ? h.sq : 0.0),
                          u2f(octet_max(in ? f2u(h.top) : 0u))};
    if (last) add_grad_sums(stats + static_cast<size_t>(last - 1u) * kStatSlots, sum, lane);
  }
  if (sum_of && sum_of != last) add_grad_sums(stats + static_cast<size_t>(sum_of - 1u) * kStatSlots, w, lane);
}

// The accumulators to host memory, and zero in their place: one launch instead of a copy and a fill.
__global__ __launch_bounds__(256) void take_stats_kernel(uint64_t* host, uint64_t* acc, uint64_t n) {
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  host[i] = acc[i];
  acc[i] = 0u;
}

}  // namespace

// -------------------------------------------------------------------- launchers
int launch_zero(const ZeroArgs& a, void* stream) {
  const uint64_t threads = static_cast<uint64_t>(a.n_tiles) * 64;
  hipLaunchKernelGGL(zero_kernel, dim3(static_cast<uint32_t>((threads + 255) / 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), a);
  return static_cast<int>(hipGetLastError());
}

int launch_repack_many(RepackManyArgs a, uint64_t code_bytes, void* stream) {
  a.chunk = a.total_tiles < 8192u ? 1u : 4u;  // (a launch that single tiles do not fill: every wave one)
  const uint32_t need = a.total_tiles / a.chunk + (a.total_tiles % a.chunk != 0);
  const uint32_t groups = need < (1u << 25) ? need : 1u << 25;  // (64 threads each: HIP counts the threads of a launch in 32 bits)
  // Codes that the 256 MB cache in front of the memory may still hold from the step before are read without the hint, which
  // would keep them out of it (codes of 4 to 5 bits, two states in turn: 130 M elements, 146 MB of reads and writes, 27.8 us
  // against 32.1; 200 M 37.6 against 43.2; 300 M, 338 MB, 58.4 against 59.9), those of larger launches with it (340 M, 383 MB,
  // 65.4 us against 66.4; 2.85 GB 521 against 527).
  const bool once = code_bytes >= kRepackOnceBytes;
  hipLaunchKernelGGL(once ? repack_many_kernel<true> : repack_many_kernel<false>, dim3(groups), dim3(64), 0, static_cast<hipStream_t>(stream), a);
  return static_cast<int>(hipGetLastError());
}

int launch_grad_stats(const TensorDesc* desc, uint32_t n_tensors, uint32_t total_tiles, double* stats, bool grad_bf16,
                      uint32_t n_cu, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  // One workgroup per CU, at least one tile per wave.  (0.12 G bf16 gradients in 100 tensors with read-back and decision
  // 85.6 us, 86.5 with two per CU, 91 with four of four waves; 30 M fp32 in one tensor 43.5, 47, 63; 1.5 G 885, 907, 940.)
  const uint64_t most = n_cu, rounds = (total_tiles + most * kGradWaves - 1) / (most * kGradWaves);
  const uint32_t per_group = static_cast<uint32_t>(rounds * kGradWaves);
  const dim3 grid((total_tiles + per_group - 1) / per_group), block(64 * kGradWaves);
  if (grad_bf16) hipLaunchKernelGGL(grad_stats_kernel<true>, grid, block, 0, s, desc, n_tensors, total_tiles, per_group, stats);
  else hipLaunchKernelGGL(grad_stats_kernel<false>, grid, block, 0, s, desc, n_tensors, total_tiles, per_group, stats);
  return static_cast<int>(hipGetLastError());
}

int launch_take_stats(double* host, double* acc, uint64_t n, void* stream) {
  hipLaunchKernelGGL(take_stats_kernel, dim3(static_cast<uint32_t>((n + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     reinterpret_cast<uint64_t*>(host), reinterpret_cast<uint64_t*>(acc), n);
  return static_cast<int>(hipGetLastError());
}

int launch_upload(void* dst, const void* pinned, uint64_t bytes, void* stream) {
  const uint64_t n = bytes / sizeof(uint4);
  hipLaunchKernelGGL(upload_kernel, dim3(static_cast<uint32_t>((n + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<uint4*>(dst), static_cast<const uint4*>(pinned), n);
  return static_cast<int>(hipGetLastError());
}

int launch_upload_by_value(void* dst, const void* host, uint64_t bytes, void* stream) {
  for (uint64_t at = 0; at < bytes; at += sizeof(UploadChunk)) {
    UploadChunk chunk;
    const uint64_t here = bytes - at < sizeof(UploadChunk) ? bytes - at : sizeof(UploadChunk);
    std::memcpy(&chunk, static_cast<const char*>(host) + at, here);
    hipLaunchKernelGGL(upload_by_value_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream),
                       reinterpret_cast<uint4*>(static_cast<char*>(dst) + at), static_cast<uint32_t>(here / sizeof(uint4)), chunk);
    if (const hipError_t e = hipGetLastError(); e != hipSuccess) return static_cast<int>(e);
  }
  return 0;
}

int launch_fill_zero(uint32_t* p, uint64_t words, void* stream) {
  hipLaunchKernelGGL(fill_zero_kernel, dim3(static_cast<uint32_t>((words + 255) / 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), p, words);
  return static_cast<int>(hipGetLastError());
}

}  // namespace stq
