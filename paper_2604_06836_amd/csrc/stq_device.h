// Structures shared by the host API and the gfx950 kernels of this library.
#pragma once
#include <cstdint>

namespace stq {

constexpr int kTile = 2048;         // elements per tile = 64 lanes x 32 codes
constexpr int kWavesPerGroup = 8;   // 512-thread workgroups
constexpr int kGradWaves = 8;       // waves of a workgroup of grad_stats_kernel
constexpr int kStatSlots = 16;      // 8-byte accumulator slots per tensor
constexpr uint32_t kLgTicketClasses = 3;  // the ticket counters of a launch, at most (see step_kernel)
constexpr uint32_t kSchedStride = 64;   // words from one counter to the next: each has cache lines of its own
constexpr uint32_t kSchedWords = kSchedStride << kLgTicketClasses;

// Device-resident description of one tensor for the step kernel.
struct TensorDesc {
  float* param;
  const void* grad;
  uint32_t* m_codes;
  float* m_scales;
  uint32_t* v_codes;
  float* v_scales;
  uint64_t numel;
  uint32_t tile_begin;  // index of this tensor's first tile in the launch-wide tile order
  uint32_t n_tiles;
  uint32_t bm, bv;      // widths of the stored codes
  uint32_t* m_out;      // where the new codes go: the same buffers, or others when a width changes
  uint32_t* v_out;
  uint32_t bm_out, bv_out;
};

// Accumulator slots (doubles unless noted).
enum StatSlot {
  kGSum = 0, kGAbsSum, kGSqSum, kMSum, kMSqSum, kMErrSq, kVSum, kVSqSum, kVErrSq,
  kMaxGM,   // two uint32: bit patterns of max|g| (low word) and max|m| (high word)
  kMaxV     // low uint32: bit pattern of max v
};

// A launch of the step kernel: its work ...
struct StepWork {
  const TensorDesc* desc;
  const uint32_t* tables;  // kTabWords words, see stq_tables.h
  uint32_t* sched;         // kSchedWords words, zero between launches: the ticket counters; null: nothing is drawn (see
                           // step_kernel)
  uint32_t n_tensors;
  uint32_t total_tiles;
  uint32_t lg_classes;     // log2 of the number of ticket counters
  uint32_t unit_rows;      // rows of a unit of scheduling: 2 (a quarter tile) or 4 (a half)
  bool write_through;      // with halves: parameters and whole words of 2- to 8-bit codes go through the L2 to memory at once
};
// ... and the rest of its arguments.
struct StepArgs {
  double* stats;           // [n_tensors][kStatSlots]
  float beta1, omb1, beta2, omb2;
  float ibc1, ibc2;        // reciprocal bias corrections 1/(1-beta^t)
  float eps, lr, decay;    // decay = 1 - lr*weight_decay
  uint32_t lgK;            // log2 of the block size: 6, 7 or 8
  uint32_t look_ahead;     // 0: a wave walks from tensor to tensor to that of its next unit; else it searches, this many
                           // entries of the table first
};

struct ZeroArgs {
  uint32_t* m_codes; float* m_scales; uint32_t* v_codes; float* v_scales;
  uint64_t numel;
  uint32_t n_tiles, bm, bv, scales_per_tile;
};

// One width change inside a batched re-pack launch.
struct RepackJob {
  const uint32_t* src; uint32_t* dst;
  uint64_t numel;
  uint32_t tile_begin, n_tiles;  // position in the launch-wide tile order
  uint32_t b_old, b_new;
  uint32_t lut;                  // index of the conversion table, see repack_lut_index
  uint32_t pad;
};
constexpr uint32_t kRepackLuts = 2 * 7 * 7;  // (state, old width, new width)
constexpr uint32_t repack_lut_index(uint32_t state, uint32_t b_old, uint32_t b_new) {
  return (state * 7 + (b_old - 2)) * 7 + (b_new - 2);
}
struct RepackManyArgs {
  const RepackJob* jobs;
  uint32_t n_jobs, total_tiles;
  uint32_t chunk;        // consecutive tiles a wave converts, set by the launcher
  const uint32_t* luts;  // [kRepackLuts][256] words
};

// Launchers implemented in stq_step.hip and stq_kernels.hip.  `stream` is a hipStream_t.  Return a hipError_t as int.
// stats: 0 none, 1 every statistic, 2 the gradient's only.
int launch_step(const StepWork& w, const StepArgs& a, bool grad_bf16, int stats, int mode, uint32_t groups, void* stream);
int launch_zero(const ZeroArgs& a, void* stream);
constexpr uint64_t kRepackOnceBytes = 350ull << 20;  // see launch_repack_many
int launch_repack_many(RepackManyArgs a, uint64_t code_bytes, void* stream);  // code_bytes: read and written
int launch_grad_stats(const TensorDesc* desc, uint32_t n_tensors, uint32_t total_tiles, double* stats, bool grad_bf16,
                      uint32_t n_cu, void* stream);
int launch_take_stats(double* host, double* acc, uint64_t n, void* stream);
int launch_upload(void* dst, const void* pinned, uint64_t bytes, void* stream);  // a multiple of 16 bytes
int launch_upload_by_value(void* dst, const void* host, uint64_t bytes, void* stream);  // the same, for a stream being recorded
int launch_fill_zero(uint32_t* p, uint64_t words, void* stream);

}  // namespace stq
