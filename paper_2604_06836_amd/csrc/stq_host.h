// Host-side internals shared by the sources that implement the C ABI: the context, argument
// checks, and the one place that configures and launches the step kernel over a device-resident
// tensor table.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "stq.h"
#include "stq_device.h"

namespace stq {

constexpr int kRingGroups = 3, kRingGroup = 8;   // pinned staging slots of a kind of upload: groups with an event each (see
constexpr int kRing = kRingGroups * kRingGroup;  // take_slot).  All but one group, sixteen uploads, may always be under way.
constexpr uint64_t kTicketMinTiles = 4096;  // launches of at least this many tiles, 8.4 M elements, draw tickets (see launch_table)
constexpr int kDescTables = 8;  // device-resident tensor tables kept: a caller that alternates between a
                                // few argument sets (two gradient buffers, say) uploads each only once
constexpr int kHeldTables = 4;  // of these, at most so many are never written again, since a recorded launch reads them
constexpr int kRecordedTable = kDescTables;  // one more, written by recorded launches only, each of which uploads it anew

}  // namespace stq

struct stq_ctx {
  int device = -1;
  uint32_t max_tensors = 0;
  uint32_t n_cu = 0;
  uint64_t ticket_min_tiles = stq::kTicketMinTiles;  // see stq_set_schedule
  uint32_t* d_tables = nullptr;
  stq::TensorDesc* d_desc[stq::kDescTables + 1] = {};  // parts of one allocation
  double* d_stats = nullptr;
  uint32_t* d_sched = nullptr;   // ticket counters of the step kernel (zero between launches), kSchedWords for each of d_desc:
                                 // launches that overlap although they should not then have counters of their own
  stq::TensorDesc* h_stage = nullptr;        // pinned, kRing slots of max_tensors
  hipEvent_t stage_done[stq::kRingGroups] = {};
  int ring_pos = 0;
  uint32_t* d_luts = nullptr;                // every conversion table of the re-pack, kRepackLuts x 256 words
  stq::RepackJob* d_jobs = nullptr;          // 2 * max_tensors
  stq::RepackJob* h_jobs = nullptr;          // pinned, kRing slots of 2 * max_tensors
  hipEvent_t jobs_done[stq::kRingGroups] = {};
  int jobs_pos = 0;
  double* h_stats = nullptr;                 // pinned, max_tensors * kStatSlots
  std::vector<stq::TensorDesc> uploaded[stq::kDescTables];  // what each d_desc currently holds
  hipStream_t uploaded_on[stq::kDescTables] = {};            // the stream that uploaded it
  bool held[stq::kDescTables] = {};                          // a recorded launch reads it
  int n_held = 0;
  std::vector<stq::TensorDesc> descs;        // descriptors of the call in progress (capacity max_tensors)
  void* static_scratch = nullptr;            // this device's static table of stq_step_static
  int desc_pos = 0;                          // next table to replace
  std::vector<uint64_t> stat_count;          // elements accumulated per tensor since the last stq_stats
};

namespace stq {

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

inline int check_bits(uint32_t b) { return (b >= 2 && b <= 8) ? STQ_OK : STQ_EBITS; }
inline bool is_wide(uint32_t b) { return b == 16 || b == 32; }
// widths a state can be stored at: the quantized ones, and 16 (bfloat16) and 32 (fp32) as they are
inline int check_bits_stored(uint32_t b) { return (is_wide(b) || check_bits(b) == STQ_OK) ? STQ_OK : STQ_EBITS; }

inline int lg_block(uint32_t K) {
  switch (K) { case 64: return 6; case 128: return 7; case 256: return 8; default: return -1; }
}

// The next slot of a ring, to be written by the host.  A group's slots are free again once the event that followed
// the upload from the last of them has passed (an event for each slot would put a barrier behind every upload).  Asking is cheap
// and almost always enough (the ring is long); waiting is the rare fallback -- on this runtime a wait on an event
// can take as long as the work queued behind it.
inline int take_slot(hipEvent_t* done, int* pos, int* slot) {
  const int k = *pos;
  if (k % kRingGroup == 0) {
    const hipEvent_t group = done[k / kRingGroup];
    const hipError_t q = hipEventQuery(group);
    if (q != hipSuccess) {
      (void)hipGetLastError();
      if (q != hipErrorNotReady || hipEventSynchronize(group) != hipSuccess) return STQ_EHIP;
    }
  }
  *pos = (k + 1) % kRing;
  *slot = k;
  return STQ_OK;
}
// After the upload from `slot` has been enqueued on s.
inline int slot_in_use(hipEvent_t* done, int slot, hipStream_t s) {
  if (slot % kRingGroup != kRingGroup - 1) return STQ_OK;
  return hipEventRecord(done[slot / kRingGroup], s) == hipSuccess ? STQ_OK : STQ_EHIP;
}

// Whether work enqueued on s is recorded into a graph instead of run.  What a recorded launch reads at its replays must not
// be memory that later calls write again: not a staging slot, nor a table that is kept for one argument set after the other.
// (The default stream cannot be captured.)
inline bool recording(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (!s) return false;
  if (hipStreamIsCapturing(s, &status) != hipSuccess) { (void)hipGetLastError(); return false; }
  return status == hipStreamCaptureStatusActive;
}

struct DeviceGuard {  // makes the context's device current for the duration of a call
  int prev = -1; bool ok = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) return;
    ok = (prev == dev) || hipSetDevice(dev) == hipSuccess;
    if (prev == dev) prev = -1;
  }
  ~DeviceGuard() { if (ok && prev >= 0) (void)hipSetDevice(prev); }
};

// Checks the hyper-parameters of a step (Adam's own preconditions).
int check_hparams(const stq_hparams* hp);

// Fills the descriptors of n tensors at the widths of `plan` (new codes in place) and the launch-wide tile count.
int build_descs(const stq_ctx* ctx, const stq_tensor* t, uint32_t n, const stq_bits* plan, uint32_t K,
                bool need_param_grad, std::vector<TensorDesc>& out, uint32_t* total_tiles);

// Launches the step kernel over the device-resident table `d_desc` of n tensors / total_tiles tiles.
// mode: 0 in place, 1 widths change, 2 some state is (or may become) 16 or 32 bits wide.
// sched: the kSchedWords ticket counters the launch uses, those of its table.
int launch_table(stq_ctx* ctx, const TensorDesc* d_desc, uint32_t n, uint32_t total_tiles, double* d_stats,
                 const stq_hparams* hp, int mode, void* stream, uint32_t* sched);

}  // namespace stq
