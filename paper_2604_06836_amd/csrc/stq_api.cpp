// Host side of the C ABI declared in include/stq.h: argument checks, the device-resident
// tensor table, kernel launches, statistics read-back.  Compiled by hipcc (HIP runtime calls).
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "stq_host.h"
#include "stq_tables.h"

using namespace stq;

namespace stq {

int build_descs(const stq_ctx* ctx, const stq_tensor* t, uint32_t n, const stq_bits* plan, uint32_t K,
                bool need_param_grad, std::vector<TensorDesc>& out, uint32_t* total_tiles) {
  if (!ctx || !t || !plan || n == 0 || n > ctx->max_tensors) return STQ_EINVAL;
  out.resize(n);
  if (lg_block(K) < 0) return STQ_EBLOCK;
  uint64_t tiles = 0;
  for (uint32_t l = 0; l < n; ++l) {
    if (int e = check_bits_stored(plan[l].m_bits)) return e;
    if (int e = check_bits_stored(plan[l].v_bits)) return e;
    if (t[l].numel == 0) return STQ_EINVAL;
    if (!t[l].m_codes || !t[l].m_scales || !t[l].v_codes || !t[l].v_scales) return STQ_EINVAL;
    if (need_param_grad && (!t[l].param || !t[l].grad)) return STQ_EINVAL;
    if (!aligned(t[l].m_codes, 256) || !aligned(t[l].m_scales, 256) || !aligned(t[l].v_codes, 256) ||
        !aligned(t[l].v_scales, 256))
      return STQ_EALIGN;
    if (need_param_grad && (!aligned(t[l].param, 16) || !aligned(t[l].grad, 16))) return STQ_EALIGN;
    const uint64_t nt = (t[l].numel + kTile - 1) / kTile;
    if (tiles + nt > 0xFFFFFFFFull) return STQ_EINVAL;
    TensorDesc& d = out[l];
    d.param = static_cast<float*>(t[l].param);
    d.grad = t[l].grad;
    d.m_codes = static_cast<uint32_t*>(t[l].m_codes);
    d.m_scales = t[l].m_scales;
    d.v_codes = static_cast<uint32_t*>(t[l].v_codes);
    d.v_scales = t[l].v_scales;
    d.numel = t[l].numel;
    d.tile_begin = static_cast<uint32_t>(tiles);
    d.n_tiles = static_cast<uint32_t>(nt);
    d.bm = plan[l].m_bits;
    d.bv = plan[l].v_bits;
    d.m_out = d.m_codes;  // in place unless a caller redirects them
    d.v_out = d.v_codes;
    d.bm_out = d.bm;
    d.bv_out = d.bv;
    tiles += nt;
  }
  *total_tiles = static_cast<uint32_t>(tiles);
  return STQ_OK;
}

}  // namespace stq

// ---------------------------------------------------------------- static scratch
// Device memory of stq_step_static, the entry point that allocates nothing: the tensor table its
// kernel reads.  One copy per GPU, held until the process ends.  In host code the array's name is only
// a stand-in for the symbol: the address that kernels and copies use comes from hipGetSymbolAddress,
// once per device (stq_init), and is kept in g_static_scratch.
namespace {

constexpr uint32_t kStaticMaxTensors = STQ_STATIC_MAX_TENSORS;
constexpr size_t kStaticTableBytes = sizeof(TensorDesc) * kStaticMaxTensors;
constexpr size_t kStaticScratchBytes = kStaticTableBytes + 4 * kSchedWords;  // the table, then the ticket counters
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
void* g_static_scratch[kMaxDevices];  // per device, null until a context was created on it

// With `device` current: the address of that device's copy of `scratch`.
int static_scratch_address(int device, void** out) {
  if (device < 0 || device >= kMaxDevices) return STQ_EDEVICE;
  if (!g_static_scratch[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return STQ_EHIP;
    g_static_scratch[device] = p;
  }
  *out = g_static_scratch[device];
  return STQ_OK;
}

}  // namespace

extern "C" {

const char* stq_strerror(int code) {
  switch (code) {
    case STQ_OK: return "ok";
    case STQ_EINVAL: return "invalid argument";
    case STQ_EALIGN: return "misaligned device buffer";
    case STQ_EBITS: return "bit-width not one of 2..8 (or, for a stored state, 16 or 32)";
    case STQ_EBLOCK: return "block size must be 64, 128 or 256";
    case STQ_EDEVICE: return "device missing or not gfx950";
    case STQ_EHIP: return "HIP runtime error";
    case STQ_ESTATE: return "no statistics accumulated";
    case STQ_ELIMIT: return "more tensors than the static scratch of stq_step_static holds";
    default: return "unknown error";
  }
}

int stq_state_bytes(uint64_t numel, uint32_t block, uint32_t bits, uint64_t* code_bytes,
                    uint64_t* scale_bytes) {
  if (numel == 0 || (!code_bytes && !scale_bytes)) return STQ_EINVAL;
  if (lg_block(block) < 0) return STQ_EBLOCK;
  if (int e = check_bits_stored(bits)) return e;
  const uint64_t tiles = (numel + kTile - 1) / kTile;
  if (code_bytes) *code_bytes = tiles * 64ull * bits * 4ull;
  if (scale_bytes) *scale_bytes = tiles * (kTile / block) * 4ull;
  return STQ_OK;
}

int stq_table(int which, uint32_t bits, float* out, uint32_t n) {
  if (!out) return STQ_EINVAL;
  if (which == 0) {
    for (uint32_t j = 0; j < n && j < static_cast<uint32_t>(kGLen); ++j) out[j] = table_G(static_cast<int>(j));
    return kGLen;
  }
  if (int e = check_bits(bits)) return e;
  const int b = static_cast<int>(bits);
  int len;
  switch (which) {
    case 1: len = (1 << b) - 1; for (int u = 0; u < len && u < static_cast<int>(n); ++u) out[u] = table_R(b, u); break;
    case 2: len = (1 << b);     for (int c = 0; c < len && c < static_cast<int>(n); ++c) out[c] = table_L(b, c); break;
    case 3: len = (1 << b) - 1; for (int k = 0; k < len && k < static_cast<int>(n); ++k) out[k] = table_T(b, k); break;
    default: return STQ_EINVAL;
  }
  return len;
}

int stq_init(stq_ctx** out, int device, uint32_t max_tensors) {
  if (!out || max_tensors == 0 || max_tensors > (1u << 20)) return STQ_EINVAL;
  *out = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count) return STQ_EDEVICE;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return STQ_EDEVICE;
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return STQ_EDEVICE;
  std::vector<uint32_t> img;
  if (!build_table_image(img)) return STQ_EINVAL;

  stq_ctx* c = new (std::nothrow) stq_ctx();
  if (!c) return STQ_EINVAL;
  c->device = device;
  c->max_tensors = max_tensors;
  c->n_cu = static_cast<uint32_t>(prop.multiProcessorCount);
  DeviceGuard g(device);
  bool ok = g.ok;
  ok = ok && static_scratch_address(device, &c->static_scratch) == STQ_OK;
  ok = ok && hipMalloc(&c->d_tables, img.size() * 4) == hipSuccess;
  ok = ok && hipMalloc(&c->d_desc[0], sizeof(TensorDesc) * max_tensors * (kRecordedTable + 1)) == hipSuccess;
  for (int k = 1; k <= kRecordedTable && ok; ++k) c->d_desc[k] = c->d_desc[0] + static_cast<size_t>(max_tensors) * k;
  ok = ok && hipMalloc(&c->d_stats, sizeof(double) * kStatSlots * max_tensors) == hipSuccess;
  ok = ok && hipMalloc(&c->d_sched, 4 * kSchedWords * (kRecordedTable + 1)) == hipSuccess;
  ok = ok && hipMemset(c->d_sched, 0, 4 * kSchedWords * (kRecordedTable + 1)) == hipSuccess;
  ok = ok && hipHostMalloc(&c->h_stats, sizeof(double) * kStatSlots * max_tensors, hipHostMallocDefault) == hipSuccess;
  ok = ok && hipHostMalloc(&c->h_stage, sizeof(TensorDesc) * max_tensors * kRing, hipHostMallocDefault) == hipSuccess;
  ok = ok && hipHostMalloc(&c->h_jobs, sizeof(RepackJob) * 2 * max_tensors * kRing, hipHostMallocDefault) == hipSuccess;
  for (int k = 0; k < kRingGroups && ok; ++k) {
    ok = ok && hipEventCreateWithFlags(&c->stage_done[k], hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&c->jobs_done[k], hipEventDisableTiming) == hipSuccess;
  }
  ok = ok && hipMemcpy(c->d_tables, img.data(), img.size() * 4, hipMemcpyHostToDevice) == hipSuccess;
  // every conversion table of the re-pack: (state, old width, new width) -> 256 codes, one word each
  std::vector<uint32_t> luts(static_cast<size_t>(kRepackLuts) * 256);
  for (int st = 0; st < 2; ++st)
    for (int bo = kMinBits; bo <= kMaxBits; ++bo)
      for (int bn = kMinBits; bn <= kMaxBits; ++bn) {
        uint8_t one[256];
        build_repack_lut(st, bo, bn, one);
        uint32_t* dst = &luts[static_cast<size_t>(repack_lut_index(st, bo, bn)) * 256];
        for (int i = 0; i < 256; ++i) dst[i] = one[i];
      }
  ok = ok && hipMalloc(&c->d_luts, luts.size() * 4) == hipSuccess;
  ok = ok && hipMemcpy(c->d_luts, luts.data(), luts.size() * 4, hipMemcpyHostToDevice) == hipSuccess;
  ok = ok && hipMalloc(&c->d_jobs, sizeof(RepackJob) * 2 * max_tensors) == hipSuccess;
  ok = ok && hipMemset(c->d_stats, 0, sizeof(double) * kStatSlots * max_tensors) == hipSuccess;
  ok = ok && hipDeviceSynchronize() == hipSuccess;
  if (!ok) { stq_destroy(c); return STQ_EHIP; }
  c->stat_count.assign(max_tensors, 0);
  c->descs.reserve(max_tensors);
  for (int k = 0; k < kDescTables; ++k) c->uploaded[k].reserve(max_tensors);
  *out = c;
  return STQ_OK;
}

int stq_set_schedule(stq_ctx* ctx, uint64_t ticket_min_tiles) {
  if (!ctx) return STQ_EINVAL;
  ctx->ticket_min_tiles = ticket_min_tiles ? ticket_min_tiles : kTicketMinTiles;
  return STQ_OK;
}

int stq_destroy(stq_ctx* c) {
  if (!c) return STQ_EINVAL;
  DeviceGuard g(c->device);
  (void)hipDeviceSynchronize();
  if (c->d_tables) (void)hipFree(c->d_tables);
  if (c->d_desc[0]) (void)hipFree(c->d_desc[0]);
  if (c->d_stats) (void)hipFree(c->d_stats);
  if (c->d_sched) (void)hipFree(c->d_sched);
  if (c->h_stats) (void)hipHostFree(c->h_stats);
  if (c->d_luts) (void)hipFree(c->d_luts);
  if (c->d_jobs) (void)hipFree(c->d_jobs);
  if (c->h_jobs) (void)hipHostFree(c->h_jobs);
  if (c->h_stage) (void)hipHostFree(c->h_stage);
  for (int k = 0; k < kRingGroups; ++k) {
    if (c->jobs_done[k]) (void)hipEventDestroy(c->jobs_done[k]);
    if (c->stage_done[k]) (void)hipEventDestroy(c->stage_done[k]);
  }
  delete c;
  return STQ_OK;
}

int stq_zero_state(stq_ctx* ctx, const stq_tensor* tensors, uint32_t n, const stq_bits* plan,
                   uint32_t block, void* stream) {
  std::vector<TensorDesc> descs;
  uint32_t total = 0;
  if (int e = build_descs(ctx, tensors, n, plan, block, false, descs, &total)) return e;
  DeviceGuard g(ctx->device);
  if (!g.ok) return STQ_EHIP;
  for (uint32_t l = 0; l < n; ++l) {
    ZeroArgs a;
    a.m_codes = descs[l].m_codes; a.m_scales = descs[l].m_scales;
    a.v_codes = descs[l].v_codes; a.v_scales = descs[l].v_scales;
    a.numel = descs[l].numel; a.n_tiles = descs[l].n_tiles;
    a.bm = descs[l].bm; a.bv = descs[l].bv; a.scales_per_tile = kTile / block;
    if (launch_zero(a, stream) != 0) return STQ_EHIP;
  }
  return STQ_OK;
}

}  // extern "C"

namespace stq {

int check_hparams(const stq_hparams* hp) {
  if (!hp) return STQ_EINVAL;
  if (hp->step == 0 || hp->grad_dtype > 1) return STQ_EINVAL;
  // Adam's own preconditions: finite lr >= 0 and weight decay, 0 <= beta < 1, finite eps > 0
  if (!(hp->lr >= 0.0f) || !std::isfinite(hp->lr) || !std::isfinite(hp->weight_decay)) return STQ_EINVAL;
  if (!(hp->beta1 >= 0.0f && hp->beta1 < 1.0f) || !(hp->beta2 >= 0.0f && hp->beta2 < 1.0f)) return STQ_EINVAL;
  if (!(hp->eps > 0.0f) || !std::isfinite(hp->eps)) return STQ_EINVAL;
  if (lg_block(hp->block) < 0) return STQ_EBLOCK;
  return STQ_OK;
}

int launch_table(stq_ctx* ctx, const TensorDesc* d_desc, uint32_t n, uint32_t total, double* d_stats,
                 const stq_hparams* hp, int mode, void* stream, uint32_t* sched) {
  StepWork w;
  StepArgs a;
  w.desc = d_desc;
  w.n_tensors = n;
  w.total_tiles = total;
  w.tables = ctx->d_tables;
  a.stats = d_stats;
  a.beta1 = hp->beta1;
  a.omb1 = 1.0f - hp->beta1;
  a.beta2 = hp->beta2;
  a.omb2 = 1.0f - hp->beta2;
  // reciprocal bias corrections 1/(1 - beta^t): double arithmetic, one rounding to fp32
  a.ibc1 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(hp->beta1), static_cast<double>(hp->step))));
  a.ibc2 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(hp->beta2), static_cast<double>(hp->step))));
  a.eps = hp->eps;
  a.lr = hp->lr;
  a.decay = 1.0f - hp->lr * hp->weight_decay;
  a.lgK = static_cast<uint32_t>(lg_block(hp->block));

  // statistics: all of them, or only the gradient's (the flag for all wins)
  const int stats = (hp->flags & STQ_FLAG_STATS) ? 1 : ((hp->flags & STQ_FLAG_STATS_GRAD) ? 2 : 0);
  const bool fp32_grads = hp->grad_dtype == 0, wide = mode == 2;
  const uint32_t wpg = kWavesPerGroup;
  // Units (see step_kernel): half tiles, which two workgroups per CU take with 128 registers a wave.  Quarter tiles, with
  // three workgroups per CU, in launches whose quarters all fit at once, where a wave with half the work is done sooner
  // (1 M parameters 5.8 us, with halves 6.9; 3.0 M 9.0 and 10.3, 3.2 M 11.4 and 10.4).  With statistics only the smallest of
  // these (0.5 M 25.4 and 25.6, 1.0 M 28.9 and 27.7, 3.0 M 41.6 and 34.7: what a unit leaves of them costs as much for a
  // quarter) and those of small tensors, each of which is left by itself (300 tensors of 3000 elements 31.6 and 34.3, 1000 of
  // 768 40.2 and 42.4).
  const bool quarters = total * 4ull <= static_cast<uint64_t>(ctx->n_cu) * 3 * wpg && (!stats || total <= ctx->n_cu || total < 16ull * n);
  // Tickets drawn, in one order over the chip, or every workgroup's own (see step_kernel).  fp32 gradients: 9.0 M
  // parameters 24.5 us drawn and 25.1 not, 16 M 39.2 and 41.1, 60 M 145 and 153; bf16: 12.5 M 28.0 and 27.4, 16 M 33.7
  // and 35.0, 60 M 114 and 117; wide states: 12.5 M 47.8 and 48.1, 9.0 M 38.1 and 37.1.
  const bool draws = (fp32_grads && !wide ? total : total * 2ull / 3) >= ctx->ticket_min_tiles;
  // Workgroups per CU.  States of 16 and 32 bits beside fp32 gradients have twice the bytes of others per element: one
  // workgroup has enough of them in flight, and keeps the window narrower (16- and 32-bit states, 90 M: 357 us, 389 with
  // two; 8 and 16 bits 130 M: 386 and 402, but 30 M 94 and 86; with bf16 gradients 130 M 360 and 356).
  uint32_t per_cu = quarters ? 3 : (wide && fp32_grads && draws && total >= 30000u ? 1 : 2);
  uint32_t lg_parts = quarters ? 2 : 1;
#ifdef STQ_TUNING_ENV  // measurement builds only: launch shape from the environment
  if (const char* e = std::getenv("STQ_LG_PARTS")) { lg_parts = std::strtoul(e, nullptr, 10) == 2 ? 2 : 1; per_cu = lg_parts == 2 ? 3 : 2; }
  if (const char* e = std::getenv("STQ_GROUPS_PER_CU")) per_cu = std::strtoul(e, nullptr, 10);
#endif
  w.sched = draws ? sched : nullptr;
  w.unit_rows = 8u >> lg_parts;
  const uint64_t units = static_cast<uint64_t>(total) << lg_parts;
  const uint64_t need_groups = (units + wpg - 1) / wpg, max_groups = static_cast<uint64_t>(ctx->n_cu) * per_cu;
  const uint32_t groups = static_cast<uint32_t>(need_groups < max_groups ? need_groups : max_groups);
  // Eight counters (where every one has as many workgroups: fewer CUs than the card has, or a small launch) as long as the
  // draws of the start count, one in larger launches, where the classes would drift apart (9 M parameters 22.5 us with
  // eight and 26.9 with one, 130 M 267.5 and 270.5, 300 M 616 and 613; 3.5 G 7.20 ms and 7.00).
  w.lg_classes = total < 100000u && groups % (8u << kLgTicketClasses) == 0 ? kLgTicketClasses : 0;
#ifdef STQ_TUNING_ENV
  if (const char* e = std::getenv("STQ_CLASSES")) w.lg_classes = std::strtoul(e, nullptr, 10);
#endif
  // Large launches write through: parameters and the code words of quantized states leave the L2 at once, with the reads that
  // make room for them no longer waiting for a line to be written (0.1 G parameters: bf16 gradients 214.4 us, written through
  // 211.5, fp32 240.2 and 238.0; 0.2 G 404 and 400, 460 and 455; 1.56 G bf16 3082 and 3051; transitions 1.4 % less, 16-bit states,
  // of which only the parameters are, 1.0 %).  The line lies above the launches that lose by it, fp32 gradients of 40 to 60 M
  // parameters (one tensor: 40 M 88.0 and 89.5, 60 M 129.1 and 133.2; 50 tensors of 62 M 136.7 and 137.6; why is not known).
  // Others below it would have up to 1 % less (50 tensors: fp32 81 M 196.9 and 195.8, 31 M 72.5 and 71.7, bf16 62 M 122.3 and
  // 121.7; wide states 30 M 127.9 and 126.7) or nothing (bf16, 50 tensors of 81 M 171.8 and 171.8, one of 30 M 60.9 and 61.1).
  // With every statistic, where the vector instructions count, 0.5 G 1340 and 1340: not built.
  w.write_through = total >= 45000u;
  // How a wave finds the tensor of its next unit (see step_kernel).  A walk costs one scalar load after the other for each
  // tensor it passes, a search one or two vector loads, which take as long as some of them while the memory system is busy.
  // With at most 8 tensors to the next unit on average a wave walks (148 tensors of 124 M elements, 5 to pass: 256 us, with
  // a search 258); beyond, it searches a window of 64 entries first (600 of 131,072 elements, 32 to pass: 193 us, walking
  // 222; 1000 of 67,591, 60 to pass: 170 and 318), from 64 on one of 4096 (4000 of 16,384, 256 to pass: 157 us, with 64
  // first 164, walking 1089; 4000 of 768: 22, 35 and 449).
  const uint64_t passed = (static_cast<uint64_t>(groups) * wpg >> lg_parts) * n / total;
  a.look_ahead = passed <= 8 ? 0u : (passed < 64 ? 64u : 4096u);
#ifdef STQ_TUNING_ENV
  if (const char* e = std::getenv("STQ_LOOK")) a.look_ahead = std::strtoul(e, nullptr, 10);
#endif
  return launch_step(w, a, hp->grad_dtype == 1, stats, mode, groups, stream) == 0 ? STQ_OK : STQ_EHIP;
}

}  // namespace stq

namespace {

// n descriptors into `dst` in stream order, through a pinned staging slot.
int upload_descs(stq_ctx* ctx, const std::vector<TensorDesc>& descs, TensorDesc* dst, hipStream_t s) {
  const size_t bytes = sizeof(TensorDesc) * descs.size();
  if (recording(s)) return launch_upload_by_value(dst, descs.data(), bytes, s) == 0 ? STQ_OK : STQ_EHIP;
  int k = -1;
  if (int e = take_slot(ctx->stage_done, &ctx->ring_pos, &k)) return e;
  TensorDesc* const slot = ctx->h_stage + static_cast<size_t>(ctx->max_tensors) * k;
  std::memcpy(slot, descs.data(), bytes);
  const int launched = launch_upload(dst, slot, bytes, s);
  if (int e = slot_in_use(ctx->stage_done, k, s)) return e;
  return launched == 0 ? STQ_OK : STQ_EHIP;
}

// Index of a device-resident tensor table that holds `descs`: one that already does (uploaded on this
// same stream, so the kernel is ordered after the upload), else the oldest, overwritten in stream order
// (after the kernels that read it).  A launch that is recorded reads its table at every replay, so one on the device is held
// from then on, and where that cannot be, the table is uploaded with the launch, into one that no call takes to be there
// (recording it uploads nothing yet).
int resident_table(stq_ctx* ctx, const std::vector<TensorDesc>& descs, hipStream_t s, int* out) {
  const size_t n = descs.size();
  int table = -1;
  for (int k = 0; k < kDescTables && table < 0; ++k)
    if (ctx->uploaded_on[k] == s && ctx->uploaded[k].size() == n &&
        std::memcmp(ctx->uploaded[k].data(), descs.data(), sizeof(TensorDesc) * n) == 0)
      table = k;
  if (recording(s)) {
    if (table >= 0 && !ctx->held[table] && ctx->n_held < kHeldTables) {
      ctx->held[table] = true;
      ++ctx->n_held;
    }
    if (table < 0 || !ctx->held[table]) {
      table = kRecordedTable;
      if (int e = upload_descs(ctx, descs, ctx->d_desc[table], s)) return e;
    }
  } else if (table < 0) {
    while (ctx->held[ctx->desc_pos]) ctx->desc_pos = (ctx->desc_pos + 1) % kDescTables;
    table = ctx->desc_pos;
    ctx->uploaded[table].clear();  // whatever happens below, the old contents are no longer claimed
    if (int e = upload_descs(ctx, descs, ctx->d_desc[table], s)) return e;
    ctx->desc_pos = (table + 1) % kDescTables;
    ctx->uploaded[table] = descs;
    ctx->uploaded_on[table] = s;
  }
  *out = table;
  return STQ_OK;
}

// Kernel variant for a set of descriptors: 0 in place, 1 widths change, 2 some state is (or becomes)
// 16 or 32 bits wide.
int mode_of(const TensorDesc* descs, uint32_t n, bool changes) {
  for (uint32_t l = 0; l < n; ++l) {
    const TensorDesc& d = descs[l];
    if (is_wide(d.bm) || is_wide(d.bv) || is_wide(d.bm_out) || is_wide(d.bv_out)) return 2;
  }
  return changes ? 1 : 0;
}

// One launch of the step kernel.  new_plan/new_codes are null for the in-place step.
int step_impl(stq_ctx* ctx, const stq_tensor* tensors, uint32_t n, const stq_bits* plan,
              const stq_bits* new_plan, const stq_codes* new_codes, const stq_hparams* hp, void* stream) {
  if (int e = check_hparams(hp)) return e;
  if (!ctx) return STQ_EINVAL;
  std::vector<TensorDesc>& descs = ctx->descs;  // reserved at stq_init: no allocation per call
  uint32_t total = 0;
  if (int e = build_descs(ctx, tensors, n, plan, hp->block, true, descs, &total)) return e;
  if (new_plan) {
    for (uint32_t l = 0; l < n; ++l) {
      TensorDesc& d = descs[l];
      if (int e = check_bits_stored(new_plan[l].m_bits)) return e;
      if (int e = check_bits_stored(new_plan[l].v_bits)) return e;
      const uintptr_t span = static_cast<uintptr_t>(d.n_tiles) * 256;
      struct { uint32_t b_old, b_new; uint32_t* cur; void* dst; uint32_t** out; } st[2] = {
          {d.bm, new_plan[l].m_bits, d.m_codes, new_codes[l].m_codes, &d.m_out},
          {d.bv, new_plan[l].v_bits, d.v_codes, new_codes[l].v_codes, &d.v_out}};
      for (auto& x : st) {
        if (x.b_new == x.b_old && (x.dst == nullptr || x.dst == x.cur)) continue;  // stays in place
        // another width (or another buffer): the destination must be a distinct, aligned buffer
        if (!x.dst) return STQ_EINVAL;
        if (!aligned(x.dst, 256)) return STQ_EALIGN;
        const uintptr_t s0 = reinterpret_cast<uintptr_t>(x.cur), s1 = s0 + span * x.b_old;
        const uintptr_t d0 = reinterpret_cast<uintptr_t>(x.dst), d1 = d0 + span * x.b_new;
        if (s0 < d1 && d0 < s1) return STQ_EINVAL;
        *x.out = static_cast<uint32_t*>(x.dst);
      }
      d.bm_out = new_plan[l].m_bits;
      d.bv_out = new_plan[l].v_bits;
    }
  }
  DeviceGuard g(ctx->device);
  if (!g.ok) return STQ_EHIP;
  hipStream_t s = static_cast<hipStream_t>(stream);

  int table = -1;
  if (int e = resident_table(ctx, descs, s, &table)) return e;

  const int mode = mode_of(descs.data(), n, new_plan != nullptr);
  uint32_t* const sched = ctx->d_sched + static_cast<size_t>(table) * kSchedWords;
  if (int e = launch_table(ctx, ctx->d_desc[table], n, total, ctx->d_stats, hp, mode, stream, sched)) return e;
  if ((hp->flags & (STQ_FLAG_STATS | STQ_FLAG_STATS_GRAD)) != 0)
    for (uint32_t l = 0; l < n; ++l) ctx->stat_count[l] += tensors[l].numel;
  return STQ_OK;
}

}  // namespace

extern "C" {

int stq_step(stq_ctx* ctx, const stq_tensor* tensors, uint32_t n, const stq_bits* plan,
             const stq_hparams* hp, void* stream) {
  return step_impl(ctx, tensors, n, plan, nullptr, nullptr, hp, stream);
}

int stq_step_transition(stq_ctx* ctx, const stq_tensor* tensors, uint32_t n, const stq_bits* plan_old,
                        const stq_bits* plan_new, const stq_codes* new_codes, const stq_hparams* hp,
                        void* stream) {
  if (!plan_new || !new_codes) return STQ_EINVAL;
  return step_impl(ctx, tensors, n, plan_old, plan_new, new_codes, hp, stream);
}

int stq_step_static(stq_ctx* ctx, const stq_tensor* tensors, uint32_t n, const stq_bits* plan,
                    const stq_hparams* hp, void* stream) {
  if (int e = check_hparams(hp)) return e;
  if (!ctx || !tensors || !plan || n == 0) return STQ_EINVAL;
  if (n > kStaticMaxTensors) return STQ_ELIMIT;
  if (n > ctx->max_tensors) return STQ_EINVAL;
  DeviceGuard g(ctx->device);
  if (!g.ok) return STQ_EHIP;
  hipStream_t s = static_cast<hipStream_t>(stream);
  std::vector<TensorDesc>& descs = ctx->descs;  // reserved at stq_init: no allocation per call
  uint32_t total = 0;
  if (int e = build_descs(ctx, tensors, n, plan, hp->block, true, descs, &total)) return e;
  const int mode = mode_of(descs.data(), n, false);
  TensorDesc* table = static_cast<TensorDesc*>(ctx->static_scratch);
  uint32_t* sched = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(ctx->static_scratch) + kStaticTableBytes);
  if (int e = upload_descs(ctx, descs, table, s)) return e;
  // the scheduling words must be zero when the kernel starts: a kernel leaves them so, but the array is shared
  // by every caller on this GPU and may hold what an aborted launch left
  if (launch_fill_zero(sched, kSchedWords, stream) != 0) return STQ_EHIP;
  if (int e = launch_table(ctx, table, n, total, ctx->d_stats, hp, mode, stream, sched)) return e;
  if ((hp->flags & (STQ_FLAG_STATS | STQ_FLAG_STATS_GRAD)) != 0)
    for (uint32_t l = 0; l < n; ++l) ctx->stat_count[l] += tensors[l].numel;
  return STQ_OK;
}

int stq_grad_stats(stq_ctx* ctx, const stq_tensor* tensors, uint32_t n, uint32_t block, uint32_t grad_dtype,
                   void* stream) {
  if (grad_dtype > 1) return STQ_EINVAL;
  if (!ctx || !tensors || n == 0 || n > ctx->max_tensors) return STQ_EINVAL;
  std::vector<stq_bits> any(n, stq_bits{8, 8});  // the widths play no part here
  std::vector<TensorDesc> descs;
  uint32_t total = 0;
  if (int e = build_descs(ctx, tensors, n, any.data(), block, true, descs, &total)) return e;
  DeviceGuard g(ctx->device);
  if (!g.ok) return STQ_EHIP;
  int table = -1;
  if (int e = resident_table(ctx, descs, static_cast<hipStream_t>(stream), &table)) return e;
  if (launch_grad_stats(ctx->d_desc[table], n, total, ctx->d_stats, grad_dtype == 1, ctx->n_cu, stream) != 0)
    return STQ_EHIP;
  for (uint32_t l = 0; l < n; ++l) ctx->stat_count[l] += tensors[l].numel;
  return STQ_OK;
}

int stq_stats(stq_ctx* ctx, stq_layer_stats* out, uint32_t n, void* stream) {
  if (!ctx || !out || n == 0 || n > ctx->max_tensors) return STQ_EINVAL;
  for (uint32_t l = 0; l < n; ++l) if (ctx->stat_count[l] == 0) return STQ_ESTATE;
  DeviceGuard g(ctx->device);
  if (!g.ok) return STQ_EHIP;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // (Pinned memory of hipHostMalloc is the device's to write too.  Looking for a mark that the kernel writes behind its results,
  // instead of waiting for the stream, returns 3 to 5 us sooner, but before the stream is idle and without what it would report.)
  if (launch_take_stats(ctx->h_stats, ctx->d_stats, static_cast<uint64_t>(kStatSlots) * n, stream) != 0) return STQ_EHIP;
  if (hipStreamSynchronize(s) != hipSuccess) return STQ_EHIP;
  for (uint32_t l = 0; l < n; ++l) {
    const double* a = ctx->h_stats + static_cast<size_t>(l) * kStatSlots;
    stq_layer_stats& o = out[l];
    o.count = ctx->stat_count[l];
    o.g_sum = a[kGSum]; o.g_abs_sum = a[kGAbsSum]; o.g_sq_sum = a[kGSqSum];
    o.m_sum = a[kMSum]; o.m_sq_sum = a[kMSqSum]; o.m_err_sq = a[kMErrSq];
    o.v_sum = a[kVSum]; o.v_sq_sum = a[kVSqSum]; o.v_err_sq = a[kVErrSq];
    uint32_t mx[4];
    std::memcpy(mx, &a[kMaxGM], 16);
    std::memcpy(&o.g_absmax, &mx[0], 4);
    std::memcpy(&o.m_absmax, &mx[1], 4);
    std::memcpy(&o.v_absmax, &mx[2], 4);
    ctx->stat_count[l] = 0;
  }
  return STQ_OK;
}

int stq_repack(stq_ctx* ctx, uint64_t numel, uint32_t block, int state, const void* src,
               uint32_t src_bits, void* dst, uint32_t dst_bits, void* stream) {
  // one job of stq_repack_many: the same checks, the same kernel
  if (state != 0 && state != 1) return STQ_EINVAL;
  stq_repack_job j;
  j.numel = numel;
  j.src_codes = src;
  j.dst_codes = dst;
  j.state = static_cast<uint8_t>(state);
  j.src_bits = static_cast<uint8_t>(src_bits <= 255 ? src_bits : 255);
  j.dst_bits = static_cast<uint8_t>(dst_bits <= 255 ? dst_bits : 255);
  return stq_repack_many(ctx, &j, 1, block, stream);
}

int stq_repack_many(stq_ctx* ctx, const stq_repack_job* jobs, uint32_t n, uint32_t block, void* stream) {
  if (!ctx || !jobs || n == 0 || n > 2 * ctx->max_tensors) return STQ_EINVAL;
  if (lg_block(block) < 0) return STQ_EBLOCK;
  std::vector<RepackJob> table(n);
  uint64_t total = 0, code_bytes = 0;
  for (uint32_t i = 0; i < n; ++i) {
    const stq_repack_job& j = jobs[i];
    if (!j.src_codes || !j.dst_codes || j.numel == 0 || j.state > 1) return STQ_EINVAL;
    if (int e = check_bits(j.src_bits)) return e;
    if (int e = check_bits(j.dst_bits)) return e;
    if (!aligned(j.src_codes, 256) || !aligned(j.dst_codes, 256)) return STQ_EALIGN;
    const uint64_t tiles = (j.numel + kTile - 1) / kTile;
    if (total + tiles > 0xFFFFFFFFull) return STQ_EINVAL;
    const uintptr_t s0 = reinterpret_cast<uintptr_t>(j.src_codes), s1 = s0 + tiles * 256 * j.src_bits;
    const uintptr_t d0 = reinterpret_cast<uintptr_t>(j.dst_codes), d1 = d0 + tiles * 256 * j.dst_bits;
    if (s0 < d1 && d0 < s1) return STQ_EINVAL;
    RepackJob& r = table[i];
    r.src = static_cast<const uint32_t*>(j.src_codes);
    r.dst = static_cast<uint32_t*>(j.dst_codes);
    r.numel = j.numel;
    r.tile_begin = static_cast<uint32_t>(total);
    r.n_tiles = static_cast<uint32_t>(tiles);
    r.b_old = j.src_bits;
    r.b_new = j.dst_bits;
    r.lut = repack_lut_index(j.state, j.src_bits, j.dst_bits);
    r.pad = 0;
    total += tiles;
    code_bytes += tiles * 256 * (j.src_bits + j.dst_bits);
  }
  DeviceGuard g(ctx->device);
  if (!g.ok) return STQ_EHIP;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (recording(s)) {
    if (launch_upload_by_value(ctx->d_jobs, table.data(), sizeof(RepackJob) * n, stream) != 0) return STQ_EHIP;
  } else {
    int k = -1;
    if (int e = take_slot(ctx->jobs_done, &ctx->jobs_pos, &k)) return e;
    RepackJob* const slot = ctx->h_jobs + 2 * static_cast<size_t>(ctx->max_tensors) * k;
    std::memcpy(slot, table.data(), sizeof(RepackJob) * n);
    const int launched = launch_upload(ctx->d_jobs, slot, sizeof(RepackJob) * n, stream);
    if (int e = slot_in_use(ctx->jobs_done, k, s)) return e;
    if (launched != 0) return STQ_EHIP;
  }
  RepackManyArgs a;
  a.jobs = ctx->d_jobs;
  a.n_jobs = n;
  a.total_tiles = static_cast<uint32_t>(total);
  a.luts = ctx->d_luts;
  return launch_repack_many(a, code_bytes, stream) == 0 ? STQ_OK : STQ_EHIP;
}

}  // extern "C"
