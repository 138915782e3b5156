// Host-side internals of librel: the context, its scratch arena, error
// plumbing and launch helpers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/rel.h"

struct ScratchBuf {
  void* ptr = nullptr;
  size_t bytes = 0;
  size_t clean = 0;    // leading bytes known to be empty between calls (tables that their last kernel empties)
  bool dirty = false;  // a call that was to leave them empty has not said so
};

// Scratch slots a context keeps between calls (each grows on demand, never shrinks).
enum ScratchId : int {
  SCR_JOIN_TABLE = 0,  // fused pipeline's join table
  SCR_GROUP_TABLE,     // fused pipeline's group table / per-dim-row aggregates
  SCR_COUNTERS,        // small device counters
  SCR_SCAN_STATE,      // decoupled look-back tile states
  SCR_PART_A,          // partitioned pipeline buffers
  SCR_PART_B,
  SCR_PART_C,
  SCR_PART_D,
  SCR_PART_E,
  SCR_SKETCH,
  SCR_MLP,
  SCR_DENSE,           // dense join index entries
  SCR_WG_COUNTS,       // per-workgroup counts of a streaming kernel
  SCR_GROUP_CLEAN,     // plain path's group table, left empty by its finalize
  SCR_ROW_AGG,         // plain path's per-dim-row aggregates, left zero by its finalize
  SCR_STAGE,           // per-workgroup staged groups for the merge kernel
  SCR_MINMAX,          // per-workgroup key minimum and maximum of the join index build
  SCR_SELECT,          // row bits and tile counts of a selection
  SCR_GROUPBY,         // partitioned rows of a stand-alone group-by
  SCR_COUNT
};

// Device counter words inside SCR_COUNTERS (int64 each).
enum CounterId : int {
  CNT_ROWS_PASSED = 0,
  CNT_JOIN_MATCHES,
  CNT_TICKET,
  CNT_GROUPS,
  CNT_AUX0,
  CNT_AUX1,
  CNT_AUX2,
  CNT_AUX3,
  CNT_WORDS = 16
};

// Per-kernel timing with HIP events recorded on the context's stream around
// each launch (enabled on request; used by the benchmark to time the dominant
// kernel inside the timed region).
struct KernelTiming {
  std::string name;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pending;
  double total_ms = 0.0;
  int64_t launches = 0;
};

struct rel_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  uint64_t stream_turn = 0;  // how often the stream was set: a stream's address may come back as another stream's
  int num_cus = 256;
  size_t lds_per_block = 65536;
  // Device status words (64 x u32, one allocation). Word 0 is the sticky word
  // rel_ctx_sync reads; word 1 belongs to a synchronising fused call, which
  // clears it first and reads it at its end, so that bits left by earlier
  // calls are neither charged to it nor dropped. d_status is the word that
  // kernels launched now report to.
  uint32_t* d_status_words = nullptr;
  uint32_t* d_status = nullptr;
  // Pinned host words that a kernel at the end of a synchronising call writes
  // (kReportWords of them), and whether such a call may have left word 1 set.
  int64_t* report = nullptr;
  bool sync_word_dirty = false;
  std::string err;
  ScratchBuf scratch[SCR_COUNT];
  bool timing = false;
  std::vector<KernelTiming> timings;
  std::vector<hipEvent_t> event_pool;
  // A second stream of the library's own (default priority) for work that can
  // run beside the caller's stream, with the fork / join events; made on first use.
  hipStream_t aux = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // Under table_mu (a table may be destroyed by another thread than the one
  // that uses the context): memory of the last destroyed join table, for the
  // next one of its size, with the stream_turn that it was used in; and the
  // number of join tables alive. A context destroyed before its tables keeps this
  // struct (all else freed) until the last of them is gone.
  std::mutex table_mu;
  ScratchBuf spare;
  uint64_t spare_turn = 0;
  int tables = 0;
  bool closed = false;
};

struct rel_join_table {
  rel_ctx* ctx = nullptr;
  uint64_t* slots = nullptr;
  size_t bytes = 0;
  uint32_t log2cap = 0;
  int64_t m = 0;
  bool may_be_dense = false;  // dense or hash by the keys' range, known on the device only
  bool wide = false;          // built with a payload column
  uint64_t turn = 0;           // the context's stream_turn when it was built
  mutable bool keep = true;    // all its work went to that stream, and none was recorded
};

namespace relh {

constexpr int kReportWords = 8;

rel_status fail(rel_ctx* ctx, rel_status s, const char* fmt, ...);
rel_status hip_fail(rel_ctx* ctx, hipError_t e, const char* what);
// Device buffer of at least `bytes` in scratch slot `id` (contents undefined).
rel_status scratch(rel_ctx* ctx, int id, size_t bytes, void** out);
// Device memory; what the context keeps for a next join table is given back when
// there is none left. REL_OOM otherwise (not noted as the context's error).
rel_status device_alloc(rel_ctx* ctx, size_t bytes, void** out);
// The stream's work is being recorded, not run (or the runtime cannot say).
bool capturing(hipStream_t stream);
// Takes memory that a call can do without: *taken says whether there was any.
template <class Take>
rel_status if_memory(rel_ctx* ctx, Take&& take, bool* taken) {
  const std::string err = ctx->err;
  const rel_status s = take();
  *taken = s == REL_OK;
  if (s != REL_OOM) return s;
  ctx->err = err;  // (no failure of the call's)
  return REL_OK;
}
// Scratch that is empty between calls: every call finds it so and its last
// kernels leave it so, which it tells by scratch_emptied once they are enqueued.
// Memory that is not known to be empty (a first use, a larger one, one after a
// call that failed on the way) is emptied by fill(p). A recorded fill counts for
// the recorded call only: it has not run when the next call is made.
template <class Fill>
rel_status scratch_empty(rel_ctx* ctx, int id, size_t bytes, void** out, Fill&& fill) {
  rel_status s = scratch(ctx, id, bytes, out);
  if (s != REL_OK) return s;
  ScratchBuf& b = ctx->scratch[id];
  if (b.clean < bytes) {
    s = fill(*out);
    if (s == REL_OK && !capturing(ctx->stream)) b.clean = bytes;
  }
  b.dirty = true;
  return s;
}
inline void scratch_emptied(rel_ctx* ctx, int id) { ctx->scratch[id].dirty = false; }
int64_t* counters(rel_ctx* ctx);  // valid after ensure_counters
rel_status ensure_counters(rel_ctx* ctx);

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

inline uint32_t log2_ceil(uint64_t x) {
  uint32_t l = 0;
  while ((1ull << l) < x) ++l;
  return l;
}

// Grid for a grid-stride kernel over `items` work items with `per_block` items per block.
inline unsigned grid_for(const rel_ctx* ctx, int64_t items, int64_t per_block, int blocks_per_cu = 8) {
  int64_t g = (items + per_block - 1) / per_block;
  const int64_t cap = (int64_t)ctx->num_cus * blocks_per_cu;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// Fill helpers (plain kernels, so that the calls stay legal inside a captured graph).
rel_status fill_u64(rel_ctx* ctx, void* p, size_t n_u64, uint64_t v);
// Address of this device's fixed scratch array for the allocation-free entry
// point (rel_filter.hip); the device must be current.
rel_status noalloc_scratch_init(rel_ctx* ctx, int device);
rel_status fill_u32(rel_ctx* ctx, void* p, size_t n_u32, uint32_t v);

// Records a start event on construction and a stop event on destruction when
// the context's timing is enabled; otherwise does nothing.
// aux_fork orders the auxiliary stream after the work already on ctx->stream
// (creating it on first use); aux_join makes ctx->stream wait for everything
// enqueued on the auxiliary stream since.
rel_status aux_fork(rel_ctx* ctx);
rel_status aux_join(rel_ctx* ctx);

class KernelTimer {
 public:
  KernelTimer(rel_ctx* ctx, const char* name);
  ~KernelTimer();

 private:
  rel_ctx* ctx_;
  int slot_ = -1;
  hipEvent_t start_ = nullptr;
};

}  // namespace relh

#define REL_HIP_CHECK(ctx, expr)                                 \
  do {                                                           \
    hipError_t e_ = (expr);                                      \
    if (e_ != hipSuccess) return relh::hip_fail((ctx), e_, #expr); \
  } while (0)

#define REL_LAUNCH_CHECK(ctx, what)                                 \
  do {                                                              \
    hipError_t e_ = hipGetLastError();                              \
    if (e_ != hipSuccess) return relh::hip_fail((ctx), e_, (what)); \
  } while (0)
