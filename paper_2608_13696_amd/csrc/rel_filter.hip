// Selection vectors of one int32 column against a literal.
//
// rel_filter_compact takes two passes (rel_select.h): a bit per row, then the
// bits as row ids. It is bound by HBM: 4 B per row read, 4 B per selected row
// and 2 bits per row written and read again. 60M rows, 28.2M selected: 68 us
// (5.2 TB/s) against 106 us for the single pass below, whose lanes read 128
// consecutive bytes each and whose tiles wait for their predecessors' counts.
//
// rel_filter_compact_noalloc has too little scratch for a bit per row, so it
// keeps a single pass with decoupled look-back (Merrill and Garland, 2016):
// groups of four consecutive tiles are handed out by an atomic ticket, not by
// blockIdx, so every group a workgroup waits on belongs to a workgroup that is
// already running and that publishes its own count before it looks back: the
// wait always ends. The first wave does the look-back, reading 64 predecessor
// states per round. A thread tests 32 consecutive rows (eight 16-byte loads);
// the tile's selected row numbers are staged in LDS in output order and
// written out by consecutive lanes.
#include <mutex>

#include "rel_device.h"
#include "rel_host.h"
#include "rel_select.h"

namespace {

using namespace rel;

constexpr int kBlock = 256;
constexpr int kIPT = 32;  // rows per thread: eight 16-byte loads
constexpr int64_t kTile = (int64_t)kBlock * kIPT;
// Consecutive tiles a workgroup takes with one ticket. Every ticket is an
// atomic on one cache line, and atomics on one line serialise on this chip
// at about 12 ns each; four tiles per ticket keep that line out of the way.
constexpr int64_t kTilesPerTicket = 4;

template <int OP>
__device__ __forceinline__ bool pred(int32_t v, int32_t lit) {
  if (OP == REL_LT) return v < lit;
  if (OP == REL_LE) return v <= lit;
  if (OP == REL_GT) return v > lit;
  if (OP == REL_GE) return v >= lit;
  if (OP == REL_EQ) return v == lit;
  return v != lit;
}

// First pass: the step's eight loads of a lane are issued before any is
// tested, and all lanes' loads of one chunk are consecutive. Non-temporal:
// 60M rows in 42 us (5.9 TB/s) against 52 us with ordinary loads; sixteen
// loads in flight, or tiles twice as large, measured the same.
template <int OP>
__global__ __launch_bounds__(kSelBlock) void k_filter_bits(const int32_t* __restrict__ col, int64_t n, int32_t lit,
                                                           int64_t tile_rows, uint32_t* __restrict__ bits,
                                                           uint32_t* __restrict__ counts) {
  const int64_t t0 = (int64_t)blockIdx.x * tile_rows;
  const uint32_t wave = threadIdx.x / kWave, lane = lane_id();
  uint32_t c = 0;
  for (int64_t s = 0; s < tile_rows; s += kSelStep) {
    const int64_t base = t0 + s + (int64_t)wave * kSelWaveRows;
    const int64_t r0 = base + 4 * lane;
    uint32_t nib = 0;
    if (base + kSelWaveRows <= n) {
      int4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = ld_once(reinterpret_cast<const int4*>(col + r0 + k * kSelChunk));
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        nib |= (uint32_t)pred<OP>(v[k].x, lit) << (4 * k);
        nib |= (uint32_t)pred<OP>(v[k].y, lit) << (4 * k + 1);
        nib |= (uint32_t)pred<OP>(v[k].z, lit) << (4 * k + 2);
        nib |= (uint32_t)pred<OP>(v[k].w, lit) << (4 * k + 3);
      }
    } else if (base < n) {
      for (int k = 0; k < 8; ++k)
        for (int j = 0; j < 4; ++j) {
          const int64_t r = r0 + k * kSelChunk + j;
          if (r < n) nib |= (uint32_t)pred<OP>(col[r], lit) << (4 * k + j);
        }
    }
    c += store_bits(bits, base, nib);
  }
  store_tile_count(counts, c);
}

// Second pass. A thread holds 64 rows' bits and their place in the output
// (one scan per step). Many selected rows: each wave goes through its 64
// words, one per step, with lane l writing the id of the word's row l; the
// selected ids of 64 rows are consecutive in the output, so every store of a
// wave is one run. That costs about ten instructions per word whatever it
// holds (26 us for 60M rows), so a step with at most kSelSparse of its rows
// selected has each thread list its own word's rows in LDS instead, from
// where they leave with consecutive lanes (8% of 60M rows: 26 -> 12 us; at a
// quarter, where the two meet, the whole filter takes 59 us this way and 65
// us the other).
__global__ __launch_bounds__(kSelBlock) void k_select_expand(const uint64_t* __restrict__ bits,
                                                             const uint32_t* __restrict__ counts, int64_t tile_rows,
                                                             int32_t* __restrict__ out, int64_t* __restrict__ d_count) {
  __shared__ uint32_t s_scan[kSelBlock / kWave];
  __shared__ uint32_t s_red[kSelBlock / kWave];
  __shared__ int32_t s_rows[kSelSparse];
  const int64_t t0 = (int64_t)blockIdx.x * tile_rows;
  uint64_t w = bits[t0 / 64 + threadIdx.x];
  constexpr int kLoads = (int)(kSelMaxTiles / kSelBlock);
  uint32_t part = 0;
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    const uint32_t i = threadIdx.x + k * kSelBlock;
    part += i < blockIdx.x ? counts[i] : 0u;
  }
  part = wave_sum(part);
  if (lane_id() == 0) s_red[threadIdx.x / kWave] = part;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int v = 0; v < kSelBlock / kWave; ++v) before += s_red[v];
  if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) *d_count = (int64_t)before + counts[blockIdx.x];
  const uint32_t lane = lane_id();
  for (int64_t s = 0; s < tile_rows; s += kSelSub) {
    if (s != 0) w = bits[(t0 + s) / 64 + threadIdx.x];
    uint32_t total;
    const uint32_t mine = block_excl_scan<kSelBlock>((uint32_t)__popcll(w), s_scan, &total);
    const uint32_t off = before + mine;
    if (total <= (uint32_t)kSelSparse) {
      const int32_t row = (int32_t)(t0 + s) + (int32_t)threadIdx.x * 64;
      for (uint32_t o = mine; w != 0; w &= w - 1) s_rows[o++] = row + __ffsll((long long)w) - 1;
      __syncthreads();
      for (uint32_t j = threadIdx.x; j < total; j += kSelBlock) out[before + j] = s_rows[j];
      before += total;  // (the next step's scan has a barrier before s_rows is written again)
      continue;
    }
    before += total;
    const uint32_t w_lo = (uint32_t)w, w_hi = (uint32_t)(w >> 32);
    const int32_t row0 = (int32_t)(t0 + s) + (int32_t)(threadIdx.x - lane) * 64 + (int32_t)lane;
#pragma unroll 8
    for (int k = 0; k < kWave; ++k) {
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)w_lo, k);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)w_hi, k);
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)off, k);
      if (__builtin_amdgcn_inverse_ballot_w64((uint64_t)hi << 32 | lo))
        out[__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, o))] = row0 + 64 * k;
    }
  }
}

// Row bits of one thread for one tile: bit k = row r0 + k passes.
template <int OP>
__device__ __forceinline__ uint32_t tile_bits(const int32_t* __restrict__ col, int64_t n, int32_t lit, int64_t r0) {
  uint32_t bits = 0;
  if (r0 + kIPT <= n) {
#pragma unroll
    for (int v = 0; v < kIPT / 4; ++v) {
      const int4 x = *reinterpret_cast<const int4*>(col + r0 + 4 * v);
      bits |= (uint32_t)pred<OP>(x.x, lit) << (4 * v);
      bits |= (uint32_t)pred<OP>(x.y, lit) << (4 * v + 1);
      bits |= (uint32_t)pred<OP>(x.z, lit) << (4 * v + 2);
      bits |= (uint32_t)pred<OP>(x.w, lit) << (4 * v + 3);
    }
  } else {
    for (int k = 0; k < kIPT; ++k)
      if (r0 + k < n) bits |= (uint32_t)pred<OP>(col[r0 + k], lit) << k;
  }
  return bits;
}

// One workgroup per ticket, and a ticket is kTilesPerTicket consecutive
// tiles (a group): the group's rows are all tested first, its count is
// published and looked back once (the look-back state is per group, so no
// group waits on the end of another group's writes), then its tiles are
// staged and written one after another. Per-thread counts of the group's
// tiles travel packed in one 64-bit word, 16 bits per tile (a tile holds at
// most 8192 rows), so one scan serves them all.
template <int OP>
__global__ __launch_bounds__(kBlock) void k_filter_compact(const int32_t* __restrict__ col, int64_t n, int32_t lit,
                                                           int32_t* __restrict__ out, uint64_t* __restrict__ state,
                                                           int64_t* __restrict__ ticket, int64_t* __restrict__ d_count,
                                                           int64_t ngroups) {
  static_assert(kTile < (1 << 16) && kTilesPerTicket * 16 <= 64, "packed per-tile counts");
  __shared__ int64_t s_group;
  __shared__ int64_t s_excl;
  __shared__ uint64_t s_wave[kBlock / kWave];
  __shared__ int32_t s_rows[kTile];
  if (threadIdx.x == 0) s_group = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)ticket, 1ull);
  __syncthreads();
  const int64_t group = s_group;
  const int64_t t0 = group * kTilesPerTicket;
  uint32_t bits[kTilesPerTicket];
  uint64_t c = 0;
#pragma unroll
  for (int g = 0; g < kTilesPerTicket; ++g) {
    const int64_t r0 = (t0 + g) * kTile + (int64_t)threadIdx.x * kIPT;
    bits[g] = r0 < n ? tile_bits<OP>(col, n, lit, r0) : 0u;
    c |= (uint64_t)__popc(bits[g]) << (16 * g);
  }

  // Exclusive scan of the packed counts over the workgroup: wave scan, then wave totals.
  const uint32_t lane = lane_id();
  const uint32_t wave = threadIdx.x / kWave;
  uint64_t incl = c;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint64_t t = (uint64_t)__shfl_up((unsigned long long)incl, o, kWave);
    if (lane >= (uint32_t)o) incl += t;
  }
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  uint64_t wave_off = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kBlock / kWave; ++w) {
    const uint64_t t = s_wave[w];
    wave_off += (uint32_t)w < wave ? t : 0ull;
    total += t;
  }
  const uint64_t my_off = wave_off + incl - c;
  uint32_t group_total = 0;
#pragma unroll
  for (int g = 0; g < kTilesPerTicket; ++g) group_total += (uint32_t)(total >> (16 * g)) & 0xFFFFu;

  // Publish, then look back (the first wave).
  if (wave == 0) {
    const uint64_t excl = lookback_prefix(state, group, group_total);
    if (threadIdx.x == 0) {
      s_excl = (int64_t)excl;
      if (group == ngroups - 1) *d_count = s_excl + group_total;
    }
  }
  uint32_t before = 0;  // rows of the group's earlier tiles
#pragma unroll
  for (int g = 0; g < kTilesPerTicket; ++g) {
    const int64_t r0 = (t0 + g) * kTile + (int64_t)threadIdx.x * kIPT;
    const uint32_t tile_total = (uint32_t)(total >> (16 * g)) & 0xFFFFu;
    uint32_t o = (uint32_t)(my_off >> (16 * g)) & 0xFFFFu;
    for (int k = 0; k < kIPT; ++k)
      if (bits[g] & (1u << k)) s_rows[o++] = (int32_t)(r0 + k);
    __syncthreads();
    int32_t* dst = out + s_excl + before;
    for (uint32_t j = threadIdx.x; j < tile_total; j += kBlock) dst[j] = s_rows[j];
    before += tile_total;
    __syncthreads();  // s_rows is reused by the next tile
  }
}

template <int OP>
void launch_bits(hipStream_t stream, const int32_t* col, int32_t lit, const relh::SelectPlan& p) {
  hipLaunchKernelGGL(k_filter_bits<OP>, dim3((unsigned)p.ntiles), dim3(kSelBlock), 0, stream, col, p.n, lit, p.tile_rows,
                     p.bits, p.counts);
}

void launch_bits_op(hipStream_t stream, rel_cmp op, const int32_t* col, int32_t lit, const relh::SelectPlan& p) {
  switch (op) {
    case REL_LT: launch_bits<REL_LT>(stream, col, lit, p); break;
    case REL_LE: launch_bits<REL_LE>(stream, col, lit, p); break;
    case REL_GT: launch_bits<REL_GT>(stream, col, lit, p); break;
    case REL_GE: launch_bits<REL_GE>(stream, col, lit, p); break;
    case REL_EQ: launch_bits<REL_EQ>(stream, col, lit, p); break;
    case REL_NE: launch_bits<REL_NE>(stream, col, lit, p); break;
  }
}

template <int OP>
void launch(hipStream_t stream, const int32_t* col, int64_t n, int32_t lit, int32_t* out, uint64_t* state,
            int64_t* ticket, int64_t* d_count, int64_t ntiles) {
  const int64_t ngroups = (ntiles + kTilesPerTicket - 1) / kTilesPerTicket;
  hipLaunchKernelGGL(k_filter_compact<OP>, dim3((unsigned)ngroups), dim3(kBlock), 0, stream, col, n, lit, out, state,
                     ticket, d_count, ngroups);
}

void launch_op(hipStream_t stream, rel_cmp op, const int32_t* col, int64_t n, int32_t lit, int32_t* out,
               uint64_t* state, int64_t* ticket, int64_t* d_count, int64_t ntiles) {
  switch (op) {
    case REL_LT: launch<REL_LT>(stream, col, n, lit, out, state, ticket, d_count, ntiles); break;
    case REL_LE: launch<REL_LE>(stream, col, n, lit, out, state, ticket, d_count, ntiles); break;
    case REL_GT: launch<REL_GT>(stream, col, n, lit, out, state, ticket, d_count, ntiles); break;
    case REL_GE: launch<REL_GE>(stream, col, n, lit, out, state, ticket, d_count, ntiles); break;
    case REL_EQ: launch<REL_EQ>(stream, col, n, lit, out, state, ticket, d_count, ntiles); break;
    case REL_NE: launch<REL_NE>(stream, col, n, lit, out, state, ticket, d_count, ntiles); break;
  }
}

// ---- the allocation-free variant ---------------------------------------------------------------------------------------
//
// Its look-back tile states and its ticket live in a fixed device array: word
// 0 is the ticket, words 1.. the states of up to kNoAllocTiles tiles (1 MiB),
// so it compacts at most kNoAllocTiles * kTile = 2^30 rows. Every device that
// runs the library holds its own copy until the process ends. In host code
// the array's name is not a device address; the address is looked up once
// per device (noalloc_scratch_init, from rel_ctx_create) and kept here.
constexpr int64_t kNoAllocTiles = 1 << 17;
constexpr int64_t kNoAllocMaxRows = kNoAllocTiles * kTile;
static __device__ __align__(256) uint64_t scratch[1 + kNoAllocTiles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

namespace relh {

rel_status select_plan(rel_ctx* ctx, int64_t n, SelectPlan* out) {
  SelectPlan p;
  p.n = n;
  p.tile_rows = kSelSub * ((n + kSelSub * kSelMaxTiles - 1) / (kSelSub * kSelMaxTiles));
  p.ntiles = (n + p.tile_rows - 1) / p.tile_rows;
  const int64_t words = p.ntiles * p.tile_rows / 32;
  void* mem;
  const rel_status s = scratch(ctx, SCR_SELECT, (size_t)(words + p.ntiles) * 4, &mem);
  if (s != REL_OK) return s;
  p.bits = (uint32_t*)mem;
  p.counts = p.bits + words;
  *out = p;
  return REL_OK;
}

rel_status select_expand(rel_ctx* ctx, const SelectPlan& p, int32_t* out_idx, int64_t* d_out_count) {
  hipLaunchKernelGGL(k_select_expand, dim3((unsigned)p.ntiles), dim3(kSelBlock), 0, ctx->stream, (const uint64_t*)p.bits,
                     (const uint32_t*)p.counts, p.tile_rows, out_idx, d_out_count);
  REL_LAUNCH_CHECK(ctx, "select_expand");
  return REL_OK;
}

// Looks up this device's copy of the fixed scratch array (the device must be
// current). Called by rel_ctx_create; later calls for the same device return
// at once.
rel_status noalloc_scratch_init(rel_ctx* ctx, int device) {
  if (device < 0 || device >= kMaxDevices) return fail(ctx, REL_UNSUPPORTED, "device index %d above %d", device, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return REL_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(::scratch));
  if (e != hipSuccess || p == nullptr) {
    (void)hipGetLastError();
    return fail(ctx, REL_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", device, hipGetErrorString(e));
  }
  g_scratch_ptr[device] = p;
  return REL_OK;
}

}  // namespace relh

extern "C" rel_status rel_filter_compact(rel_ctx* ctx, const int32_t* col, int64_t n, rel_cmp op, int32_t literal,
                                         int32_t* out_idx, int64_t out_cap, int64_t* d_out_count) {
  if (!ctx || n < 0 || !d_out_count || (n > 0 && (!col || !out_idx)) || op < REL_LT || op > REL_NE)
    return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_compact: bad argument");
  if (col && !relh::aligned16(col)) return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_compact: column not 16-byte aligned");
  if (n >= (1ll << 31)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_filter_compact: n >= 2^31");
  if (out_cap < n) return relh::fail(ctx, REL_CAPACITY, "rel_filter_compact: out_cap < n");
  if (n == 0) return relh::fill_u64(ctx, d_out_count, 1, 0);
  rel_status s;
  relh::SelectPlan p;
  if ((s = relh::select_plan(ctx, n, &p)) != REL_OK) return s;
  relh::KernelTimer kt(ctx, "filter_compact");
  launch_bits_op(ctx->stream, op, col, literal, p);
  REL_LAUNCH_CHECK(ctx, "filter_compact");
  return relh::select_expand(ctx, p, out_idx, d_out_count);
}

// rel_filter_compact with its scratch in the fixed array: no allocation, only
// two fill kernels and the compaction kernel on the context's stream.
extern "C" rel_status rel_filter_compact_noalloc(rel_ctx* ctx, const int32_t* col, int64_t n, rel_cmp op,
                                                 int32_t literal, int32_t* out_idx, int64_t out_cap,
                                                 int64_t* d_out_count) {
  if (!ctx || n < 0 || !d_out_count || (n > 0 && (!col || !out_idx)) || op < REL_LT || op > REL_NE)
    return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_compact_noalloc: bad argument");
  if (n > kNoAllocMaxRows)
    return relh::fail(ctx, REL_UNSUPPORTED, "rel_filter_compact_noalloc: n = %lld above the maximum of %lld rows",
                      (long long)n, (long long)kNoAllocMaxRows);
  if (col && !relh::aligned16(col))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_compact_noalloc: column not 16-byte aligned");
  if (out_cap < n) return relh::fail(ctx, REL_CAPACITY, "rel_filter_compact_noalloc: out_cap < n");
  void* base = (ctx->device >= 0 && ctx->device < kMaxDevices) ? g_scratch_ptr[ctx->device] : nullptr;
  if (!base) return relh::fail(ctx, REL_HIP, "rel_filter_compact_noalloc: scratch address of device %d unknown", ctx->device);
  if (n == 0) return relh::fill_u64(ctx, d_out_count, 1, 0);
  const int64_t ntiles = (n + kTile - 1) / kTile;
  uint64_t* words = (uint64_t*)base;
  // the ticket and this call's tile states start at zero (the array keeps the last call's contents)
  rel_status s = relh::fill_u64(ctx, words, (size_t)(1 + ntiles), 0);
  if (s != REL_OK) return s;
  launch_op(ctx->stream, op, col, n, literal, out_idx, words + 1, (int64_t*)words, d_out_count, ntiles);
  REL_LAUNCH_CHECK(ctx, "filter_compact_noalloc");
  return REL_OK;
}
