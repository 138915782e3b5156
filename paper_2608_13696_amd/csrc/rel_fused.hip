// The fused filter -> probe -> aggregate pipeline (build, one streaming
// kernel, finalize) and the standalone hash group-by.
//
// The streaming kernel reads the fact columns once with 16-byte vector loads,
// several rows per thread (the paper's Recommendation 1: overlap latency with
// instruction-level parallelism), evaluates the compiled predicate, probes the
// join table and updates the group state:
//   * few groups: a per-workgroup LDS table (the shared-memory aggregation of
//     Section 7); a workgroup that ends with few groups stages them with plain
//     stores and one workgroup merges the stages, else it flushes its table
//     to device memory;
//   * many groups: a device-memory table updated with device-scope atomics;
//   * group key == join key (GROUP BY fk): a groupjoin, aggregating straight
//     into per-dim-row accumulators so no second hash table exists.
#include <algorithm>

#include "rel_device.h"
#include "rel_host.h"
#include "rel_ops.h"

namespace {

using namespace rel;

enum Mode : int { M_PRIO_FLAG = REL_GROUP_PRIO_FLAG, M_FK = REL_GROUP_FK, M_DIM_GRP = REL_GROUP_DIM_GRP };
enum GPlace : int { G_LDS = 0, G_GLOBAL = 1, G_ROWAGG = 2 };

constexpr int kBlock = 256;
constexpr int kLdsBlock = 1024;  // fused kernel with an LDS group table over many rows: one workgroup per CU
constexpr int kIPT = 4;  // rows per thread per tile: one 16-byte load per int32 column
constexpr int kLdsSlots = 1024;
constexpr int kLdsProbe = 32;
constexpr int kLdsCacheProbe = 4;
// A table sized from a prediction gives up after this many probe steps (at a
// load of 0.5 linear probing practically never walks that far), so that an
// undersized table reports overflow instead of degrading to a linear scan.
constexpr uint32_t kPlannedProbe = 256;
// Groups a workgroup of the LDS variant may stage for the merge kernel (more
// and it adds them to the device table itself): 32 with a full grid, and as
// many more with fewer workgroups as keep the merge's work the same, up to half
// of what the merge's LDS table holds (a workgroup that has more would only have
// the one that merges add to the device table for it: 5000 rows, 3600 groups: 74
// us without that limit, 37 with it).
constexpr int kStageMax = 32;
constexpr int kStageTotal = 256 * kStageMax;

// Where the LDS variant's workgroups leave their groups: `cap` slots and a
// number per workgroup, and a word set when any row or group went to the
// device table instead.
struct Stage {
  GroupSlot* slots;
  uint32_t* n;
  int32_t cap;
  uint32_t* touched;
};

struct FusedArgs {
  const int32_t* fk;
  const int64_t* price;
  const int32_t* qty;
  const int32_t* day;
  const int8_t* flag;
  int64_t n;
  int32_t day_lt;
  JoinIndex join;
  GroupView groups;
  RowAgg* row_agg;
  uint64_t* wg_counts;  // per workgroup: rows passed, join matches, dense index entries
  Stage stage;  // LDS variant
  int32_t lds_probe;  // LDS probe budget before a row goes to device memory
};

template <int MODE>
__device__ __forceinline__ int64_t group_key(int32_t payload, int32_t fk, int8_t flag) {
  if (MODE == M_PRIO_FLAG) return (int64_t)payload * 256 + (int64_t)(uint8_t)flag;
  if (MODE == M_DIM_GRP) return (int64_t)payload;
  return (int64_t)fk;
}

// One thread's rows of a tile: kIPT consecutive rows, loaded with 16-byte loads.
// `once`: non-temporal ones, which leave L2 to a dense join index and an LDS group
// table's few device rows (6M rows: the whole query 75.3 us against 80.7 with
// ordinary ones; the same when the columns are in the last-level cache). Beside a
// hash index, which L2 does not hold, or a group table in device memory ordinary
// ones are better (4.7M rows, 853K sparse keys: 95.2 against 98.1 us; 571K rows
// into 294 groups of a device table: 339.6 against 344.3).
struct FusedRows {
  int32_t d[kIPT], f[kIPT], q[kIPT];
  int64_t p[kIPT];
  uint32_t fl;  // the four flag bytes
  int nv;       // rows in range
};

template <int MODE>
__device__ __forceinline__ void load_fused(const FusedArgs& a, int64_t r0, bool once, FusedRows& r) {
  if (r0 + kIPT <= a.n) {
    r.nv = kIPT;
    int4 dv, fv, qv;
    longlong2 p01, p23;
    if (once) {
      dv = ld_once(reinterpret_cast<const int4*>(a.day + r0));
      fv = ld_once(reinterpret_cast<const int4*>(a.fk + r0));
      qv = ld_once(reinterpret_cast<const int4*>(a.qty + r0));
      p01 = ld_once(reinterpret_cast<const longlong2*>(a.price + r0));
      p23 = ld_once(reinterpret_cast<const longlong2*>(a.price + r0 + 2));
    } else {
      dv = *reinterpret_cast<const int4*>(a.day + r0);
      fv = *reinterpret_cast<const int4*>(a.fk + r0);
      qv = *reinterpret_cast<const int4*>(a.qty + r0);
      p01 = *reinterpret_cast<const longlong2*>(a.price + r0);
      p23 = *reinterpret_cast<const longlong2*>(a.price + r0 + 2);
    }
    r.d[0] = dv.x; r.d[1] = dv.y; r.d[2] = dv.z; r.d[3] = dv.w;
    r.f[0] = fv.x; r.f[1] = fv.y; r.f[2] = fv.z; r.f[3] = fv.w;
    r.q[0] = qv.x; r.q[1] = qv.y; r.q[2] = qv.z; r.q[3] = qv.w;
    r.p[0] = p01.x; r.p[1] = p01.y; r.p[2] = p23.x; r.p[3] = p23.y;
    r.fl = MODE == M_PRIO_FLAG ? *reinterpret_cast<const uint32_t*>(a.flag + r0) : 0u;
  } else {
    r.nv = r0 < a.n ? (int)(a.n - r0) : 0;
    r.fl = 0;
#pragma unroll
    for (int k = 0; k < kIPT; ++k) {
      const bool ok = k < r.nv;
      r.d[k] = ok ? a.day[r0 + k] : 0;
      r.f[k] = ok ? a.fk[r0 + k] : 0;
      r.q[k] = ok ? a.qty[r0 + k] : 0;
      r.p[k] = ok ? a.price[r0 + k] : 0;
      if (MODE == M_PRIO_FLAG && ok) r.fl |= (uint32_t)(uint8_t)a.flag[r0 + k] << (8 * k);
    }
  }
}

// End of the LDS variant: a table holding at most `cap` groups is compacted
// into the workgroup's stage, and their number (0 otherwise) goes to stage_n; a
// fuller one goes to the device table with atomics. Few groups shared by every
// workgroup would otherwise mean hundreds of workgroups adding into the same
// few device slots at the kernel's end, and atomics on one cache line
// serialise (about 12 ns each on this chip).
template <int NT>
__device__ void stage_or_flush(LdsGroups<kLdsSlots>& lds, const GroupView& groups, const Stage& st, uint64_t dev_rows) {
  static_assert(kLdsSlots % NT == 0, "whole LDS slots per thread");
  constexpr int kPer = kLdsSlots / NT;
  __shared__ uint32_t s_scan[NT / kWave];
  __shared__ uint64_t s_red[NT / kWave];
  const int t = threadIdx.x;
  uint32_t mine = 0, total;
#pragma unroll
  for (int k = 0; k < kPer; ++k) mine += lds.count[t + k * NT] != 0;
  uint32_t pos = block_excl_scan<NT>(mine, s_scan, &total);
  dev_rows = block_sum_u64<NT>(dev_rows, s_red);
  const bool fits = total <= (uint32_t)st.cap;
  GroupSlot* to = st.slots + (int64_t)blockIdx.x * st.cap;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int s = t + k * NT;
    if (lds.count[s] == 0) continue;
    if (fits) to[pos++] = GroupSlot{lds.key[s], lds.sum_price[s], lds.sum_qty[s], lds.count[s]};
    else group_add(groups, lds.key[s], lds.sum_price[s], lds.sum_qty[s], lds.count[s]);
  }
  if (t == 0) {
    st.n[blockIdx.x] = fits ? total : 0u;
    if (dev_rows != 0 || !fits) *st.touched = 1u;
  }
}

// Persistent: each workgroup walks tiles with a grid stride and loads its next
// tile while it probes and aggregates the current one. With an LDS group
// table there is one large workgroup per CU, so the table is flushed to device
// memory once per CU (few groups means few, heavily shared device slots).
template <int MODE, int GP, int NT>
__global__ __launch_bounds__(NT) void k_fused(FusedArgs a) {
  __shared__ LdsGroups<GP == G_LDS ? kLdsSlots : 1> lds;
  if (GP == G_LDS) {
    lds.init(threadIdx.x, NT);
    __syncthreads();
  }
  uint64_t passed = 0, matched = 0, dev_rows = 0;
  const DenseRange dr = dense_range(a.join);
  const bool once = GP == G_LDS && dr.dense;
  constexpr int64_t tile_rows = (int64_t)NT * kIPT;
  const int64_t ntiles = (a.n + tile_rows - 1) / tile_rows;
  int64_t tile = blockIdx.x;
  FusedRows cur, nxt;
  if (tile < ntiles) load_fused<MODE>(a, tile * tile_rows + (int64_t)threadIdx.x * kIPT, once, cur);
  // this workgroup's share of the dense index's duplicate check (a count of
  // its entries), while its first tile loads
  uint64_t entries = 0;
  if (dr.dense) {
    const int64_t words = dense_words(a.join, dr);
    const int64_t per = (words + gridDim.x - 1) / gridDim.x;
    const int64_t w0 = (int64_t)blockIdx.x * per;
    entries = dense_count_entries<NT>(a.join, w0, min(words, w0 + per));
  }
  for (; tile < ntiles; tile += gridDim.x) {
    const int64_t tn = tile + gridDim.x;
    if (tn < ntiles) load_fused<MODE>(a, tn * tile_rows + (int64_t)threadIdx.x * kIPT, once, nxt);
    // every row's first join read (its dense entry, or its first hash slot)
    // is issued before any is examined, so the tile's random reads overlap
    // instead of following one another
    bool pass[kIPT];
    uint64_t first[kIPT];
#pragma unroll
    for (int k = 0; k < kIPT; ++k) {
      pass[k] = k < cur.nv && cur.d[k] < a.day_lt;
      if (dr.dense) first[k] = pass[k] ? dense_entry(a.join, dr, cur.f[k]) : 0u;
      else first[k] = pass[k] ? a.join.hash.slots[join_first_index(a.join.hash, cur.f[k])] : kJoinEmpty;
    }
#pragma unroll
    for (int k = 0; k < kIPT; ++k) {
      // no early exits: the device-memory update below is a wave-wide call
      passed += pass[k];
      int32_t pl = 0;
      bool hit;
      if (dr.dense) {
        hit = first[k] != 0;
        if (hit) pl = dense_payload(a.join, (uint32_t)first[k]);
      } else {
        hit = pass[k] && join_finish(a.join.hash, cur.f[k], first[k], &pl);
      }
      matched += hit;
      const uint64_t sp = (uint64_t)cur.p[k], sq = (uint64_t)(int64_t)cur.q[k];
      if (GP == G_ROWAGG) {
        if (hit) {
          RowAgg* r = &a.row_agg[pl];
          dev_add<uint64_t>(&r->sum_price, sp);
          dev_add<uint64_t>(&r->sum_qty, sq);
          dev_add<uint64_t>(&r->count, 1ull);
        }
      } else {
        const int64_t key = hit ? group_key<MODE>(pl, cur.f[k], (int8_t)(cur.fl >> (8 * k))) : 0;
        bool global = hit;
        if (GP == G_LDS && hit) {
          const int s = lds.find(key, a.lds_probe);
          if (s >= 0) {
            lds.add(s, sp, sq, 1ull);
            global = false;
          }
        }
        if (GP == G_LDS) dev_rows += global;
        group_add_wave(a.groups, global, key, sp, sq);
      }
    }
    cur = nxt;
  }
  if constexpr (GP == G_LDS) {
    __syncthreads();
    stage_or_flush<NT>(lds, a.groups, a.stage, dev_rows);
  }
  // the totals go out with plain stores, one triple per workgroup; the merge
  // or finalize kernel adds them up
  __shared__ uint64_t s_red[3][NT / kWave];
  passed = block_sum_u64<NT>(passed, s_red[0]);
  matched = block_sum_u64<NT>(matched, s_red[1]);
  entries = block_sum_u64<NT>(entries, s_red[2]);
  if (threadIdx.x == 0) {
    a.wg_counts[3 * blockIdx.x] = passed;
    a.wg_counts[3 * blockIdx.x + 1] = matched;
    a.wg_counts[3 * blockIdx.x + 2] = entries;
  }
}

// One workgroup merges the stages of the LDS variant in its own LDS table.
// When nothing went to the device table and every merged group found an LDS
// slot, it writes the output itself (groups, their number, the two counters)
// and sets `done`, and the finalize kernel returns at once; otherwise it adds
// its groups to the device table and the finalize kernel (or, where none
// follows, this launch) scans that. Other workgroups of the launch empty the
// join index meanwhile.
constexpr int kMergeUnroll = 4;
constexpr int kMaxStages = 1024;  // streaming workgroups at most

struct MergeArgs {
  Stage stage;
  int64_t n_wg;
  const uint64_t* wg_counts;  // (null: none)
  int64_t* counters;
  GroupView groups;
  uint32_t* done;
  JoinIndex join;  // for the dense index's entry count
  const uint32_t* few;  // clear: the stages were not written (null: they were)
  // where no finalize kernel follows: when groups went to the device table, the
  // others write the output from its nslots slots, on the merging workgroup's word
  int64_t nslots;
  uint32_t* ticket;
  uint32_t* word;
};
enum MergeWord : uint32_t { kMergePending = 0, kMergeWritten, kMergeDrain };

// The per-workgroup counts summed by NT threads (valid in thread 0): rows
// passed and join matches into counters[0] and [1]; a dense index with fewer
// entries than build rows had a repeated key.
template <int NT>
__device__ void sum_totals(uint64_t p, uint64_t q, uint64_t e, bool write, const JoinIndex& jx, int64_t* counters,
                           uint32_t* status) {
  __shared__ uint64_t s_red[3][NT / kWave];
  p = wave_sum_u64(p);
  q = wave_sum_u64(q);
  e = wave_sum_u64(e);
  if (lane_id() == 0) {
    s_red[0][threadIdx.x / kWave] = p;
    s_red[1][threadIdx.x / kWave] = q;
    s_red[2][threadIdx.x / kWave] = e;
  }
  __syncthreads();
  if (threadIdx.x != 0 || !write) return;
  p = q = e = 0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) {
    p += s_red[0][w];
    q += s_red[1][w];
    e += s_red[2][w];
  }
  counters[0] = (int64_t)p;
  counters[1] = (int64_t)q;
  if (jx.mm != nullptr && dense_range(jx).dense && e != (uint64_t)jx.m) set_status(status, kDevDupKey);
}

template <int NT>
__device__ void sum_wg_counts(const uint64_t* wg, int64_t n_wg, const JoinIndex& jx, int64_t* counters,
                              uint32_t* status) {
  uint64_t p = 0, q = 0, e = 0;
  for (int64_t i = threadIdx.x; i < n_wg; i += NT) {
    p += wg[3 * i];
    q += wg[3 * i + 1];
    e += wg[3 * i + 2];
  }
  sum_totals<NT>(p, q, e, true, jx, counters, status);
}

struct OutArgs;

// Stand-alone group-by over key[row], row = sel ? sel[k] : k, straight into the
// device table.
__device__ __forceinline__ void groupby_device(const relh::GroupRows& in, const GroupView& g) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < in.n; k += stride) {
    const int64_t row = in.sel ? (int64_t)in.sel[k] : k;
    group_add(g, in.key[row], (uint64_t)in.price[row], (uint64_t)(int64_t)in.qty[row], 1ull);
  }
}

__global__ __launch_bounds__(kBlock) void k_groupby_global(relh::GroupRows in, GroupView g) { groupby_device(in, g); }

// The same through an LDS table per workgroup, with the device table behind
// it; groups leave as in the fused kernel's LDS variant (stage_or_flush).
// kGbAhead rows per thread are loaded before any is added: 4.2M selected rows
// of 15 groups take 26 us (125 us with one row at a time in 256-thread
// workgroups that each flushed to the device table).
constexpr int kGbAhead = 4;
__global__ __launch_bounds__(kLdsBlock) void k_groupby_lds(relh::GroupRows in, const uint32_t* __restrict__ few, GroupView g,
                                                           int32_t probe, bool device_if_many,
                                                           Stage st) {
  __shared__ LdsGroups<kLdsSlots> lds;
  if (*few == 0) {
    if (device_if_many) groupby_device(in, g);
    return;
  }
  lds.init(threadIdx.x, kLdsBlock);
  __syncthreads();
  uint64_t dev_rows = 0;
  const int64_t step = (int64_t)gridDim.x * kLdsBlock;
  for (int64_t k0 = blockIdx.x * (int64_t)kLdsBlock + threadIdx.x; k0 < in.n; k0 += kGbAhead * step) {
    int64_t row[kGbAhead], key[kGbAhead];
    uint64_t sp[kGbAhead], sq[kGbAhead];
#pragma unroll
    for (int u = 0; u < kGbAhead; ++u) {
      const int64_t k = k0 + u * step;
      row[u] = k < in.n ? (in.sel ? (int64_t)in.sel[k] : k) : -1;
    }
#pragma unroll
    for (int u = 0; u < kGbAhead; ++u) {
      const int64_t r = row[u] >= 0 ? row[u] : 0;
      key[u] = in.key[r];
      sp[u] = (uint64_t)in.price[r];
      sq[u] = (uint64_t)(int64_t)in.qty[r];
    }
#pragma unroll
    for (int u = 0; u < kGbAhead; ++u) {
      if (row[u] < 0) continue;
      const int s = key[u] != kGroupEmpty ? lds.find(key[u], probe) : -1;
      if (s >= 0) {
        lds.add(s, sp[u], sq[u], 1ull);
      } else {
        group_add(g, key[u], sp[u], sq[u], 1ull);
        ++dev_rows;
      }
    }
  }
  __syncthreads();
  stage_or_flush<kLdsBlock>(lds, g, st, dev_rows);
}

__global__ void k_init_groups(GroupSlot* __restrict__ slots, int64_t nslots) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < nslots; i += stride) {
    GroupSlot s;
    s.key = kGroupEmpty;
    s.sum_price = 0;
    s.sum_qty = 0;
    s.count = 0;
    slots[i] = s;
  }
}

struct OutArgs {
  int64_t* key;
  int64_t* sum_price;
  int64_t* sum_qty;
  int64_t* count;
  int64_t cap;
  int64_t* d_n;
  uint32_t* status;
  // the streaming kernel's per-workgroup (rows passed, join matches), summed
  // into counters[0] and [1] by the first group of tiles; n_wg = 0: none
  const uint64_t* wg_counts;
  int64_t n_wg;
  int64_t* counters;
  const uint32_t* done;  // set: the merge kernel wrote the output (may be null)
  JoinIndex join;        // for the dense index's entry count (mm null: none)
  const uint64_t* base;  // groups that were written before this kernel's, which follow them (may be null)
  const uint32_t* touched;  // with base: clear when the table holds no group
  int64_t limit;            // with base: more groups than this overflow the table that the caller sized
};

// Part `part` of `parts` of the device table's groups to the output, by one
// workgroup, leaving them empty; *o.d_n counts the groups. The slots are read
// past L1, which may hold what they were before other workgroups' atomics.
__device__ __forceinline__ void drain_groups(const GroupView& g, int64_t nslots, uint32_t part, uint32_t parts, const OutArgs& o) {
  __shared__ uint32_t s_scan[kLdsBlock / kWave];
  __shared__ int64_t s_pos;
  constexpr int kAhead = 8;
  const int64_t step = kAhead * kLdsBlock;
  for (int64_t i0 = part * step; i0 < nslots; i0 += parts * step) {
    uint64_t c[kAhead];
    uint32_t bits = 0, total;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int64_t i = i0 + k * kLdsBlock + threadIdx.x;
      c[k] = i < nslots ? __hip_atomic_load(&g.slots[i].count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) bits |= (uint32_t)(c[k] != 0) << k;
    const uint32_t before = block_excl_scan<kLdsBlock>((uint32_t)__popc(bits), s_scan, &total);
    if (total == 0) continue;
    if (threadIdx.x == 0) s_pos = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)o.d_n, total);
    __syncthreads();
    int64_t pos = s_pos + before;
#pragma unroll 1
    for (; bits != 0; bits &= bits - 1, ++pos) {
      const int64_t i = i0 + (__ffs((int)bits) - 1) * kLdsBlock + threadIdx.x;
      GroupSlot* s = &g.slots[i];
      if (pos < o.cap) {
        o.key[pos] = i == nslots - 1 ? kGroupEmpty : __hip_atomic_load(&s->key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        o.sum_price[pos] = (int64_t)__hip_atomic_load(&s->sum_price, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        o.sum_qty[pos] = (int64_t)__hip_atomic_load(&s->sum_qty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        o.count[pos] = (int64_t)__hip_atomic_load(&s->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        set_status(o.status, kDevOverflow);
      }
      *s = GroupSlot{kGroupEmpty, 0, 0, 0};
    }
  }
}

// ENDS: no finalize kernel follows (MergeArgs::nslots).
template <bool ENDS>
__global__ __launch_bounds__(kLdsBlock) void k_group_merge(MergeArgs m, OutArgs o) {
  __shared__ LdsGroups<kLdsSlots> lds;
  __shared__ uint32_t s_lost;  // a group went to the device table here
  __shared__ uint32_t s_wcnt[kLdsBlock / kWave];
  const int t = threadIdx.x;
  if (!ENDS && blockIdx.x > 0) {
    join_index_wipe(m.join, (int64_t)(blockIdx.x - 1) * kLdsBlock + t, (int64_t)(gridDim.x - 1) * kLdsBlock);
    return;
  }
  if (!ENDS && m.few != nullptr && *m.few == 0) return;
  // the loads that nothing before them decides, in flight while the table is set
  // up; among them this workgroup's turn: the others wait for the word of the one
  // that merges, so that is one that runs, the first to start
  __shared__ uint32_t s_role;
  uint32_t turn = 0;
  if (ENDS && t == 0) turn = dev_add_ret<uint32_t>(m.ticket, 1u);
  const uint32_t touched = *m.stage.touched;
  const uint32_t c0 = t < m.n_wg ? m.stage.n[t] : 0u;
  uint64_t wp = 0, wq = 0, we = 0;  // this thread's share of the streaming workgroups' totals (at most one each)
  if (m.wg_counts && t < m.n_wg) {
    wp = m.wg_counts[3 * t];
    wq = m.wg_counts[3 * t + 1];
    we = m.wg_counts[3 * t + 2];
  }
  lds.init(t, kLdsBlock);
  if (t == 0) s_lost = 0;
  // The stages' groups laid end to end, each stage padded to the largest one's
  // size rounded up to a power of two: all threads load a few each.
  static_assert(kMaxStages == kLdsBlock, "one stage per thread");
  __shared__ uint32_t s_cnt[kMaxStages];
  __shared__ uint32_t s_most[kLdsBlock / kWave];
  {
    uint32_t most = c0;
    s_cnt[t] = c0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, d, kWave));
    if (lane_id() == 0) s_most[t / kWave] = most;
  }
  if (ENDS && t == 0) s_role = turn;
  __syncthreads();
  if constexpr (ENDS) {
    const uint32_t role = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_role);
    if (role > 0) {
      join_index_wipe(m.join, (int64_t)(role - 1) * kLdsBlock + t, (int64_t)(gridDim.x - 1) * kLdsBlock);
      __shared__ uint32_t s_word;
      if (t == 0) {
        uint32_t w;
        while ((w = __hip_atomic_load(m.word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == kMergePending) __builtin_amdgcn_s_sleep(4);
        s_word = w;
      }
      __syncthreads();
      if (s_word == kMergeDrain) drain_groups(m.groups, m.nslots, role - 1, gridDim.x - 1, o);
      return;
    }
  }
  uint32_t most = 0;
#pragma unroll
  for (int w = 0; w < kLdsBlock / kWave; ++w) most = max(most, s_most[w]);
  const uint32_t lb = most > 1 ? 32u - (uint32_t)__clz((int)(most - 1)) : 0u;
  const uint32_t nflat = most > 0 ? (uint32_t)m.n_wg << lb : 0u;
  for (uint32_t f0 = t; f0 - t < nflat; f0 += kLdsBlock * kMergeUnroll) {
    GroupSlot e[kMergeUnroll];
#pragma unroll
    for (int u = 0; u < kMergeUnroll; ++u) {
      const uint32_t f = f0 + u * kLdsBlock, w = f >> lb, j = f & ((1u << lb) - 1u);
      if (f < nflat && j < s_cnt[w]) e[u] = m.stage.slots[(int64_t)w * m.stage.cap + j];
      else e[u].count = 0;
    }
#pragma unroll
    for (int u = 0; u < kMergeUnroll; ++u) {
      if (e[u].count == 0) continue;
      const int s = lds.find(e[u].key, kLdsProbe);
      if (s >= 0) {
        lds.add(s, e[u].sum_price, e[u].sum_qty, e[u].count);
      } else {
        group_add(m.groups, e[u].key, e[u].sum_price, e[u].sum_qty, e[u].count);
        s_lost = 1;
      }
    }
  }
  // the streaming kernel's per-workgroup counts (the barriers inside also end
  // the merge)
  sum_totals<kLdsBlock>(wp, wq, we, m.wg_counts != nullptr, m.join, m.counters, o.status);
  const bool occ = lds.count[t] != 0;
  if (touched != 0 || s_lost != 0) {
    if (t == 0) *m.stage.touched = 1u;
    if (occ) group_add(m.groups, lds.key[t], lds.sum_price[t], lds.sum_qty[t], lds.count[t]);
    if (!ENDS) return;
    if (t == 0) __hip_atomic_store((unsigned long long*)o.d_n, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_device_atomics();  // (every wave's, before the word goes out)
    __syncthreads();
    if (t == 0) __hip_atomic_store(m.word, (uint32_t)kMergeDrain, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  // (at once: the others' way out is as long as what is left here)
  if (ENDS && t == 0) __hip_atomic_store(m.word, (uint32_t)kMergeWritten, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t ball = wave_ballot(occ);
  const uint32_t wave = t / kWave;
  if (lane_id() == 0) s_wcnt[wave] = (uint32_t)__popcll(ball);
  __syncthreads();
  uint32_t total = 0, before = 0;
#pragma unroll
  for (uint32_t w = 0; w < kLdsBlock / kWave; ++w) {
    const uint32_t c = s_wcnt[w];
    before += w < wave ? c : 0u;
    total += c;
  }
  if (occ) {
    const int64_t pos = before + mask_rank(ball);
    if (pos < o.cap) {
      o.key[pos] = lds.key[t];
      o.sum_price[pos] = (int64_t)lds.sum_price[t];
      o.sum_qty[pos] = (int64_t)lds.sum_qty[t];
      o.count[pos] = (int64_t)lds.count[t];
    } else {
      set_status(o.status, kDevOverflow);
    }
  }
  if (t == 0) {
    *o.d_n = (int64_t)total;
    *m.done = 1u;
  }
}

// Group finalization: stream compaction of the occupied slots into the
// output. Each workgroup takes a group of kFinTilesPerTicket consecutive
// tiles by ticket, counts the group's occupied slots (per tile, packed 16
// bits a tile in one word for a single scan),
// and finds its output offset by decoupled look-back, so no single output
// counter is contended. A thread's slots are kBlock apart, so each count read
// of a wave covers consecutive slots; the groups come out in tile order and,
// inside a tile, thread by thread (the output order is unspecified).
constexpr int kFinIPT = 8;
constexpr int64_t kFinTile = (int64_t)kBlock * kFinIPT;
// Consecutive tiles per ticket (one look-back per group of them): tickets
// are atomics on one cache line, which serialise on this chip at about 12 ns
// each.
constexpr int64_t kFinTilesPerTicket = 4;

// Group table; the last slot holds the key INT64_MIN. With `clean` each slot
// read is emptied again, so that the table needs no clearing before its next
// use (only occupied slots are written, instead of the whole table).
struct SlotSource {
  GroupSlot* slots;
  int64_t side;
  bool clean;
  __device__ bool occupied(int64_t i) const { return slots[i].count != 0; }
  __device__ void get(int64_t i, int64_t* key, uint64_t* sp, uint64_t* sq, uint64_t* cnt) const {
    const GroupSlot g = slots[i];
    *key = i == side ? kGroupEmpty : g.key;
    *sp = g.sum_price;
    *sq = g.sum_qty;
    *cnt = g.count;
    drop(i);
  }
  __device__ void drop(int64_t i) const {  // (a group past the output's end, too)
    if (clean) slots[i] = GroupSlot{kGroupEmpty, 0, 0, 0};
  }
};

struct RowAggSource {  // groupjoin accumulators, zeroed as they are read; the key is the dim row's pk
  RowAgg* agg;
  const int32_t* pk;
  __device__ bool occupied(int64_t i) const { return agg[i].count != 0; }
  __device__ void get(int64_t i, int64_t* key, uint64_t* sp, uint64_t* sq, uint64_t* cnt) const {
    const RowAgg r = agg[i];
    *key = pk[i];
    *sp = r.sum_price;
    *sq = r.sum_qty;
    *cnt = r.count;
    drop(i);
  }
  __device__ void drop(int64_t i) const { agg[i] = RowAgg{0, 0, 0}; }
};

// (four waves per SIMD: with 156 registers instead of 128 it took 114 us instead of 101 over 2M slots)
template <class Src>
__global__ __launch_bounds__(kBlock, 4) void k_finalize(Src src, int64_t nitems, OutArgs o, uint64_t* __restrict__ state,
                                                     int64_t* __restrict__ ticket, int64_t ngroups) {
  static_assert(kFinTile < (1 << 16) && kFinTilesPerTicket * 16 <= 64, "packed per-tile counts");
  __shared__ int64_t s_group;
  __shared__ uint64_t s_excl;
  __shared__ uint64_t s_wave[kBlock / kWave];
  if (o.done != nullptr && *o.done != 0) return;
  const uint64_t base = o.base != nullptr ? *o.base : 0ull;
  if (o.base != nullptr && *o.touched == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      *o.d_n = (int64_t)base;
      if ((int64_t)base > o.limit) set_status(o.status, kDevOverflow);
    }
    return;
  }
  if (threadIdx.x == 0) s_group = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)ticket, 1ull);
  __syncthreads();
  const int64_t group = s_group;
  const int64_t t0 = group * kFinTilesPerTicket;
  uint32_t bits[kFinTilesPerTicket];
  uint64_t c = 0;
#pragma unroll
  for (int g = 0; g < kFinTilesPerTicket; ++g) {
    const int64_t i0 = (t0 + g) * kFinTile + (int64_t)threadIdx.x;  // slot of bit k: i0 + k * kBlock
    bits[g] = 0;
#pragma unroll
    for (int k = 0; k < kFinIPT; ++k) {
      const int64_t i = i0 + (int64_t)k * kBlock;
      if (i < nitems && src.occupied(i)) bits[g] |= 1u << k;
    }
    c |= (uint64_t)__popc(bits[g]) << (16 * g);
  }
  const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
  uint64_t incl = c;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint64_t t = (uint64_t)__shfl_up((unsigned long long)incl, d, kWave);
    if (lane >= (uint32_t)d) incl += t;
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
  for (int g = 0; g < kFinTilesPerTicket; ++g) group_total += (uint32_t)(total >> (16 * g)) & 0xFFFFu;
  if (wave == 0) {
    const uint64_t excl = lookback_prefix(state, group, group_total);
    if (threadIdx.x == 0) {
      s_excl = base + excl;
      if (group == ngroups - 1) {
        *o.d_n = (int64_t)(base + excl + group_total);
        if (o.base != nullptr && *o.d_n > o.limit) set_status(o.status, kDevOverflow);
      }
    }
  }
  __syncthreads();
  int64_t before = 0;  // groups of the earlier tiles of this ticket
#pragma unroll
  for (int g = 0; g < kFinTilesPerTicket; ++g) {
    const int64_t i0 = (t0 + g) * kFinTile + (int64_t)threadIdx.x;
    int64_t pos = (int64_t)s_excl + before + (int64_t)((my_off >> (16 * g)) & 0xFFFFu);
    for (int k = 0; k < kFinIPT; ++k) {
      if (!(bits[g] & (1u << k))) continue;
      if (pos < o.cap) {
        int64_t key;
        uint64_t sp, sq, cnt;
        src.get(i0 + (int64_t)k * kBlock, &key, &sp, &sq, &cnt);
        o.key[pos] = key;
        o.sum_price[pos] = (int64_t)sp;
        o.sum_qty[pos] = (int64_t)sq;
        o.count[pos] = (int64_t)cnt;
      } else {
        src.drop(i0 + (int64_t)k * kBlock);
        set_status(o.status, kDevOverflow);
      }
      ++pos;
    }
    before += (total >> (16 * g)) & 0xFFFFu;
  }
  // (as the merge kernel does when there is one)
  if (group == 0 && o.n_wg > 0) sum_wg_counts<kBlock>(o.wg_counts, o.n_wg, o.join, o.counters, o.status);
}

// Tiles of the finalize kernel over nitems slots (with no items, one empty
// tile still sums the per-workgroup counts), and its look-back state.
int64_t finalize_tiles(int64_t nitems) { return nitems > 0 ? (nitems + kFinTile - 1) / kFinTile : 1; }

rel_status finalize_state(rel_ctx* ctx, int64_t nitems, uint64_t** st) {
  void* p;
  rel_status s = relh::scratch(ctx, SCR_SCAN_STATE, (size_t)finalize_tiles(nitems) * 8, &p);
  *st = (uint64_t*)p;
  return s;
}

__global__ __launch_bounds__(kBlock) void k_index_wipe(JoinIndex x) {
  join_index_wipe(x, blockIdx.x * (int64_t)kBlock + threadIdx.x, (int64_t)gridDim.x * kBlock);
}

// Workgroups of nt threads that empty a join index (beside another kernel's work: one per CU).
unsigned wipe_grid(rel_ctx* ctx, const JoinIndex& x, int nt, int per_cu = 1) {
  const int64_t words = std::max<int64_t>((int64_t)x.hash.mask + 2, x.dense_cap / 4);
  return relh::grid_for(ctx, words, (int64_t)nt * 8, per_cu);
}

// zeroed: the look-back state (finalize_state) and the ticket counter are
// already zero (an earlier kernel of the call cleared them), else they are
// cleared here.
template <class Src>
rel_status finalize(rel_ctx* ctx, const Src& src, int64_t nitems, const OutArgs& o, bool zeroed = false) {
  // (when the kernel runs, its last group of tiles writes the group count)
  if (nitems == 0 && o.n_wg == 0) return relh::fill_u64(ctx, o.d_n, 1, 0);
  rel_status s;
  const int64_t ntiles = finalize_tiles(nitems);
  uint64_t* st;
  if ((s = finalize_state(ctx, nitems, &st)) != REL_OK) return s;
  int64_t* ticket = relh::counters(ctx) + CNT_TICKET;
  if (!zeroed) {
    if ((s = relh::fill_u64(ctx, st, (size_t)ntiles, 0)) != REL_OK) return s;
    if ((s = relh::fill_u64(ctx, ticket, 1, 0)) != REL_OK) return s;
  }
  relh::KernelTimer kt(ctx, "finalize");
  const int64_t ngroups = (ntiles + kFinTilesPerTicket - 1) / kFinTilesPerTicket;
  hipLaunchKernelGGL(k_finalize<Src>, dim3((unsigned)ngroups), dim3(kBlock), 0, ctx->stream, src, nitems, o, (uint64_t*)st,
                     ticket, ngroups);
  REL_LAUNCH_CHECK(ctx, "finalize");
  return REL_OK;
}

// Stages for `grid` workgroups.
rel_status take_stage(rel_ctx* ctx, unsigned grid, uint32_t* touched, Stage* out) {
  const int cap = grid >= 256 ? kStageMax : std::min(kLdsSlots / 2, kStageTotal / (int)grid);
  const size_t slots = (size_t)grid * cap * sizeof(GroupSlot);
  void* p;
  rel_status s = relh::scratch(ctx, SCR_STAGE, slots + (size_t)grid * 4, &p);
  *out = Stage{(GroupSlot*)p, (uint32_t*)((char*)p + slots), cap, touched};
  return s;
}

rel_status init_groups(rel_ctx* ctx, GroupSlot* slots, int64_t nslots) {
  const unsigned grid = relh::grid_for(ctx, nslots, 256 * 4, 4);
  relh::KernelTimer kt(ctx, "group_table_init");
  hipLaunchKernelGGL(k_init_groups, dim3(grid), dim3(256), 0, ctx->stream, slots, nslots);
  REL_LAUNCH_CHECK(ctx, "init_groups");
  return REL_OK;
}

// An empty group table in SCR_GROUP_CLEAN.
rel_status clean_groups(rel_ctx* ctx, int64_t nslots, void** out) {
  return relh::scratch_empty(ctx, SCR_GROUP_CLEAN, (size_t)nslots * sizeof(GroupSlot), out,
                             [&](void* p) { return init_groups(ctx, (GroupSlot*)p, nslots); });
}

bool out_ok(const rel_groups_out* out) {
  return out && out->key && out->sum_price && out->sum_qty && out->count && out->d_n_groups && out->cap >= 0;
}

OutArgs out_args(rel_ctx* ctx, const rel_groups_out* out) {
  return OutArgs{out->key, out->sum_price, out->sum_qty, out->count, out->cap, out->d_n_groups, ctx->d_status,
                 nullptr, 0, nullptr, nullptr, JoinIndex{}, nullptr, nullptr, 0};
}

// Group-table capacity (power of two) for `expected` distinct keys at load `load`.
uint32_t group_log2cap(int64_t expected, double load) {
  if (expected < 1) expected = 1;
  uint32_t l = relh::log2_ceil((uint64_t)((double)expected / load) + 1);
  return l < 4 ? 4 : l;
}

// Fact rows up to which a plain LDS call runs in 256-thread workgroups (60K rows,
// 15 groups: the kernel takes 8.2 us, 12.8 in 15 of 1024 threads). More of them
// would also mean more tables to add to the device table where a workgroup has
// more groups than it may stage (120K rows, 400 groups: the call takes 57 us in
// 118 workgroups of 256 threads, 36 in 30 of 1024; 250K rows: 89 and 42).
constexpr int64_t kSmallRows = 1 << 16;
// Workgroups per CU that update a group table in device memory. Its atomics are the
// bound, and more of them at once collide more; with fewer, rows that match nothing
// wait for their reads. With 3, 4 and as many as registers allow (6), in us: 30M
// rows into 65K groups 2009, 2008, 2045; 6M rows into 700 groups 1229, 1241, 1250;
// 6M rows of sparse keys into 500K groups 548, 548, 555; 6M rows, a quarter of them
// matching, into 100 groups 1014, 998, 1000.
constexpr int kGlobalPerCu = 4;
// The merge kernel ends a plain LDS call of at most so many fact rows and slots
// of the device table: its workgroups write the output from the table when groups
// went there, 8192 slots at a time (60K rows, 131073 slots: 3600 groups 35 us
// with one launch fewer, 49 us with a finalize kernel after it; one workgroup
// going through all of them took 197; 15 groups 18.5 and 21.5 us). Beyond these
// sizes the launch no longer counts.
constexpr int64_t kMergeEndsRows = 1 << 18, kMergeEndsSlots = 1 << 20;

template <int MODE>
rel_status launch_fused(rel_ctx* ctx, int gp, const FusedArgs& a, unsigned grid) {
  relh::KernelTimer kt(ctx, "probe_agg");
  if (gp == G_LDS && a.n <= kSmallRows)
    hipLaunchKernelGGL((k_fused<MODE, G_LDS, kBlock>), dim3(grid), dim3(kBlock), 0, ctx->stream, a);
  else if (gp == G_LDS)
    hipLaunchKernelGGL((k_fused<MODE, G_LDS, kLdsBlock>), dim3(grid), dim3(kLdsBlock), 0, ctx->stream, a);
  else if (gp == G_GLOBAL)
    hipLaunchKernelGGL((k_fused<MODE, G_GLOBAL, kBlock>), dim3(grid), dim3(kBlock), 0, ctx->stream, a);
  else
    hipLaunchKernelGGL((k_fused<MODE, G_ROWAGG, kBlock>), dim3(grid), dim3(kBlock), 0, ctx->stream, a);
  REL_LAUNCH_CHECK(ctx, "fused");
  return REL_OK;
}

#define TRY(x)                      \
  do {                              \
    rel_status s_ = (x);            \
    if (s_ != REL_OK) return s_;    \
  } while (0)

// Fact tables at least this large take the radix-partitioned path unless a
// plan says otherwise ...
constexpr int64_t kPartitionMinRows = 1 << 20;
// ... and, grouping by a dim attribute, at least this many dim rows. Below
// it the plain path's join index (a dense array of 4 B per key when the keys
// are dense, 16 MB at this size) stays in the caches.
constexpr int64_t kPartitionMinDim = 1 << 22;

// A stand-alone group-by of many groups partitions its rows from this many on
// (twice as many when a sample has to say whether there are many groups).
// Measured, partitioned against the device table: 32K rows 37 and 37 us, 64K 39
// and 41, 128K 41 and 51, 1M 65 and 205, 4M 178 and 611; with the sample, 64K
// rows 56 and 47 us, 128K 59 and 62.
constexpr int64_t kGroupbyPartitionRows = 1 << 16;

rel_status sync_stats(rel_ctx* ctx, const rel_fact* fact, const rel_dim* dim, const rel_query* q, const rel_plan* plan,
                      rel_groups_out* out, rel_stats* stats, int64_t* cnt, int64_t join_cap, int64_t group_cap,
                      int join_place, int group_place);

}  // namespace

extern "C" {

rel_status rel_groupby_agg(rel_ctx* ctx, const int64_t* key, const int64_t* price, const int32_t* qty,
                           const int32_t* sel, int64_t n, const rel_table_opts* opts, rel_groups_out* out) {
  if (!ctx || n < 0 || !out_ok(out) || (n > 0 && (!key || !price || !qty)))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_groupby_agg: bad argument");
  if (n >= (1ll << 31)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_groupby_agg: n >= 2^31");
  const double load = (opts && opts->max_load > 0.f) ? (opts->max_load > 0.9f ? 0.9 : opts->max_load) : 0.5;
  const bool hinted = opts && opts->capacity_hint > 0;
  const int64_t expected = hinted ? opts->capacity_hint : (n < (1ll << 30) ? n : (1ll << 30));
  const int placement = opts ? opts->placement : REL_PLACE_AUTO;
  if (placement == REL_PLACE_PARTITIONED) return relh::fail(ctx, REL_UNSUPPORTED, "rel_groupby_agg: partitioned placement");
  const uint32_t l = group_log2cap(expected, load);
  if (l > 31) return relh::fail(ctx, REL_UNSUPPORTED, "rel_groupby_agg: capacity above 2^31");
  if (n == 0) return relh::fill_u64(ctx, out->d_n_groups, 1, 0);
  // Which way: LDS tables over the rows as they come when the caller expects
  // few groups; partitioned for many groups of many rows, the device table for
  // many groups of fewer rows; for an unknown number of groups a sample of the
  // keys decides between few and many on the device.
  const bool few_expected = expected <= kLdsSlots / 2;
  const bool lds = placement == REL_PLACE_LDS || (placement == REL_PLACE_AUTO && (few_expected || !hinted));
  const bool many = placement == REL_PLACE_GLOBAL || (placement == REL_PLACE_AUTO && !few_expected);
  bool partition = placement == REL_PLACE_AUTO && many && n >= (hinted ? kGroupbyPartitionRows : 2 * kGroupbyPartitionRows);
  const int64_t nslots = (1ll << l) + 1;
  void* tbl;  // (left empty by the finalize kernel)
  TRY(clean_groups(ctx, nslots, &tbl));
  const uint32_t probe = hinted ? kPlannedProbe : (uint32_t)(1ull << l);
  const GroupView g{(GroupSlot*)tbl, (uint32_t)((1ull << l) - 1), 32u - l, ctx->d_status, probe};
  const relh::GroupRows in{key, price, qty, sel, n};
  TRY(relh::ensure_counters(ctx));
  int64_t* cnt = relh::counters(ctx);
  uint32_t* flags = (uint32_t*)(cnt + CNT_AUX1);  // [0] touched, [1] done
  uint32_t* few = (uint32_t*)(cnt + CNT_AUX2);
  uint64_t* state;
  TRY(finalize_state(ctx, nslots, &state));
  // (20 B per row: without them the device table, which is slower, serves)
  if (partition) TRY(relh::if_memory(ctx, [&] { return relh::groupby_memory(ctx, n, expected); }, &partition));
  const unsigned grid = relh::grid_for(ctx, n, partition || !many ? kLdsBlock * kGbAhead : kLdsBlock, 1);
  Stage stage{};
  if (lds) TRY(take_stage(ctx, grid, flags, &stage));
  const int mode = !many ? relh::GB_FEW : !lds ? relh::GB_MANY : relh::GB_SAMPLE;
  TRY(relh::groupby_begin(ctx, in, mode, few, (uint64_t*)cnt, CNT_AUX2, state, finalize_tiles(nslots)));
  OutArgs oa = out_args(ctx, out);
  if (lds) {
    relh::KernelTimer kt(ctx, "groupby");
    hipLaunchKernelGGL(k_groupby_lds, dim3(grid), dim3(kLdsBlock), 0, ctx->stream, in, (const uint32_t*)few, g,
                       few_expected || placement == REL_PLACE_LDS ? kLdsProbe : kLdsCacheProbe, !partition, stage);
    MergeArgs mg{stage, (int64_t)grid, nullptr, cnt, g, flags + 1, JoinIndex{}, few, 0, nullptr, nullptr};
    hipLaunchKernelGGL(k_group_merge<false>, dim3(1), dim3(kLdsBlock), 0, ctx->stream, mg, oa);
    oa.done = flags + 1;
    REL_LAUNCH_CHECK(ctx, "groupby");
  } else if (!partition) {
    relh::KernelTimer kt(ctx, "groupby");
    hipLaunchKernelGGL(k_groupby_global, dim3(relh::grid_for(ctx, n, kBlock * 4, 8)), dim3(kBlock), 0, ctx->stream, in, g);
    REL_LAUNCH_CHECK(ctx, "groupby");
  }
  if (partition) {
    const relh::DirectOut direct{out->key, out->sum_price, out->sum_qty, out->count, out->cap, (uint64_t*)(cnt + CNT_GROUPS), flags};
    TRY(relh::groupby_partitioned(ctx, in, expected, few, g, direct));
    oa.base = direct.n_direct;
    oa.touched = flags;
    oa.limit = hinted ? nslots : INT64_MAX;
  }
  TRY(finalize(ctx, SlotSource{(GroupSlot*)tbl, nslots - 1, true}, nslots, oa, true));
  relh::scratch_emptied(ctx, SCR_GROUP_CLEAN);
  return REL_OK;
}

rel_status rel_filter_join_agg(rel_ctx* ctx, const rel_fact* fact, const rel_dim* dim, const rel_query* q,
                               const rel_plan* plan, rel_groups_out* out, rel_stats* stats) {
  if (!ctx || !fact || !dim || !q || !out_ok(out)) return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_join_agg: null argument");
  const int64_t n = fact->n, m = dim->m;
  const int gb = q->group_by;
  if (n < 0 || m < 0 || gb < REL_GROUP_PRIO_FLAG || gb > REL_GROUP_DIM_GRP)
    return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_join_agg: bad size or group_by");
  if (n > 0 && (!fact->fk || !fact->price_cents || !fact->qty || !fact->day || (gb == REL_GROUP_PRIO_FLAG && !fact->flag)))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_join_agg: missing fact column");
  if (m > 0 && (!dim->pk || (gb == REL_GROUP_PRIO_FLAG && !dim->prio) || (gb == REL_GROUP_DIM_GRP && !dim->grp)))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_join_agg: missing dim column");
  const void* cols[] = {fact->fk, fact->price_cents, fact->qty, fact->day, fact->flag, dim->pk, dim->prio, dim->grp};
  for (const void* c : cols)
    if (c && !relh::aligned16(c)) return relh::fail(ctx, REL_INVALID_ARG, "rel_filter_join_agg: column not 16-byte aligned");
  if (n >= (1ll << 31) || m >= (1ll << 30)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_filter_join_agg: table too large");
  TRY(relh::ensure_counters(ctx));
  int64_t* cnt = relh::counters(ctx);
  const bool planned = plan && plan->group_capacity > 0;
  // A call that synchronises reports through its own status word, cleared
  // here; the others leave their bits in the sticky word for rel_ctx_sync.
  struct StatusScope {
    rel_ctx* c;
    uint32_t* saved;
    ~StatusScope() { c->d_status = saved; }
  } scope{ctx, ctx->d_status};
  if (stats != nullptr || (planned && plan->allow_fallback)) {
    ctx->d_status = ctx->d_status_words + 1;
    if (ctx->sync_word_dirty) TRY(relh::fill_u32(ctx, ctx->d_status, 1, 0));
    ctx->sync_word_dirty = true;  // until k_report of this call has cleared it again
  } else {
    ctx->d_status = ctx->d_status_words;  // also inside a synchronising call's fallback run
  }

  // Radix partitioning of both sides: asked for, or chosen for large inputs
  // (for a dim-attribute group key only when the dim side is large enough that
  // its join table would not stay in L2).
  const int jp = plan ? plan->join_placement : REL_PLACE_AUTO;
  const bool part = jp == REL_PLACE_PARTITIONED ||
                    (jp == REL_PLACE_AUTO && n >= kPartitionMinRows && (gb == REL_GROUP_FK || m >= kPartitionMinDim));
  if (part && gb == REL_GROUP_FK) {
    // with fact rows, the partitioning's first kernel clears the two counters
    if (n == 0) TRY(relh::fill_u64(ctx, cnt, 2, 0));
    TRY(relh::partitioned_groupjoin(ctx, fact, dim, q->day_lt, out, cnt));
    return sync_stats(ctx, fact, dim, q, plan, out, stats, cnt, m, m, REL_PLACE_PARTITIONED, REL_PLACE_PARTITIONED);
  }

  FusedArgs a{};
  a.fk = fact->fk;
  a.price = fact->price_cents;
  a.qty = fact->qty;
  a.day = fact->day;
  a.flag = fact->flag;
  a.n = n;
  a.day_lt = q->day_lt;

  int gp;
  int64_t group_cap = 0;
  uint32_t gl = 0;
  void* gt = nullptr;
  bool eager = false, by_partials = false, clean_table = false;
  relh::Partials partials{};
  int64_t partials_expected = 0;
  if (gb == REL_GROUP_FK) {
    gp = G_ROWAGG;  // group key == join key: per-dim-row accumulators
    group_cap = m;
    const size_t bytes = (size_t)(m > 0 ? m : 1) * sizeof(RowAgg);
    TRY(relh::scratch_empty(ctx, SCR_ROW_AGG, bytes, &gt, [&](void* p) {
      relh::KernelTimer kt(ctx, "group_table_init");
      return relh::fill_u64(ctx, p, bytes / 8, 0);
    }));
    a.row_agg = (RowAgg*)gt;
  } else {
    const int64_t ub = gb == REL_GROUP_PRIO_FLAG ? (n < 65536 ? n : 65536) : (n < m ? n : m);
    const int64_t expected = planned ? plan->group_capacity : ub;
    int placement = plan ? plan->group_placement : REL_PLACE_AUTO;
    if (placement == REL_PLACE_PARTITIONED) return relh::fail(ctx, REL_UNSUPPORTED, "rel_filter_join_agg: partitioned group-by");
    if (placement == REL_PLACE_AUTO) placement = (gb == REL_GROUP_PRIO_FLAG || expected <= kLdsSlots / 2) ? REL_PLACE_LDS : REL_PLACE_GLOBAL;
    gp = placement == REL_PLACE_LDS ? G_LDS : G_GLOBAL;
    // With more groups than the LDS table holds, LDS acts as a cache in front of
    // the device-memory table (it keeps the keys each workgroup meets first,
    // which under skew are the hot ones); a short probe budget bounds the cost
    // of rows whose key is not cached.
    a.lds_probe = expected <= relh::kLdsGroupCap ? kLdsProbe : kLdsCacheProbe;
    gl = group_log2cap(expected, 0.5);
    if (gl > 31) return relh::fail(ctx, REL_UNSUPPORTED, "rel_filter_join_agg: group table above 2^31 slots");
    group_cap = 1ll << gl;
    eager = part && gb == REL_GROUP_DIM_GRP && (gp != G_LDS || a.lds_probe != kLdsProbe);
    // The partial sums of a planned call are partitioned by group and summed in
    // LDS; the device table takes three atomics for each. Measured, device table
    // against partitioned partials, uniform keys, half of the rows selected: 250K
    // rows 142 and 123 us, 4M 261 and 188, 16M 738 and 403, 60M with 1000 groups
    // 5080 and 1357, with 15M groups 3462 and 2134 (1% of the rows selected: 138
    // and 144, 262 and 255, 718 and 644, 1296 and 666). A call without a plan
    // would gain as much (60M rows, 1M groups: 1.86 ms to 1.19), but keeps the
    // table: a planned run pays 0.15 ms for its sketch and its read by the host
    // (1.34 ms), and is held to be no slower than the plain one. Without memory
    // for the partials the table serves, too.
    clean_table = !part || (eager && planned);
    if (clean_table) {
      TRY(clean_groups(ctx, group_cap + 1, &gt));  // emptied again by the kernel that reads it
    } else {
      TRY(relh::scratch(ctx, SCR_GROUP_TABLE, (size_t)(group_cap + 1) * sizeof(GroupSlot), &gt));
      TRY(init_groups(ctx, (GroupSlot*)gt, group_cap + 1));
    }
    if (eager && planned) {
      // (last, after the memory that the call cannot do without)
      uint64_t* state;
      TRY(finalize_state(ctx, group_cap + 1, &state));
      TRY(relh::partitioned_memory(ctx, n, m));
      int64_t rows;
      unsigned wgs;
      size_t bytes;
      relh::partials_bounds(ctx, n, m, &rows, &wgs, &bytes);
      TRY(relh::if_memory(ctx, [&] {
        return relh::partials_take(ctx, rows, wgs, expected, bytes, (uint32_t*)(cnt + CNT_AUX2), &partials);
      }, &by_partials));
      partials_expected = expected;
    }
    a.groups = GroupView{(GroupSlot*)gt, (uint32_t)(group_cap - 1), 32u - gl, ctx->d_status,
                         planned ? kPlannedProbe : (uint32_t)group_cap};
  }

  if (part) {
    // the same group table behind a per-workgroup LDS table (probe budget 0:
    // none); grouping by dim.grp with more groups than LDS holds aggregates per
    // dim key first
    TRY(relh::fill_u64(ctx, cnt, CNT_AUX2 + 1, 0));
    TRY(relh::partitioned_join_agg(ctx, fact, dim, q->day_lt, gb, gt, gl, a.groups.max_probe,
                                   gp == G_LDS ? a.lds_probe : 0, eager, by_partials ? &partials : nullptr, cnt));
    OutArgs oa = out_args(ctx, out);
    if (by_partials) {
      uint32_t* flags = (uint32_t*)(cnt + CNT_AUX1);  // [0] touched, [1] stays 0
      const relh::DirectOut direct{out->key, out->sum_price, out->sum_qty, out->count, out->cap, (uint64_t*)(cnt + CNT_GROUPS), flags};
      TRY(relh::partials_reduce(ctx, partials, partials_expected, flags + 1, a.groups, direct));
      oa.base = direct.n_direct;
      oa.touched = flags;
      oa.limit = planned ? group_cap + 1 : INT64_MAX;
    }
    TRY(finalize(ctx, SlotSource{(GroupSlot*)gt, group_cap, clean_table}, group_cap + 1, oa));
    if (clean_table) relh::scratch_emptied(ctx, SCR_GROUP_CLEAN);
    return sync_stats(ctx, fact, dim, q, plan, out, stats, cnt, m, group_cap, REL_PLACE_PARTITIONED,
                      gp == G_LDS ? REL_PLACE_LDS : REL_PLACE_GLOBAL);
  }

  // Join index: a dense array when the dim keys span at most 2m values, else
  // a hash table of plain sizing (2m rounded up to a power of two); both in
  // device memory, the choice made on the device. Its first kernel also
  // zeroes the counter words (rows passed, join matches, the finalize ticket,
  // the merge kernel's two flags) and the finalize kernel's look-back state.
  const int64_t fin_items = gp == G_ROWAGG ? m : group_cap + 1;
  uint64_t* fin_state;
  TRY(finalize_state(ctx, fin_items, &fin_state));
  const relh::ZeroSpans zero{{(uint64_t*)cnt, fin_state}, {CNT_AUX2, finalize_tiles(fin_items)}};
  const uint32_t jl = relh::join_log2cap(m, nullptr);
  const void* payload = gb == REL_GROUP_PRIO_FLAG ? (const void*)dim->prio : gb == REL_GROUP_DIM_GRP ? (const void*)dim->grp : nullptr;
  const int pkind = gb == REL_GROUP_PRIO_FLAG ? relh::PAY_I8 : gb == REL_GROUP_DIM_GRP ? relh::PAY_I32 : relh::PAY_ROW_ID;
  const bool merge_ends = gp == G_LDS && n > 0 && n <= kMergeEndsRows && group_cap <= kMergeEndsSlots;
  const unsigned grid = gp == G_ROWAGG   ? relh::grid_for(ctx, n, kBlock * kIPT, 8)
                        : gp == G_GLOBAL ? relh::grid_for(ctx, n, kBlock * kIPT, kGlobalPerCu)
                        : n <= kSmallRows ? relh::grid_for(ctx, n, kBlock * kIPT, 1)
                                          : relh::grid_for(ctx, n, kLdsBlock * kIPT, 1);
  uint32_t* flags = (uint32_t*)(cnt + CNT_AUX1);  // [0] touched, [1] done
  // (all memory of the call is taken before the first kernel that fills a table)
  void* wc;
  TRY(relh::scratch(ctx, SCR_WG_COUNTS, (size_t)grid * 24, &wc));
  if (gp == G_LDS) TRY(take_stage(ctx, grid, flags, &a.stage));
  JoinIndex jx{};
  TRY(relh::join_index_build(ctx, dim->pk, payload, pkind, m, n, (uint32_t*)(cnt + CNT_AUX2), zero, &jx));
  a.join = jx;

  OutArgs oa = out_args(ctx, out);
  if (n > 0) {
    a.wg_counts = (uint64_t*)wc;
    oa.wg_counts = a.wg_counts;
    oa.n_wg = grid;
    oa.counters = cnt;
    oa.join = jx;
    if (gb == REL_GROUP_PRIO_FLAG) TRY(launch_fused<M_PRIO_FLAG>(ctx, gp, a, grid));
    else if (gb == REL_GROUP_FK) TRY(launch_fused<M_FK>(ctx, gp, a, grid));
    else TRY(launch_fused<M_DIM_GRP>(ctx, gp, a, grid));
    if (gp == G_LDS) {
      const int64_t nslots = merge_ends ? group_cap + 1 : 0;
      MergeArgs mg{a.stage, (int64_t)grid, a.wg_counts, cnt, a.groups, flags + 1, jx, nullptr, nslots,
                   (uint32_t*)(cnt + CNT_TICKET), (uint32_t*)(cnt + CNT_AUX0)};
      const unsigned others = std::max(wipe_grid(ctx, jx, kLdsBlock), relh::grid_for(ctx, nslots, kLdsBlock * 8, 1));
      oa.n_wg = 0;  // the merge kernel sums the counts
      oa.done = flags + 1;
      relh::KernelTimer kt(ctx, "group_merge");
      if (merge_ends) hipLaunchKernelGGL(k_group_merge<true>, dim3(1 + others), dim3(kLdsBlock), 0, ctx->stream, mg, oa);
      else hipLaunchKernelGGL(k_group_merge<false>, dim3(1 + others), dim3(kLdsBlock), 0, ctx->stream, mg, oa);
      REL_LAUNCH_CHECK(ctx, "group_merge");
    }
  } else {
    TRY(relh::join_index_verify(ctx, jx));  // (no probing kernel runs)
  }

  // Without a merge kernel, whose other workgroups do it, a kernel of its own
  // empties the index: beside the finalize kernel's workgroups the stores hold up
  // its look-back (375K rows, 277K sparse dim keys, 221K groups: 109 us, 99 so).
  const bool wipe = gp != G_LDS || n == 0;
  if (gp == G_ROWAGG) {
    TRY(finalize(ctx, RowAggSource{(RowAgg*)gt, dim->pk}, m, oa, true));
    relh::scratch_emptied(ctx, SCR_ROW_AGG);
  } else {
    if (!merge_ends)
      TRY(finalize(ctx, SlotSource{(GroupSlot*)gt, group_cap, true}, group_cap + 1, oa, true));
    relh::scratch_emptied(ctx, SCR_GROUP_CLEAN);
  }
  if (wipe) {
    hipLaunchKernelGGL(k_index_wipe, dim3(wipe_grid(ctx, jx, kBlock, 8)), dim3(kBlock), 0, ctx->stream, jx);
    REL_LAUNCH_CHECK(ctx, "index_wipe");
  }
  relh::join_index_wiped(ctx, jx);
  return sync_stats(ctx, fact, dim, q, plan, out, stats, cnt, (int64_t)1 << jl, group_cap, REL_PLACE_GLOBAL,
                    gp == G_LDS ? REL_PLACE_LDS : REL_PLACE_GLOBAL);
}

}  // extern "C"

namespace {

__global__ void k_report(const int64_t* cnt, const int64_t* n_groups, uint32_t* status, int64_t* report) {
  report[0] = cnt[0];
  report[1] = cnt[1];
  report[2] = *n_groups;
  report[3] = (int64_t)*status;
  *status = 0;
}

// Common tail of the fused pipeline: when the caller wants statistics or a
// planned table may need the fallback, synchronise, read the counters and the
// status word, and rerun with plain sizing if a planned table overflowed.
rel_status sync_stats(rel_ctx* ctx, const rel_fact* fact, const rel_dim* dim, const rel_query* q, const rel_plan* plan,
                      rel_groups_out* out, rel_stats* stats, int64_t* cnt, int64_t join_cap, int64_t group_cap,
                      int join_place, int group_place) {
  const int64_t n = fact->n;
  const bool planned = plan && plan->group_capacity > 0;
  const bool want_sync = stats != nullptr || (planned && plan->allow_fallback);
  if (!want_sync) return REL_OK;
  // One kernel writes all that the host needs to pinned memory, and clears this
  // call's status word for the next one: three copies back cost a round trip each.
  hipLaunchKernelGGL(k_report, dim3(1), dim3(1), 0, ctx->stream, (const int64_t*)cnt, (const int64_t*)out->d_n_groups,
                     ctx->d_status, ctx->report);
  REL_LAUNCH_CHECK(ctx, "report");
  REL_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
  ctx->sync_word_dirty = false;
  const volatile int64_t* rep = ctx->report;
  const int64_t hc[2] = {rep[0], rep[1]}, ng = rep[2];
  const uint32_t bits = (uint32_t)rep[3];
  if (bits & kDevDupKey) return relh::fail(ctx, REL_DUPLICATE_KEY, "rel_filter_join_agg: duplicate pk");
  const bool overflow = (bits & kDevOverflow) != 0;
  if (overflow && ng > out->cap) return relh::fail(ctx, REL_CAPACITY, "rel_filter_join_agg: %lld groups > cap", (long long)ng);
  if (overflow && planned) {
    if (!plan->allow_fallback) return relh::fail(ctx, REL_OVERFLOW, "rel_filter_join_agg: planned table overflowed");
    rel_status s = rel_filter_join_agg(ctx, fact, dim, q, nullptr, out, stats);
    if (s == REL_OK && stats) {
      stats->overflowed = 1;
      stats->fell_back = 1;
    }
    return s;
  }
  if (overflow) return relh::fail(ctx, REL_OVERFLOW, "rel_filter_join_agg: table overflow");
  if (stats) {
    stats->rows_in = n;
    stats->rows_passed = hc[0];
    stats->join_matches = hc[1];
    stats->groups = ng;
    stats->join_capacity = join_cap;
    stats->group_capacity = group_cap;
    stats->join_placement = join_place;
    stats->group_placement = group_place;
    stats->overflowed = 0;
    stats->fell_back = 0;
  }
  return REL_OK;
}

}  // namespace
