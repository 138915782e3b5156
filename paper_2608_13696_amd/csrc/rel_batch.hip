// Batched execution of many independent fused queries.
//
// A small query alone cannot fill 256 CUs (the paper's undersaturation
// finding, Section 6.1); thousands of them issued one by one pay a launch and
// a dependency gap per kernel. Here one persistent kernel takes whole instances,
// a workgroup each (k_batch_whole), and the instances that are too large for one
// workgroup, or too sparse for its arrays, become work items of three more
// kernels that share tables in device memory: build, probe/aggregate, finalize
// (one per phase and size bucket). Workgroups pull instances, costliest first, and
// items, largest first, from ticket counters, and the whole sequence is captured once
// into a HIP graph so that a run is one graph launch.
//
// Per-bucket configuration of the shared tables (rows per thread, workgroup size, LDS or
// device-memory group table, LDS or device-memory join table, rows per work
// item) comes from a tuning table that the autotuner measures.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "rel_device.h"
#include "rel_host.h"
#include "rel_ops.h"

namespace {

using namespace rel;

constexpr int kBLdsSlots = 1024;
constexpr int kBLdsProbe = 32;
// Instances with more groups than the LDS table holds still use it as a
// cache in front of their device-memory table: the first keys a workgroup
// meets stay in LDS (one set of device atomics per key and work item instead
// of one per row), and a short probe budget bounds the cost for the others.
constexpr int kBLdsCacheProbe = 4;
constexpr int64_t kFinItemSlots = 8192;
// LDS join table: 2048 packed slots (and the side slot of key -1, as in the
// device-memory table), for instances of at most 1024 dim keys (load <= 0.5).
constexpr int kBLdsJoinBits = 11;
constexpr int kBLdsJoinSlots = 1 << kBLdsJoinBits;
constexpr uint32_t kHintProbe = 256;

// Device view of one instance (all pointers device memory).
struct BInst {
  const int32_t* fk;
  const int64_t* price;
  const int32_t* qty;
  const int32_t* day;
  const int8_t* flag;
  const int32_t* pk;
  const int8_t* prio;
  const int32_t* grp;
  int64_t n, m;
  int32_t day_lt, group_by;
  uint64_t* jslots;
  uint32_t jmask, jshift;
  GroupSlot* gslots;
  uint32_t gmask, gshift, gprobe;
  int32_t lds;    // aggregate through the workgroup's LDS table first
  int32_t ljoin;  // probe a join table built in the workgroup's LDS for each work item
  int64_t* out_key;
  int64_t* out_sp;
  int64_t* out_sq;
  int64_t* out_cnt;
  int64_t out_cap;
  int64_t* d_n;
  int64_t* stats;  // [rows passed, join matches, groups]
};

struct BItem {
  int32_t inst;
  int32_t pad;
  int64_t lo, hi;
};

// How much of a list the kernels of the shared-table path work through: its
// first `n` entries belong to instances that only they take, the others, up to
// `all`, to instances that one workgroup may take whole. Those count only when
// some of them were left, and are then skipped where they are done.
struct BList {
  int64_t n, all;
  const uint32_t* left;
  const uint32_t* done;
  __device__ __forceinline__ int64_t size() const { return n < all && *left != 0 ? all : n; }
};

// The join payload of dim row j (the group attribute, or the row id for GROUP BY fk).
__device__ __forceinline__ int32_t batch_payload(const BInst& I, int64_t j) {
  return I.group_by == REL_GROUP_PRIO_FLAG ? (int32_t)I.prio[j] : I.group_by == REL_GROUP_DIM_GRP ? I.grp[j] : (int32_t)j;
}

// First kernel of a run: the run's words and the instances' output counts.
__global__ void k_batch_reset(uint64_t* __restrict__ words, int64_t n_words, const BInst* __restrict__ inst, int32_t k) {
  const int64_t id = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = id; i < n_words; i += stride) words[i] = 0;
  for (int64_t i = id; i < k; i += stride) *inst[i].d_n = 0;
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_batch_build(const BInst* __restrict__ inst, const BItem* __restrict__ items,
                                                       int64_t* __restrict__ ticket,
                                                       uint32_t* __restrict__ status, BList list) {
  __shared__ int64_t s_item;
  const int64_t n_items = list.size();
  if (n_items == 0) return;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)ticket, 1ull);
    __syncthreads();
    const int64_t it = s_item;
    __syncthreads();
    if (it >= n_items) break;
    const BItem w = items[it];
    if (it >= list.n && list.done[w.inst] != 0) continue;
    const BInst& I = inst[w.inst];
    for (int64_t j = w.lo + threadIdx.x; j < w.hi; j += BLOCK) {
      join_insert(I.jslots, I.jmask, I.jshift, I.pk[j], batch_payload(I, j), status);
    }
  }
}

__device__ __forceinline__ int64_t batch_key(const BInst& I, int32_t pl, int32_t fk, int8_t flag) {
  if (I.group_by == REL_GROUP_PRIO_FLAG) return (int64_t)pl * 256 + (int64_t)(uint8_t)flag;
  if (I.group_by == REL_GROUP_DIM_GRP) return (int64_t)pl;
  return (int64_t)fk;
}

// An instance's join table in LDS, in the packed format of the device-memory
// table (key in the low word, payload in the high word, key -1 in the side
// slot). The workgroup builds it from the dim columns at the start of each
// work item of a small-dim instance, so the probes of the item's rows are LDS
// reads instead of device-memory reads. A repeated key is reported by the
// instance's device-memory build, which every instance still runs.
struct LdsJoin {
  uint64_t slot[kBLdsJoinSlots + 1];

  __device__ void init(int tid, int nthreads) {
    for (int s = tid; s <= kBLdsJoinSlots; s += nthreads) slot[s] = kJoinEmpty;
  }
  // At most kBLdsJoinSlots / 2 keys, so a free slot always exists.
  __device__ void insert(int32_t key, int32_t pl) {
    if (key == -1) {
      atomicCAS((unsigned long long*)&slot[kBLdsJoinSlots], (unsigned long long)kJoinEmpty, (unsigned long long)(uint32_t)pl);
      return;
    }
    const uint64_t want = (uint64_t)(uint32_t)key | ((uint64_t)(uint32_t)pl << 32);
    uint32_t h = hash32(key, 32 - kBLdsJoinBits);
    for (int step = 0; step < kBLdsJoinSlots; ++step) {
      const uint64_t old = atomicCAS((unsigned long long*)&slot[h], (unsigned long long)kJoinEmpty, (unsigned long long)want);
      if (old == kJoinEmpty || (uint32_t)old == (uint32_t)key) return;
      h = (h + 1) & (kBLdsJoinSlots - 1);
    }
  }
  __device__ __forceinline__ bool lookup(int32_t key, int32_t* pl) const {
    if (key == -1) {
      const uint64_t s = slot[kBLdsJoinSlots];
      *pl = (int32_t)(uint32_t)s;
      return s != kJoinEmpty;
    }
    uint32_t h = hash32(key, 32 - kBLdsJoinBits);
    for (int step = 0; step < kBLdsJoinSlots; ++step) {
      const uint64_t s = slot[h];
      if (s == kJoinEmpty) return false;
      if ((uint32_t)s == (uint32_t)key) {
        *pl = (int32_t)(s >> 32);
        return true;
      }
      h = (h + 1) & (kBLdsJoinSlots - 1);
    }
    return false;
  }
};

// LJ: the instance of the kernel that carries the LDS join table (16 KB more
// LDS per workgroup); only buckets whose tuning enables it launch it.
template <bool LJ>
struct LdsJoinStore {
  LdsJoin t;
};
template <>
struct LdsJoinStore<false> {};

template <int BLOCK, int IPT, bool LJ>
__global__ __launch_bounds__(BLOCK) void k_batch_probe(const BInst* __restrict__ inst, const BItem* __restrict__ items,
                                                       int64_t* __restrict__ ticket,
                                                       uint32_t* __restrict__ status, BList list) {
  __shared__ LdsGroups<kBLdsSlots> lds;
  __shared__ LdsJoinStore<LJ> ljs;
  __shared__ int64_t s_item;
  const int64_t n_items = list.size();
  if (n_items == 0) return;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)ticket, 1ull);
    __syncthreads();
    const int64_t it = s_item;
    if (it >= n_items) break;
    const BItem w = items[it];
    if (it >= list.n && list.done[w.inst] != 0) {
      __syncthreads();  // (every thread has read s_item)
      continue;
    }
    const BInst& I = inst[w.inst];
    const int lds_probe = I.lds != 0 ? kBLdsProbe : kBLdsCacheProbe;
    const JoinView jv{I.jslots, I.jmask, I.jshift};
    const GroupView gv{I.gslots, I.gmask, I.gshift, status, I.gprobe};
    bool lj = false;  // uniform over the workgroup (one item)
    if constexpr (LJ) {
      lj = I.ljoin != 0;
      if (lj) {
        ljs.t.init(threadIdx.x, BLOCK);
        __syncthreads();
        for (int64_t j = threadIdx.x; j < I.m; j += BLOCK) ljs.t.insert(I.pk[j], batch_payload(I, j));
      }
    }
    lds.init(threadIdx.x, BLOCK);
    __syncthreads();
    uint64_t passed = 0, matched = 0;
    for (int64_t r0 = w.lo + threadIdx.x; r0 < w.hi; r0 += (int64_t)BLOCK * IPT) {
      int32_t d[IPT], f[IPT], q[IPT];
      int64_t p[IPT];
      int8_t fl[IPT];
#pragma unroll
      for (int k = 0; k < IPT; ++k) {  // all loads first; strided rows keep each load coalesced
        const int64_t r = r0 + (int64_t)k * BLOCK;
        const bool ok = r < w.hi;
        d[k] = ok ? I.day[r] : 0;
        f[k] = ok ? I.fk[r] : 0;
        q[k] = ok ? I.qty[r] : 0;
        p[k] = ok ? I.price[r] : 0;
        fl[k] = (ok && I.group_by == REL_GROUP_PRIO_FLAG) ? I.flag[r] : 0;
      }
#pragma unroll
      for (int k = 0; k < IPT; ++k) {
        if (r0 + (int64_t)k * BLOCK >= w.hi || !(d[k] < I.day_lt)) continue;
        ++passed;
        int32_t pl;
        bool hit;
        if constexpr (LJ) hit = lj ? ljs.t.lookup(f[k], &pl) : join_lookup(jv, f[k], &pl);
        else hit = join_lookup(jv, f[k], &pl);
        if (!hit) continue;
        ++matched;
        const int64_t key = batch_key(I, pl, f[k], fl[k]);
        const uint64_t sp = (uint64_t)p[k], sq = (uint64_t)(int64_t)q[k];
        const int s = key != kGroupEmpty ? lds.find(key, lds_probe) : -1;
        if (s >= 0) lds.add(s, sp, sq, 1ull);
        else group_add(gv, key, sp, sq, 1ull);
      }
    }
    __syncthreads();
    lds.flush(gv, threadIdx.x, BLOCK);
    passed = wave_sum(passed);
    matched = wave_sum(matched);
    if (lane_id() == 0) {
      if (passed) dev_add<unsigned long long>((unsigned long long*)&I.stats[0], passed);
      if (matched) dev_add<unsigned long long>((unsigned long long*)&I.stats[1], matched);
    }
    __syncthreads();
  }
}

// Emit the occupied group slots of each instance: one atomic per wave on the
// instance's own output counter (instances are small, so it is not contended).
__global__ __launch_bounds__(256) void k_batch_finalize(const BInst* __restrict__ inst, const BItem* __restrict__ items,
                                                        int64_t* __restrict__ ticket,
                                                        uint32_t* __restrict__ status, BList list) {
  __shared__ int64_t s_item;
  const int64_t n_items = list.size();
  if (n_items == 0) return;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)ticket, 1ull);
    __syncthreads();
    const int64_t it = s_item;
    __syncthreads();
    if (it >= n_items) break;
    const BItem w = items[it];
    if (it >= list.n && list.done[w.inst] != 0) continue;
    const BInst& I = inst[w.inst];
    const int64_t side = (int64_t)I.gmask + 1;
    // wave-uniform trip count, so ballots see every lane
    for (int64_t base = w.lo + (threadIdx.x / kWave) * kWave; base < w.hi; base += 256) {
      const int64_t s = base + lane_id();
      bool occ = false;
      GroupSlot g{};
      if (s < w.hi) {
        g = I.gslots[s];
        occ = g.count != 0;
        if (s == side) g.key = kGroupEmpty;
      }
      const uint64_t b = wave_ballot(occ);
      if (b == 0) continue;
      int64_t pos = 0;
      if (lane_id() == 0) {
        pos = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)I.d_n, (unsigned long long)__popcll(b));
        dev_add<unsigned long long>((unsigned long long*)&I.stats[2], (unsigned long long)__popcll(b));
      }
      pos = __shfl(pos, 0, kWave) + mask_rank(b);
      if (!occ) continue;
      if (pos < I.out_cap) {
        I.out_key[pos] = g.key;
        I.out_sp[pos] = (int64_t)g.sum_price;
        I.out_sq[pos] = (int64_t)g.sum_qty;
        I.out_cnt[pos] = (int64_t)g.count;
      } else {
        set_status(status, kDevOverflow);
      }
    }
  }
}

__global__ void k_batch_init_groups(GroupSlot* __restrict__ slots, BList list) {
  const int64_t nslots = list.size();
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

__global__ void k_batch_fill(uint64_t* __restrict__ p, uint64_t v, BList list) {
  const int64_t n = list.size();
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// ---- whole instances -------------------------------------------------------------------------------------------------
//
// The kernels above pay for device memory: a compare-and-swap per dim row and
// up to four atomics per joined row, at about 27 G/s for the whole chip. When
// there are enough instances to keep every CU busy, one workgroup takes a whole
// instance instead and nothing is shared with another workgroup: no atomics on
// device memory, no group table, no merge.
//
//   1. the dim keys' and group attributes' minima and maxima;
//   2. the join table, an array over the keys' range of as few bits per entry as
//      hold 0 or the dim row's group attribute relative to the smallest, plus 1
//      (1, 2, 4, 8 or 16), filled in LDS slice by slice and streamed to memory, or
//      left in LDS when it fits beside the groups;
//   3. the fact rows: filter, lookup, and adds into LDS arrays of sums indexed
//      by the group's number;
//   4. the groups that have rows, written out in order.
//
// With more groups than the LDS arrays hold, step 3 sorts each tile's joined
// rows by chunk of groups into memory of the workgroup's own, and the chunks are
// then summed one after another. Where few dim rows have attributes of a wide
// range, the attributes that occur are numbered first, so that one chunk holds
// them. Instances whose keys or attributes are too sparse for arrays are left to
// the kernels above (`BWhole::left`).
//
// 4096 instances of 1K to 1M rows (585M rows, 12.9 GB of columns): 19.99 ms by
// the shared tables, 4.09 ms here. What bounds it is the fabric: of the large
// instances, most lookups miss the XCD's L2 and fetch a 128-byte line, as many
// bytes again as the columns. With 16-bit entries throughout it was 5.97 ms
// (31 GB fetched; 22 GB with entries of as few bits as will do), without the
// next tile's loads in flight 6.65, with two workgroups of 512 threads per CU
// 9.90 ms (half the LDS each: twice the chunks). The steps hand their values on
// in LDS (`WPlan`): in registers over the whole instance they spilled inside the
// loop over the rows (11.5 ms). A one-tile instance takes about 10 us.
constexpr int kWBlock = 1024;
constexpr int kWRows = 4;                                  // rows per thread and tile
constexpr int kWTile = kWBlock * kWRows;
constexpr int kWPool = 152 * 1024;                         // bytes of LDS for tables, sums and sorted tiles
constexpr int kWGroupBytes = 20;                           // price and quantity sums, count
constexpr int kWCap = 7168;                                // groups of one chunk
constexpr int kWMaxChunks = 128;
constexpr int kWSortBytes = kWTile * 16;                   // a sorted tile
constexpr int kWRankRows = 5120;                           // at most so many dim rows have their attributes numbered
constexpr int kWRankBytes = 65536 / 8 + 65536 / 16 + kWRankRows * 2;
constexpr int64_t kWMaxRange = (int64_t)kWCap * kWMaxChunks;  // group numbers
constexpr size_t kWMaxSpill = 8ull << 30;                  // bytes of spill memory of a batch
static_assert(kWCap * kWGroupBytes <= kWPool && kWSortBytes + 64 * 1024 <= kWPool, "LDS pool");
static_assert(kWRankRows <= kWCap && kWRankRows * (kWGroupBytes + 4) + 64 + kWRankBytes <= kWPool, "LDS pool");

struct BWhole {
  const BInst* inst;
  const int32_t* order;   // instances to take, costliest first
  int32_t n;              // their number
  int64_t* ticket;
  uint32_t* status;
  uint32_t* done;         // per instance: finished here
  uint32_t* left;         // instances of `order` that were not
  uint64_t* spill;        // per workgroup: spill_rows words of {group, quantity}, then as many prices
  uint32_t* spill_off;    // per workgroup: [tiles][kWMaxChunks + 1]
  int64_t spill_rows;     // 0: no instance may need more than one chunk
};

__device__ __forceinline__ int32_t w_attr(const BInst& I, int64_t j) {
  return I.group_by == REL_GROUP_PRIO_FLAG ? (int32_t)I.prio[j] : I.group_by == REL_GROUP_DIM_GRP ? I.grp[j] : 0;
}

// Entries of 2^lb bits, packed in words (one lookup is one word read).
struct WBits {
  uint32_t lb;
  static __device__ __forceinline__ WBits of(int64_t most) { return WBits{most <= 1 ? 0u : most <= 3 ? 1u : most <= 15 ? 2u : most <= 255 ? 3u : 4u}; }
  __device__ __forceinline__ uint32_t word(uint32_t off) const { return off >> (5 - lb); }
  __device__ __forceinline__ uint32_t shift(uint32_t off) const { return (off & ((32u >> lb) - 1u)) << lb; }
  __device__ __forceinline__ uint32_t get(uint32_t w, uint32_t off) const { return (w >> shift(off)) & ((1u << (1u << lb)) - 1u); }
  __device__ __forceinline__ uint32_t words(uint64_t entries) const { return (uint32_t)((entries + (32 >> lb) - 1) >> (5 - lb)); }
  __device__ __forceinline__ uint32_t used(uint32_t w) const {  // entries of a word that are not 0
    for (uint32_t d = (1u << lb) >> 1; d != 0; d >>= 1) w |= w >> d;
    const uint32_t low = lb == 0 ? ~0u : lb == 1 ? 0x55555555u : lb == 2 ? 0x11111111u : lb == 3 ? 0x01010101u : 0x00010001u;
    return (uint32_t)__popc(w & low);
  }
};

// Adds one joined row to the sums of group number g.
struct WSums {
  uint64_t* price;
  uint64_t* qty;
  uint32_t* count;
  __device__ __forceinline__ void add(uint32_t g, int64_t p, int32_t q) const {
    atomicAdd((unsigned long long*)&price[g], (unsigned long long)p);
    atomicAdd((unsigned long long*)&qty[g], (unsigned long long)(int64_t)q);
    atomicAdd(&count[g], 1u);
  }
  __device__ __forceinline__ void clear(uint32_t groups) const {
    for (uint32_t g = threadIdx.x; g < groups; g += kWBlock) {
      price[g] = 0;
      qty[g] = 0;
      count[g] = 0;
    }
  }
};

// Groups with rows among the sums' first `groups` to the output from row *out
// on: key0 + the group's number (or, where it is given, key0 + attr[number]).
// Every thread calls it; each wave takes a run of groups, counts first and then
// writes. `scr` is not in use by another wave.
__device__ void w_emit(const BInst& I, const WSums& s, uint32_t groups, int64_t key0, const uint16_t* attr, uint32_t* scr,
                       int64_t* out, uint32_t* status) {
  const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
  const uint32_t run = (groups + kWBlock - 1) / kWBlock * kWave, lo = wave * run, hi = min(lo + run, groups);
  uint32_t n = 0;
  for (uint32_t b = lo; b < hi; b += kWave) n += (uint32_t)__popcll(__ballot(b + lane < hi && s.count[b + lane] != 0));
  if (lane == 0) scr[wave] = n;
  __syncthreads();
  int64_t at = *out;
#pragma unroll
  for (uint32_t w = 0; w < kWBlock / kWave; ++w) {
    at += w < wave ? scr[w] : 0u;
    *out += scr[w];
  }
  for (uint32_t b = lo; b < hi; b += kWave) {
    const uint32_t g = b + lane;
    const bool has = g < hi && s.count[g] != 0;
    const uint64_t all = __ballot(has);
    const int64_t o = at + __popcll(all & ((1ull << lane) - 1));
    at += __popcll(all);
    if (!has) continue;
    if (o < I.out_cap) {
      I.out_key[o] = key0 + (attr ? (int64_t)attr[g] : (int64_t)g);
      I.out_sp[o] = (int64_t)s.price[g];
      I.out_sq[o] = (int64_t)s.qty[g];
      I.out_cnt[o] = (int64_t)s.count[g];
    } else {
      set_status(status, kDevOverflow);
    }
  }
}

// The attributes of few dim rows over a wide range, numbered in order: which
// occur, how many do before each word of 32, and the number's attribute.
struct WRanks {
  uint32_t* bits;
  uint16_t* before;
  uint16_t* attr;
  __device__ __forceinline__ uint32_t of(uint32_t a) const { return before[a >> 5] + (uint32_t)__popc(bits[a >> 5] & ((1u << (a & 31)) - 1u)); }
};

// What the steps of an instance share, in LDS (each step reads what it needs:
// kept in registers over all of them, these values spill).
struct WPlan {
  int32_t kmin, amin;
  uint32_t range;          // of the keys
  uint32_t groups;         // group numbers
  uint32_t chunks;
  uint32_t ranked, in_lds;
  uint32_t front;          // bytes of LDS in front of the join table
  uint32_t lb;             // log2 of a table entry's bits
};

struct WShared {
  uint64_t pool[kWPool / 8];
  uint32_t cnt[kWMaxChunks + 1];
  uint32_t scr[kWBlock / kWave];
  uint64_t red[3][kWBlock / kWave];  // rows passed, join matches, table entries
  int32_t mn[2][kWBlock / kWave], mx[2][kWBlock / kWave];
  WPlan p;
  int64_t item;

  __device__ __forceinline__ char* bytes() { return reinterpret_cast<char*>(pool); }
  __device__ __forceinline__ WSums sums(uint32_t groups) {
    return WSums{pool, pool + groups, reinterpret_cast<uint32_t*>(pool + 2 * (size_t)groups)};
  }
  __device__ __forceinline__ WRanks ranks() {
    uint32_t* const bits = reinterpret_cast<uint32_t*>(bytes() + kWPool - kWRankBytes);
    uint16_t* const before = reinterpret_cast<uint16_t*>(bits + 65536 / 32);
    return WRanks{bits, before, before + 65536 / 32};
  }
};

__device__ __forceinline__ uint32_t w_uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ int32_t w_uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Step 1: the ranges, and from them the plan. False: the instance is not one for arrays.
__device__ __forceinline__ bool w_plan(const BWhole& a, const BInst& I, WShared& s) {
  const uint32_t t = threadIdx.x, lane = lane_id(), wave = t / kWave;
  const int32_t m = (int32_t)I.m;
  int32_t kmin = INT32_MAX, kmax = INT32_MIN, amin = INT32_MAX, amax = INT32_MIN;
  for (int32_t b = 0; b < m; b += kWTile) {
    int32_t key[kWRows], at[kWRows];
#pragma unroll
    for (int k = 0; k < kWRows; ++k) {
      const int32_t j = min(b + (int32_t)t + k * kWBlock, m - 1);
      key[k] = I.pk[j];
      at[k] = w_attr(I, j);
    }
#pragma unroll
    for (int k = 0; k < kWRows; ++k) {
      kmin = min(kmin, key[k]);
      kmax = max(kmax, key[k]);
      amin = min(amin, at[k]);
      amax = max(amax, at[k]);
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    kmin = min(kmin, __shfl_xor(kmin, d, kWave));
    kmax = max(kmax, __shfl_xor(kmax, d, kWave));
    amin = min(amin, __shfl_xor(amin, d, kWave));
    amax = max(amax, __shfl_xor(amax, d, kWave));
  }
  if (lane == 0) {
    s.mn[0][wave] = kmin;
    s.mx[0][wave] = kmax;
    s.mn[1][wave] = amin;
    s.mx[1][wave] = amax;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWBlock / kWave; ++w) {
    kmin = min(kmin, s.mn[0][w]);
    kmax = max(kmax, s.mx[0][w]);
    amin = min(amin, s.mn[1][w]);
    amax = max(amax, s.mx[1][w]);
  }
  const int64_t range = m > 0 ? (int64_t)kmax - kmin + 1 : 0;
  const int64_t arange = m > 0 ? (int64_t)amax - amin + 1 : 0;  // 1 for GROUP BY fk
  const bool by_fk = I.group_by == REL_GROUP_FK, by_flag = I.group_by == REL_GROUP_PRIO_FLAG;
  // (numbered attributes: the sums of a chunk hold them all)
  const bool ranked = !by_fk && !by_flag && arange > kWCap && arange <= 65535 && m <= kWRankRows;
  uint32_t distinct = 0;
  if (ranked) {
    const WRanks r = s.ranks();
    static_assert(65536 / 32 == 2 * kWBlock, "two words per thread");
    r.bits[2 * t] = 0;
    r.bits[2 * t + 1] = 0;
    __syncthreads();
    for (int32_t j = (int32_t)t; j < m; j += kWBlock) {
      const uint32_t at = (uint32_t)(I.grp[j] - amin);
      atomicOr(&r.bits[at >> 5], 1u << (at & 31));
    }
    __syncthreads();
    const uint32_t w0 = r.bits[2 * t], w1 = r.bits[2 * t + 1];
    uint32_t n = block_excl_scan<kWBlock>((uint32_t)(__popc(w0) + __popc(w1)), s.scr, &distinct);
    r.before[2 * t] = (uint16_t)n;
    r.before[2 * t + 1] = (uint16_t)(n + (uint32_t)__popc(w0));
    for (uint32_t w = w0; w != 0; w &= w - 1) r.attr[n++] = (uint16_t)(64 * t + (uint32_t)__ffs((int)w) - 1u);
    for (uint32_t w = w1; w != 0; w &= w - 1) r.attr[n++] = (uint16_t)(64 * t + 32 + (uint32_t)__ffs((int)w) - 1u);
  }
  const int64_t groups = by_fk ? range : by_flag ? arange * 256 : ranked ? (int64_t)distinct : arange;
  const int64_t chunks = (groups + kWCap - 1) / kWCap;
  // (the table takes the place of the instance's hash table, of at least 2 m 8-byte slots)
  const bool fits = range <= 2 * (int64_t)m + 16 && arange <= 65535 && groups <= kWMaxRange && (chunks <= 1 || I.n <= a.spill_rows);
  if (t == 0 && fits) {
    // LDS: the sums of a chunk or a sorted tile, and behind them the join table
    // when there is room (the tile and the sums are not in use at the same time)
    const uint32_t sums_bytes = ((uint32_t)(chunks <= 1 ? groups : kWCap) * kWGroupBytes + 15) / 16 * 16;
    s.p.kmin = kmin;
    s.p.amin = amin;
    s.p.range = (uint32_t)range;
    s.p.groups = (uint32_t)groups;
    s.p.chunks = (uint32_t)chunks;
    s.p.ranked = ranked;
    s.p.front = chunks <= 1 ? sums_bytes : max(sums_bytes, (uint32_t)kWSortBytes);
    const WBits bits = WBits::of(by_fk ? 1 : ranked ? groups : arange);
    s.p.lb = bits.lb;
    s.p.in_lds = (int64_t)s.p.front + (int64_t)bits.words((uint64_t)range) * 4 <= (ranked ? kWPool - kWRankBytes : kWPool);
  }
  __syncthreads();
  return fits;
}

// Step 2: the join table, a slice of the range at a time. False: a dim key
// occurs twice, and its entry is the bitwise or of two rows' values, which may
// name a group that does not exist.
__device__ __forceinline__ bool w_build(const BWhole& a, const BInst& I, WShared& s) {
  const uint32_t t = threadIdx.x, lane = lane_id(), wave = t / kWave;
  const int32_t m = (int32_t)I.m;
  const uint32_t range = w_uni(s.p.range), kmin = (uint32_t)w_uni(s.p.kmin);
  const int32_t amin = w_uni(s.p.amin);
  const bool in_lds = w_uni(s.p.in_lds) != 0, ranked = w_uni(s.p.ranked) != 0;
  const WBits bits{w_uni(s.p.lb)};
  const WRanks ranks = s.ranks();
  uint32_t* const lds_table = reinterpret_cast<uint32_t*>(s.bytes() + (in_lds ? w_uni(s.p.front) : 0u));
  uint32_t* const mem_table = reinterpret_cast<uint32_t*>(I.jslots);
  const uint32_t slice = in_lds ? range : (uint32_t)((ranked ? kWPool - kWRankBytes : kWPool) / 4) << (5 - bits.lb);
  uint32_t entries = 0;
  // (a range below 2^32 and slices of at most 2^21 entries: `lo` may pass the range's end once, so it has 64 bits)
  for (uint64_t lo = 0; lo < range; lo += slice) {
    const uint32_t len = (uint32_t)min((uint64_t)slice, range - lo), words = bits.words(len);
    for (uint32_t i = t; i < words; i += kWBlock) lds_table[i] = 0;
    __syncthreads();
    for (int32_t b = 0; b < m; b += kWTile) {
      int32_t key[kWRows], at[kWRows];
#pragma unroll
      for (int k = 0; k < kWRows; ++k) {
        const int32_t j = min(b + (int32_t)t + k * kWBlock, m - 1);
        key[k] = I.pk[j];
        at[k] = w_attr(I, j);
      }
#pragma unroll
      for (int k = 0; k < kWRows; ++k) {
        const uint32_t off = (uint32_t)key[k] - kmin - (uint32_t)lo;
        if (b + (int32_t)t + k * kWBlock < m && off < len) {
          const uint32_t v = (uint32_t)at[k] - (uint32_t)amin;
          atomicOr(&lds_table[bits.word(off)], ((ranked ? ranks.of(v) : v) + 1u) << bits.shift(off));
        }
      }
    }
    __syncthreads();
    for (uint32_t i = t; i < words; i += kWBlock) {
      const uint32_t w = lds_table[i];
      entries += bits.used(w);
      if (!in_lds) mem_table[bits.word((uint32_t)lo) + i] = w;
    }
    if (!in_lds) __syncthreads();
  }
  const uint64_t all = wave_sum_u64(entries);
  if (lane == 0) s.red[2][wave] = all;
  const uint32_t groups = w_uni(s.p.groups);
  if (w_uni(s.p.chunks) <= 1) s.sums(groups).clear(groups);
  for (uint32_t c = t; c <= (uint32_t)kWMaxChunks; c += kWBlock) s.cnt[c] = 0;
  __syncthreads();
  uint32_t e = 0;
#pragma unroll
  for (int w = 0; w < kWBlock / kWave; ++w) e += (uint32_t)s.red[2][w];
  if (w_uni(e) == (uint32_t)m) return true;
  if (t == 0) set_status(a.status, kDevDupKey);
  return false;
}

// One thread's rows of a tile, all loads in flight together.
struct WRows {
  int32_t d[kWRows], f[kWRows], q[kWRows];
  int64_t p[kWRows];
  uint32_t fl[kWRows];
};
__device__ __forceinline__ void w_load(const BInst& I, int32_t base, int32_t n, bool by_flag, WRows& r) {
  const int32_t* const day = I.day + base;
  const int32_t* const fk = I.fk + base;
  const int32_t* const qty = I.qty + base;
  const long long* const price = (const long long*)I.price + base;
#pragma unroll
  for (int k = 0; k < kWRows; ++k) {
    const uint32_t i = threadIdx.x + k * kWBlock;
    const bool ok = (int32_t)i < n - base;
    r.d[k] = INT32_MAX;  // (a row past the end fails any day < day_lt)
    if (ok) {
      r.d[k] = ld_once(day + i);
      r.f[k] = ld_once(fk + i);
      r.q[k] = ld_once(qty + i);
      r.p[k] = ld_once(price + i);
    }
  }
  if (by_flag) {
    const int8_t* const flag = I.flag + base;
#pragma unroll
    for (int k = 0; k < kWRows; ++k) {
      const uint32_t i = threadIdx.x + k * kWBlock;
      r.fl[k] = (int32_t)i < n - base ? (uint32_t)(uint8_t)flag[i] : 0u;
    }
  }
}

// The workgroup's spill memory.
struct WSpill {
  uint64_t* gq;   // group in its chunk, quantity << 32
  int64_t* price;
  uint32_t* off;  // [tiles][kWMaxChunks + 1]
  __device__ __forceinline__ explicit WSpill(const BWhole& a)
      : gq(a.spill + (size_t)blockIdx.x * 2 * (size_t)a.spill_rows),
        price(reinterpret_cast<int64_t*>(gq + a.spill_rows)),
        off(a.spill_off + (size_t)blockIdx.x * (size_t)((a.spill_rows + kWTile - 1) / kWTile) * (kWMaxChunks + 1)) {}
};

// Step 3: the fact rows, into the sums (kSpill: sorted by chunk into the spill memory).
template <bool kSpill>
__device__ __forceinline__ void w_rows(const BWhole& a, const BInst& I, WShared& s) {
  const uint32_t t = threadIdx.x, lane = lane_id(), wave = t / kWave;
  const int32_t n = (int32_t)I.n, day_lt = I.day_lt;
  const bool by_fk = I.group_by == REL_GROUP_FK, by_flag = I.group_by == REL_GROUP_PRIO_FLAG;
  const uint32_t range = w_uni(s.p.range), kmin = (uint32_t)w_uni(s.p.kmin);
  const bool in_lds = w_uni(s.p.in_lds) != 0;
  const WBits bits{w_uni(s.p.lb)};
  const uint32_t* const lds_table = reinterpret_cast<const uint32_t*>(s.bytes() + (in_lds ? w_uni(s.p.front) : 0u));
  const uint32_t* const mem_table = reinterpret_cast<const uint32_t*>(I.jslots);
  const WSums sums = s.sums(w_uni(s.p.groups));
  const WSpill spill(a);
  uint32_t passed = 0, matched = 0, spilled = 0;
  WRows cur, nxt;
  if (n > 0) w_load(I, 0, n, by_flag, cur);
  // (fewer than 2^31 rows: `base` passes the end by less than a tile)
  for (uint32_t base = 0; base < (uint32_t)n; base += kWTile) {
    if (base + kWTile < (uint32_t)n) w_load(I, (int32_t)(base + kWTile), n, by_flag, nxt);
    uint32_t e[kWRows], g[kWRows];
#pragma unroll
    for (int k = 0; k < kWRows; ++k) {
      const bool pass = cur.d[k] < day_lt && base + t + k * kWBlock < (uint32_t)n;
      passed += pass;
      g[k] = (uint32_t)cur.f[k] - kmin;  // (a key below the smallest wraps to past the range)
      e[k] = 0;
      if (pass && g[k] < range) e[k] = in_lds ? lds_table[bits.word(g[k])] : mem_table[bits.word(g[k])];
    }
#pragma unroll
    for (int k = 0; k < kWRows; ++k) {
      e[k] = bits.get(e[k], g[k]);
      matched += e[k] != 0;
      if (!by_fk) g[k] = by_flag ? (e[k] - 1u) * 256u + cur.fl[k] : e[k] - 1u;
    }
    if constexpr (!kSpill) {
#pragma unroll
      for (int k = 0; k < kWRows; ++k)
        if (e[k] != 0) sums.add(g[k], cur.p[k], cur.q[k]);
    } else {
      // the tile's joined rows, sorted by chunk
      uint32_t rank[kWRows];
#pragma unroll
      for (int k = 0; k < kWRows; ++k) rank[k] = e[k] != 0 ? atomicAdd(&s.cnt[g[k] / kWCap], 1u) : 0u;
      __syncthreads();
      const uint32_t c = t < (uint32_t)kWMaxChunks ? s.cnt[t] : 0u;
      uint32_t total;
      const uint32_t first = block_excl_scan<kWBlock>(c, s.scr, &total);
      uint32_t* const off = spill.off + (size_t)(base / kWTile) * (kWMaxChunks + 1);
      if (t < (uint32_t)kWMaxChunks) {
        s.cnt[t] = first;
        off[t] = spilled + first;
      }
      if (t == 0) off[kWMaxChunks] = spilled + total;
      __syncthreads();
      uint64_t* const sort_gq = s.pool;
      int64_t* const sort_p = reinterpret_cast<int64_t*>(s.pool) + kWTile;
#pragma unroll
      for (int k = 0; k < kWRows; ++k)
        if (e[k] != 0) {
          const uint32_t at = s.cnt[g[k] / kWCap] + rank[k];
          sort_gq[at] = (uint64_t)(g[k] % kWCap) | (uint64_t)(uint32_t)cur.q[k] << 32;
          sort_p[at] = cur.p[k];
        }
      __syncthreads();
      for (uint32_t i = t; i < total; i += kWBlock) {
        spill.gq[spilled + i] = sort_gq[i];
        spill.price[spilled + i] = sort_p[i];
      }
      if (t < (uint32_t)kWMaxChunks) s.cnt[t] = 0;
      spilled += total;
      __syncthreads();
    }
    cur = nxt;
  }
  const uint64_t p = wave_sum_u64(passed), q = wave_sum_u64(matched);
  if (lane == 0) {
    s.red[0][wave] = p;
    s.red[1][wave] = q;
  }
  __syncthreads();
}

// Step 4: the groups, to the output. Returns their number.
__device__ __forceinline__ int64_t w_groups(const BWhole& a, const BInst& I, WShared& s) {
  const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
  const uint32_t groups = w_uni(s.p.groups), chunks = w_uni(s.p.chunks);
  // (keys: dim.grp, fk, or prio * 256 + flag, all counted from their smallest)
  const int64_t key0 = I.group_by == REL_GROUP_FK          ? (int64_t)w_uni(s.p.kmin)
                       : I.group_by == REL_GROUP_PRIO_FLAG ? (int64_t)w_uni(s.p.amin) * 256
                                                           : (int64_t)w_uni(s.p.amin);
  int64_t out = 0;
  if (chunks <= 1) {
    w_emit(I, s.sums(groups), groups, key0, w_uni(s.p.ranked) != 0 ? s.ranks().attr : nullptr, s.scr, &out, a.status);
    return out;
  }
  const WSpill spill(a);
  const uint32_t tiles = ((uint32_t)I.n + kWTile - 1) / kWTile;
  for (uint32_t c = 0; c < chunks; ++c) {
    const uint32_t here = min((uint32_t)kWCap, groups - c * kWCap);
    const WSums sums = s.sums(here);
    sums.clear(here);
    __syncthreads();
    // a wave takes the chunk's run of every 16th tile
    for (uint32_t tile = wave; tile < tiles; tile += kWBlock / kWave) {
      const uint32_t lo = spill.off[(size_t)tile * (kWMaxChunks + 1) + c], hi = spill.off[(size_t)tile * (kWMaxChunks + 1) + c + 1];
      for (uint32_t i0 = lo + lane; i0 - lane < hi; i0 += kWave * kWRows) {
        uint64_t gq[kWRows];
        int64_t p[kWRows];
#pragma unroll
        for (int k = 0; k < kWRows; ++k) {
          const uint32_t i = min(i0 + k * kWave, hi - 1);
          gq[k] = spill.gq[i];
          p[k] = spill.price[i];
        }
#pragma unroll
        for (int k = 0; k < kWRows; ++k)
          if (i0 + k * kWave < hi) sums.add((uint32_t)gq[k], p[k], (int32_t)(uint32_t)(gq[k] >> 32));
      }
    }
    __syncthreads();
    w_emit(I, sums, here, key0 + (int64_t)c * kWCap, nullptr, s.scr, &out, a.status);
    __syncthreads();
  }
  return out;
}

__global__ __launch_bounds__(kWBlock) void k_batch_whole(BWhole a) {
  __shared__ WShared s;
  const uint32_t t = threadIdx.x;
  // (at most n + 1 tickets per workgroup, whatever the ticket holds)
  for (int32_t turn = 0; turn <= a.n; ++turn) {
    if (t == 0) s.item = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)a.ticket, 1ull);
    __syncthreads();
    const int64_t item = s.item;
    if (item < 0 || item >= a.n) break;
    const int32_t inst = w_uni(a.order[item]);  // (the same on every lane: scalar loads)
    const BInst& I = a.inst[inst];
    if (!w_plan(a, I, s)) {
      if (t == 0) dev_add<uint32_t>(a.left, 1u);
      __syncthreads();
      continue;
    }
    if (!w_build(a, I, s)) {  // (the call reports the key; the instance keeps the zeros it started with)
      if (t == 0) a.done[inst] = 1u;
      __syncthreads();
      continue;
    }
    if (w_uni(s.p.chunks) <= 1) w_rows<false>(a, I, s);
    else w_rows<true>(a, I, s);
    const int64_t out = w_groups(a, I, s);
    if (t == 0) {
      uint64_t p = 0, q = 0;
      for (int w = 0; w < kWBlock / kWave; ++w) {
        p += s.red[0][w];
        q += s.red[1][w];
      }
      I.stats[0] = (int64_t)p;
      I.stats[1] = (int64_t)q;
      I.stats[2] = out;
      *I.d_n = out;
      a.done[inst] = 1u;
      if (out > (int64_t)I.gmask + 2) set_status(a.status, kDevOverflow);  // more groups than the table sized for them has slots
    }
    __syncthreads();
  }
}

const rel_batch_tuning kDefaultTuning[] = {
    {12, 4, 256, 512, 1024, 0},
    {16, 4, 256, 512, 8192, 0},
    {20, 4, 256, 512, 16384, 0},
    {31, 4, 256, 512, 65536, 0},
};

bool tuning_ok(const rel_batch_tuning& t) {
  const bool ipt = t.items_per_thread == 1 || t.items_per_thread == 2 || t.items_per_thread == 4 || t.items_per_thread == 8;
  const bool blk = t.block == 64 || t.block == 128 || t.block == 256 || t.block == 512;
  return ipt && blk && t.lds_groups_max >= 0 && t.lds_groups_max <= kBLdsSlots / 2 && t.lds_join_max >= 0 &&
         t.lds_join_max <= kBLdsJoinSlots / 2 && t.rows_per_item > 0 &&
         t.rows_per_item % (t.block * t.items_per_thread) == 0 && t.log2_rows_below > 0 && t.log2_rows_below <= 31;
}

}  // namespace

struct BucketPlan {
  rel_batch_tuning t;
  int64_t build_lo = 0, probe_lo = 0;  // where the item lists begin
  BList build{}, probe{};
};

struct rel_batch {
  rel_ctx* ctx = nullptr;
  int32_t k = 0;
  std::vector<BucketPlan> buckets;
  void* mem = nullptr;
  BInst* d_inst = nullptr;
  BItem* d_items = nullptr;
  int64_t* d_tickets = nullptr;
  int64_t* d_stats = nullptr;
  uint32_t* d_status = nullptr;  // this batch's status word, cleared at the start of every run
  uint64_t* d_join = nullptr;
  GroupSlot* d_groups = nullptr;
  int64_t fin_lo = 0;
  BList fin{};
  size_t zero_words = 0;  // tickets + stats + status word + whole-instance words
  BWhole whole{};         // the instances that one workgroup takes each
  unsigned whole_grid = 0;
  void* spill = nullptr;
  hipStream_t cap = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

template <int BLOCK, bool LJ>
void launch_probe(hipStream_t s, unsigned grid, int ipt, const BInst* inst, const BItem* items,
                  int64_t* ticket, uint32_t* status, BList list) {
  switch (ipt) {
    case 1: hipLaunchKernelGGL((k_batch_probe<BLOCK, 1, LJ>), dim3(grid), dim3(BLOCK), 0, s, inst, items, ticket, status, list); break;
    case 2: hipLaunchKernelGGL((k_batch_probe<BLOCK, 2, LJ>), dim3(grid), dim3(BLOCK), 0, s, inst, items, ticket, status, list); break;
    case 4: hipLaunchKernelGGL((k_batch_probe<BLOCK, 4, LJ>), dim3(grid), dim3(BLOCK), 0, s, inst, items, ticket, status, list); break;
    default: hipLaunchKernelGGL((k_batch_probe<BLOCK, 8, LJ>), dim3(grid), dim3(BLOCK), 0, s, inst, items, ticket, status, list); break;
  }
}

void launch_build(hipStream_t s, unsigned grid, int block, const BInst* inst, const BItem* items,
                  int64_t* ticket, uint32_t* status, BList list) {
  switch (block) {
    case 64: hipLaunchKernelGGL(k_batch_build<64>, dim3(grid), dim3(64), 0, s, inst, items, ticket, status, list); break;
    case 128: hipLaunchKernelGGL(k_batch_build<128>, dim3(grid), dim3(128), 0, s, inst, items, ticket, status, list); break;
    case 256: hipLaunchKernelGGL(k_batch_build<256>, dim3(grid), dim3(256), 0, s, inst, items, ticket, status, list); break;
    default: hipLaunchKernelGGL(k_batch_build<512>, dim3(grid), dim3(512), 0, s, inst, items, ticket, status, list); break;
  }
}

template <bool LJ>
void launch_probe_blk(hipStream_t s, unsigned grid, int block, int ipt, const BInst* inst, const BItem* items,
                      int64_t* ticket, uint32_t* status, BList list) {
  switch (block) {
    case 64: launch_probe<64, LJ>(s, grid, ipt, inst, items, ticket, status, list); break;
    case 128: launch_probe<128, LJ>(s, grid, ipt, inst, items, ticket, status, list); break;
    case 256: launch_probe<256, LJ>(s, grid, ipt, inst, items, ticket, status, list); break;
    default: launch_probe<512, LJ>(s, grid, ipt, inst, items, ticket, status, list); break;
  }
}

void launch_probe_any(hipStream_t s, unsigned grid, int block, int ipt, bool lj, const BInst* inst,
                      const BItem* items, int64_t* ticket, uint32_t* status, BList list) {
  if (lj) launch_probe_blk<true>(s, grid, block, ipt, inst, items, ticket, status, list);
  else launch_probe_blk<false>(s, grid, block, ipt, inst, items, ticket, status, list);
}

// Workgroups for a persistent kernel: enough to fill the chip, never more than the items.
unsigned persistent_grid(const rel_ctx* ctx, int64_t items, int block) {
  const int64_t per_cu = block >= 512 ? 2 : block >= 256 ? 4 : 8;
  int64_t g = (int64_t)ctx->num_cus * per_cu;
  if (g > items) g = items;
  return (unsigned)(g < 1 ? 1 : g);
}

// Rows and keys per item where the tuning's (up to 65536, found on batches of
// thousands) would leave CUs idle: a CU's share, of the rows that one kernel takes
// (a bucket's) and of one kind, as rows of instances of many groups cost some
// twenty times the others' (an update of the device table each). Where the groups
// are few, no less than what pays for an item's LDS table, which is set up and
// flushed once per item. In us: 8 instances of up to 1M rows 606 by the tuning's
// items, which kept 20 workgroups busy, 187 so; 4 of 1M rows and 100 groups 125, 86
// so, 229 with a quarter of the share; 64 of 1K to 1M rows, 1 to 65536 groups, 994
// with a CU's share of the whole batch, 670 so.
constexpr int64_t kItemMinRows = 2048, kItemMinKeys = 1024;
constexpr int64_t kKeyItemsPerCu = 4;

// The most groups that an instance can have, or its hint where that is less.
int64_t group_bound(const rel_batch_item& it, bool* hinted) {
  const int64_t ub = it.q.group_by == REL_GROUP_PRIO_FLAG ? std::min<int64_t>(it.fact.n, 65536) : std::min(it.fact.n, it.dim.m);
  *hinted = it.group_capacity > 0 && it.group_capacity < ub;
  return *hinted ? it.group_capacity : ub;
}

// More groups than an LDS table holds. (The bound of (prio, flag) is of the values
// there could be, not of those that occur.)
bool many_groups(const rel_batch_item& it) {
  bool hinted;
  return it.q.group_by != REL_GROUP_PRIO_FLAG && group_bound(it, &hinted) > kBLdsSlots / 2;
}

// What an instance costs either way, in ns: a workgroup that takes it whole while
// most CUs are idle and while all are busy, and its share of what the shared tables
// cost the chip. Fitted to 261 batches of 1 to 256 equal instances of 1K to 1M
// rows, 100 to 8M dim keys and all three group keys, timed both ways, and to 61
// batches of 8 to 2048 instances of different sizes, timed at up to 20 splits: the
// way chosen is within 0.3% of the better one on average (20% at worst), and of 44
// other batches of different sizes within 0.6% of the best measured split. Some of
// the equal ones, all by the shared tables / all whole, in us:
//   1 of 1K rows, 100 keys        28 /   30     1 of 1K rows, 1M keys         95 / 2639
//   1 of 300K, 75K, 300 groups    75 /  368     64 of 30K, 7.5K, 300 groups   94 /   49
//   16 of 30K, 3K, fk            116 /   47     16 of 300K, 75K, fk          662 /  517
//   64 of 1M, 250K, 300 groups  1343 / 1483     256 of 300K, 75K, fk        8756 /  803
// Keys count as rows do: the join table of many keys is filled in LDS slice by
// slice, with all keys read again for each, so that whole instances of 8M keys
// took 136 ms.
struct BatchCost {
  double alone, loaded, shared, shared_wait;
  int bucket;
};
BatchCost batch_cost(const rel_batch_item& it, int bucket) {
  bool hinted;
  const int64_t bound = group_bound(it, &hinted);
  const double n = (double)it.fact.n, m = (double)it.dim.m;
  const bool fk = it.q.group_by == REL_GROUP_FK, flag = it.q.group_by == REL_GROUP_PRIO_FLAG;
  const int64_t groups = fk ? it.dim.m : flag ? 0 : std::min<int64_t>(it.group_capacity > 0 ? std::min(it.group_capacity, it.dim.m) : it.dim.m, 65536);
  const int64_t chunks = std::max<int64_t>((groups + kWCap - 1) / kWCap, 1);
  const double table = m * (fk ? 1 : flag ? 8 : 16) / 8;  // bytes, of the entries' likely width
  const double front = (double)std::min<int64_t>(groups, kWCap) * kWGroupBytes;
  const bool in_lds = front + table <= kWPool, spills = chunks > 1;
  const double slices = in_lds ? 1 : std::ceil(table / kWPool);
  const double keys = 8000 + m * (0.25 + 0.25 * slices) + (spills ? 7000.0 * (double)chunks : 0);
  BatchCost c;
  c.alone = keys + n * ((in_lds ? 0.7 : 1.0) + (spills ? 0.8 : 0));
  c.loaded = keys + n * ((in_lds ? 0.8 : 1.6) + (spills ? 1.3 : 0));
  if (groups > kWMaxRange) c.alone = c.loaded = 1e15;  // (more keys than group numbers: w_plan would only find it out)
  const bool many = many_groups(it);
  double slots = 16;
  while (slots < 2 * (double)bound + 1) slots *= 2;
  c.shared = 50 + n * (many ? 0.1 : 0.005) + m * 0.06 + slots * 0.0115;
  c.shared_wait = 7000 + (many ? 25000 : 0) + (it.dim.m > kBLdsJoinSlots / 2 ? 17000 : m * 5) + (flag && it.fact.n >= 2048 ? 6400 : 0);
  c.bucket = bucket;
  return c;
}

// How many of the instances, costliest first, go by the shared tables, so that the
// times of both ways, which follow one another, add up to the least. Each bucket of
// the tuning among them is two kernels more. A split costs more than its parts'
// estimates (the whole instances that are left are not those that were expected to
// be quick, and the shared tables' kernels have few items), so it has to promise a
// tenth: 373 instances of 1K to 84K rows with the 15 costliest apart 363 us, all
// whole 226; 42 of up to 108K rows by the shared tables 152, all whole 134.
constexpr double kBucketNs = 5000, kSplitFactor = 1.1;
int32_t whole_from(const std::vector<BatchCost>& cost, int cus) {
  const int32_t k = (int32_t)cost.size();
  double after = 0, shared = 0, wait = 0, best = 0;
  for (const BatchCost& c : cost) after += c.loaded;
  uint64_t buckets = 0;  // a bit each (31 at most)
  int32_t at = 0;
  for (int32_t c = 0; c <= k; ++c) {
    const double whole = c < k ? std::max(cost[c].alone, after / cus) : 0;
    const double more = kBucketNs * std::max(__builtin_popcountll(buckets) - 1, 0);
    const double t = (whole + shared + wait + more) * (c > 0 && c < k ? kSplitFactor : 1);
    if (c == 0 || t < best) {
      best = t;
      at = c;
    }
    if (c == k) break;
    after -= cost[c].loaded;
    shared += cost[c].shared;
    wait = std::max(wait, cost[c].shared_wait);
    buckets |= 1ull << cost[c].bucket;
  }
  return at;
}

void free_batch(rel_batch* b) {
  if (!b) return;
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  if (b->cap) (void)hipStreamDestroy(b->cap);
  if (b->mem) (void)hipFree(b->mem);
  if (b->spill) (void)hipFree(b->spill);
  delete b;
}

}  // namespace

extern "C" {

rel_status rel_batch_create(rel_ctx* ctx, const rel_batch_item* items, int32_t k, const rel_batch_tuning* tuning,
                            int32_t n_tuning, rel_batch** out) {
  return rel_batch_create_as(ctx, items, k, tuning, n_tuning, REL_BATCH_AUTO, out);
}

rel_status rel_batch_create_as(rel_ctx* ctx, const rel_batch_item* items, int32_t k, const rel_batch_tuning* tuning,
                               int32_t n_tuning, int32_t way, rel_batch** out) {
  if (way < REL_BATCH_AUTO || way > REL_BATCH_WHOLE) return relh::fail(ctx, REL_INVALID_ARG, "rel_batch_create_as: bad way");
  if (!ctx || !out || k < 0 || (k > 0 && !items) || n_tuning < 0 || (n_tuning > 0 && !tuning))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_batch_create: bad argument");
  std::vector<rel_batch_tuning> tun;
  if (n_tuning > 0) tun.assign(tuning, tuning + n_tuning);
  else tun.assign(std::begin(kDefaultTuning), std::end(kDefaultTuning));
  for (size_t i = 0; i < tun.size(); ++i) {
    if (!tuning_ok(tun[i])) return relh::fail(ctx, REL_INVALID_ARG, "rel_batch_create: tuning entry %zu invalid", i);
    if (i > 0 && tun[i].log2_rows_below <= tun[i - 1].log2_rows_below)
      return relh::fail(ctx, REL_INVALID_ARG, "rel_batch_create: tuning buckets must ascend");
  }
  // validate instances
  for (int32_t i = 0; i < k; ++i) {
    const rel_batch_item& it = items[i];
    const int64_t n = it.fact.n, m = it.dim.m;
    const int gb = it.q.group_by;
    if (n < 0 || m < 0 || gb < REL_GROUP_PRIO_FLAG || gb > REL_GROUP_DIM_GRP || it.group_capacity < 0 ||
        !it.out.key || !it.out.sum_price || !it.out.sum_qty || !it.out.count || !it.out.d_n_groups || it.out.cap < 0)
      return relh::fail(ctx, REL_INVALID_ARG, "rel_batch_create: instance %d invalid", i);
    if ((n > 0 && (!it.fact.fk || !it.fact.price_cents || !it.fact.qty || !it.fact.day ||
                   (gb == REL_GROUP_PRIO_FLAG && !it.fact.flag))) ||
        (m > 0 && (!it.dim.pk || (gb == REL_GROUP_PRIO_FLAG && !it.dim.prio) || (gb == REL_GROUP_DIM_GRP && !it.dim.grp))))
      return relh::fail(ctx, REL_INVALID_ARG, "rel_batch_create: instance %d misses a column", i);
    if (n >= (1ll << 31) || m >= (1ll << 30)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_batch_create: instance %d too large", i);
  }

  rel_batch* b = new rel_batch();
  b->ctx = ctx;
  b->k = k;
  auto bucket_of = [&](int64_t n) {
    for (size_t t = 0; t < tun.size(); ++t)
      if (n < (1ll << tun[t].log2_rows_below)) return (int)t;
    return (int)tun.size() - 1;
  };

  // costliest instance first; from `order[n_shared]` on they are taken whole
  std::vector<BatchCost> costs(k), sorted_costs(k);
  for (int32_t i = 0; i < k; ++i) costs[i] = batch_cost(items[i], bucket_of(items[i].fact.n));
  std::vector<int32_t> order(k);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return costs[x].alone > costs[y].alone; });
  for (int32_t i = 0; i < k; ++i) sorted_costs[i] = costs[order[i]];
  const int32_t n_shared = way == REL_BATCH_SHARED ? k : way == REL_BATCH_WHOLE ? 0 : whole_from(sorted_costs, ctx->num_cus);
  const int32_t n_whole = k - n_shared;
  b->whole_grid = (unsigned)std::min<int32_t>(n_whole, ctx->num_cus);
  int64_t shared_keys = 0, spill_rows = 0;
  for (int32_t p = 0; p < k; ++p) {
    const rel_batch_item& it = items[order[p]];
    if (p < n_shared) {
      shared_keys += it.dim.m;
      continue;
    }
    const int64_t groups = it.q.group_by == REL_GROUP_FK         ? 2 * it.dim.m
                           : it.q.group_by == REL_GROUP_PRIO_FLAG ? 0
                           : it.group_capacity > 0                ? it.group_capacity
                                                                  : it.dim.m;
    if (groups > kWCap) spill_rows = std::max<int64_t>(spill_rows, it.fact.n);
  }
  const size_t spill_tiles = (size_t)((spill_rows + kWTile - 1) / kWTile);
  const size_t spill_bytes = (size_t)b->whole_grid * ((size_t)spill_rows * 16 + spill_tiles * (kWMaxChunks + 1) * 4);

  // table sizes and offsets
  std::vector<BInst> hinst(k);
  std::vector<size_t> joff(k), goff(k);
  size_t jw = 0, gs = 0;
  size_t jw_shared = 0, gs_shared = 0;
  for (int32_t p = 0; p < k; ++p) {
    const int32_t i = order[p];
    const rel_batch_item& it = items[i];
    const int64_t n = it.fact.n, m = it.dim.m;
    const uint32_t jl = relh::join_log2cap(m, nullptr);
    bool hinted;
    const int64_t ub = group_bound(it, &hinted);
    uint32_t gl = relh::log2_ceil((uint64_t)(std::max<int64_t>(ub, 1) * 2) + 1);
    if (gl < 4) gl = 4;
    const rel_batch_tuning& t = tun[bucket_of(n)];
    BInst& I = hinst[i];
    I.fk = it.fact.fk;
    I.price = it.fact.price_cents;
    I.qty = it.fact.qty;
    I.day = it.fact.day;
    I.flag = it.fact.flag;
    I.pk = it.dim.pk;
    I.prio = it.dim.prio;
    I.grp = it.dim.grp;
    I.n = n;
    I.m = m;
    I.day_lt = it.q.day_lt;
    I.group_by = it.q.group_by;
    I.jmask = (uint32_t)((1ull << jl) - 1);
    I.jshift = 32u - jl;
    I.gmask = (uint32_t)((1ull << gl) - 1);
    I.gshift = 32u - gl;
    I.gprobe = hinted ? kHintProbe : (uint32_t)(1ull << gl);
    I.lds = (t.lds_groups_max > 0 && ub <= t.lds_groups_max) ? 1 : 0;
    I.ljoin = (t.lds_join_max > 0 && m <= t.lds_join_max) ? 1 : 0;
    I.out_key = it.out.key;
    I.out_sp = it.out.sum_price;
    I.out_sq = it.out.sum_qty;
    I.out_cnt = it.out.count;
    I.out_cap = it.out.cap;
    I.d_n = it.out.d_n_groups;
    joff[i] = jw;
    jw += (1ull << jl) + 1;
    goff[i] = gs;
    gs += (1ull << gl) + 1;
    if (p < n_shared) {
      jw_shared = jw;
      gs_shared = gs;
    }
  }

  // work items, largest instance first inside each bucket; fewer rows per item
  // where the tuning's would leave workgroups without one
  std::vector<BItem> hitems;
  // bucket t's instances (t < 0: all), `count` elements each, in items of `step`
  auto add_items = [&](int t, auto&& count, auto&& step) {
    BList l{};
    for (int32_t p = 0; p < k; ++p) {
      const int32_t i = order[p];
      if (t >= 0 && bucket_of(items[i].fact.n) != t) continue;
      const int64_t n = count(i), rows = step(p);
      for (int64_t lo = 0; lo < n; lo += rows) hitems.push_back(BItem{i, 0, lo, std::min(n, lo + rows)});
      l.all += (n + rows - 1) / rows;
      if (p < n_shared) l.n = l.all;
    }
    return l;
  };
  b->buckets.resize(tun.size());
  for (size_t t = 0; t < tun.size(); ++t) {
    BucketPlan& bp = b->buckets[t];
    bp.t = tun[t];
    const int64_t unit = (int64_t)tun[t].block * tun[t].items_per_thread;
    int64_t bucket_rows[2] = {0, 0};  // of instances of few groups, and of many
    for (int32_t p = 0; p < n_shared; ++p) {
      const rel_batch_item& it = items[order[p]];
      if (bucket_of(it.fact.n) == (int)t) bucket_rows[many_groups(it)] += it.fact.n;
    }
    auto share = [&](bool many) {
      const int64_t even = std::max<int64_t>(bucket_rows[many] / ctx->num_cus, many ? 1 : kItemMinRows);
      return std::min<int64_t>((even + unit - 1) / unit * unit, tun[t].rows_per_item);
    };
    const int64_t few_rows = share(false), many_rows = share(true);
    const int64_t key_share = std::max<int64_t>(shared_keys / (ctx->num_cus * kKeyItemsPerCu), kItemMinKeys);
    auto rows = [&](int32_t p) { return p >= n_shared ? (int64_t)tun[t].rows_per_item : many_groups(items[order[p]]) ? many_rows : few_rows; };
    auto keys = [&](int32_t p) { return p < n_shared ? key_share : std::max<int64_t>(tun[t].rows_per_item / 4, 256); };
    bp.build_lo = (int64_t)hitems.size();
    bp.build = add_items((int)t, [&](int32_t i) { return items[i].dim.m; }, keys);
    bp.probe_lo = (int64_t)hitems.size();
    bp.probe = add_items((int)t, [&](int32_t i) { return items[i].fact.n; }, rows);
  }
  b->fin_lo = (int64_t)hitems.size();
  b->fin = add_items(-1, [&](int32_t i) { return (int64_t)hinst[i].gmask + 2; }, [](int32_t) { return kFinItemSlots; });

  // one device allocation: instances, items, tickets + stats, join tables, group tables
  const size_t n_tickets = 2 * tun.size() + 2;
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  const size_t o_inst = 0;
  const size_t o_order = al(o_inst + sizeof(BInst) * (size_t)std::max(k, 1));
  const size_t o_items = al(o_order + sizeof(int32_t) * (size_t)std::max(n_whole, 1));
  const size_t o_zero = al(o_items + sizeof(BItem) * std::max<size_t>(hitems.size(), 1));
  // tickets, per-instance stats, the batch's own status word, the number of
  // instances left and the finished ones' marks (all cleared at the start of every run)
  b->zero_words = n_tickets + 3 * (size_t)k + 2 + ((size_t)k + 1) / 2;
  const size_t o_join = al(o_zero + 8 * b->zero_words);
  const size_t o_groups = al(o_join + 8 * jw);
  const size_t total = al(o_groups + sizeof(GroupSlot) * gs);
  if (relh::device_alloc(ctx, total, &b->mem) != REL_OK) {
    free_batch(b);
    return relh::fail(ctx, REL_OOM, "rel_batch_create: %zu bytes of device memory", total);
  }
  // (after the memory that the batch cannot do without)
  if (spill_rows > 0 && (spill_bytes > kWMaxSpill || hipMalloc(&b->spill, spill_bytes) != hipSuccess)) {
    (void)hipGetLastError();
    b->spill = nullptr;
    spill_rows = 0;  // instances with more groups than one chunk go the other way
  }
  char* base = (char*)b->mem;
  b->d_inst = (BInst*)(base + o_inst);
  b->d_items = (BItem*)(base + o_items);
  b->d_tickets = (int64_t*)(base + o_zero);
  b->d_stats = b->d_tickets + n_tickets;
  b->d_status = (uint32_t*)(b->d_stats + 3 * (size_t)k);
  b->d_join = (uint64_t*)(base + o_join);
  b->d_groups = (GroupSlot*)(base + o_groups);
  for (int32_t i = 0; i < k; ++i) {
    hinst[i].jslots = b->d_join + joff[i];
    hinst[i].gslots = b->d_groups + goff[i];
    hinst[i].stats = b->d_stats + 3 * (size_t)i;
  }
  rel_status st = REL_OK;
  auto hip = [&](hipError_t x, const char* what) {
    if (x != hipSuccess && st == REL_OK) st = relh::hip_fail(ctx, x, what);
  };
  if (k > 0) hip(hipMemcpy(b->d_inst, hinst.data(), sizeof(BInst) * k, hipMemcpyHostToDevice), "copy instances");
  b->whole = BWhole{b->d_inst, (const int32_t*)(base + o_order), n_whole, b->d_tickets + n_tickets - 1, b->d_status,
                    (uint32_t*)(b->d_stats + 3 * (size_t)k + 2), (uint32_t*)(b->d_stats + 3 * (size_t)k + 1),
                    (uint64_t*)b->spill, (uint32_t*)((char*)b->spill + (size_t)b->whole_grid * (size_t)spill_rows * 16), spill_rows};
  auto list = [&](int64_t shared, int64_t all) { return BList{shared, all, b->whole.left, b->whole.done}; };
  if (n_whole > 0)
    hip(hipMemcpy((void*)b->whole.order, order.data() + n_shared, sizeof(int32_t) * n_whole, hipMemcpyHostToDevice), "copy order");
  if (!hitems.empty()) hip(hipMemcpy(b->d_items, hitems.data(), sizeof(BItem) * hitems.size(), hipMemcpyHostToDevice), "copy items");
  hip(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking), "capture stream");
  if (st != REL_OK) {
    free_batch(b);
    return st;
  }

  // capture: reset, build, probe, finalize
  hip(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal), "begin capture");
  if (st == REL_OK) {
    hipStream_t s = b->cap;
    const unsigned fg = (unsigned)ctx->num_cus * 4;
    hipLaunchKernelGGL(k_batch_reset, dim3(relh::grid_for(ctx, (int64_t)b->zero_words, 256, 4)), dim3(256), 0, s,
                       (uint64_t*)b->d_tickets, (int64_t)b->zero_words, (const BInst*)b->d_inst, k);
    if (b->whole_grid) hipLaunchKernelGGL(k_batch_whole, dim3(b->whole_grid), dim3(kWBlock), 0, s, b->whole);
    if (jw) hipLaunchKernelGGL(k_batch_fill, dim3(fg), dim3(256), 0, s, b->d_join, kJoinEmpty, list((int64_t)jw_shared, (int64_t)jw));
    if (gs) hipLaunchKernelGGL(k_batch_init_groups, dim3(fg), dim3(256), 0, s, b->d_groups, list((int64_t)gs_shared, (int64_t)gs));
    for (size_t t = 0; t < b->buckets.size(); ++t) {
      const BucketPlan& bp = b->buckets[t];
      if (bp.build.all)
        launch_build(s, persistent_grid(ctx, bp.build.all, bp.t.block), bp.t.block, b->d_inst, b->d_items + bp.build_lo,
                     b->d_tickets + 2 * t, b->d_status, list(bp.build.n, bp.build.all));
    }
    for (size_t t = 0; t < b->buckets.size(); ++t) {
      const BucketPlan& bp = b->buckets[t];
      if (bp.probe.all)
        launch_probe_any(s, persistent_grid(ctx, bp.probe.all, bp.t.block), bp.t.block, bp.t.items_per_thread,
                         bp.t.lds_join_max > 0, b->d_inst, b->d_items + bp.probe_lo, b->d_tickets + 2 * t + 1, b->d_status,
                         list(bp.probe.n, bp.probe.all));
    }
    if (b->fin.all)
      hipLaunchKernelGGL(k_batch_finalize, dim3(persistent_grid(ctx, b->fin.all, 256)), dim3(256), 0, s, b->d_inst,
                         b->d_items + b->fin_lo, b->d_tickets + 2 * tun.size(), b->d_status, list(b->fin.n, b->fin.all));
    hip(hipGetLastError(), "batch kernels");
    hipGraph_t g = nullptr;
    hipError_t ee = hipStreamEndCapture(s, &g);
    hip(ee, "end capture");
    b->graph = g;
    if (st == REL_OK) hip(hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0), "instantiate graph");
  }
  if (st != REL_OK) {
    free_batch(b);
    return st;
  }
  *out = b;
  return REL_OK;
}

rel_status rel_batch_run(rel_batch* b) {
  if (!b) return REL_INVALID_ARG;
  relh::KernelTimer kt(b->ctx, "batch_graph");
  REL_HIP_CHECK(b->ctx, hipGraphLaunch(b->exec, b->ctx->stream));
  return REL_OK;
}

rel_status rel_batch_sync(rel_batch* b, rel_stats* stats) {
  if (!b) return REL_INVALID_ARG;
  rel_ctx* ctx = b->ctx;
  REL_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
  uint32_t bits = 0;  // the last run's own status word
  REL_HIP_CHECK(ctx, hipMemcpy(&bits, b->d_status, sizeof bits, hipMemcpyDeviceToHost));
  if (stats && b->k > 0) {
    std::vector<int64_t> h(3 * (size_t)b->k);
    REL_HIP_CHECK(ctx, hipMemcpy(h.data(), b->d_stats, 8 * h.size(), hipMemcpyDeviceToHost));
    std::vector<BInst> hi(b->k);
    REL_HIP_CHECK(ctx, hipMemcpy(hi.data(), b->d_inst, sizeof(BInst) * b->k, hipMemcpyDeviceToHost));
    for (int32_t i = 0; i < b->k; ++i) {
      rel_stats& s = stats[i];
      s.rows_in = hi[i].n;
      s.rows_passed = h[3 * i];
      s.join_matches = h[3 * i + 1];
      s.groups = h[3 * i + 2];
      s.join_capacity = (int64_t)hi[i].jmask + 1;
      s.group_capacity = (int64_t)hi[i].gmask + 1;
      s.join_placement = hi[i].ljoin ? REL_PLACE_LDS : REL_PLACE_GLOBAL;
      s.group_placement = hi[i].lds ? REL_PLACE_LDS : REL_PLACE_GLOBAL;
      s.overflowed = 0;
      s.fell_back = 0;
    }
  }
  if (bits & kDevDupKey) return relh::fail(ctx, REL_DUPLICATE_KEY, "rel_batch_sync: duplicate pk");
  if (bits & kDevOverflow) return relh::fail(ctx, REL_OVERFLOW, "rel_batch_sync: a table or output overflowed");
  return REL_OK;
}

rel_status rel_batch_destroy(rel_batch* b) {
  if (!b) return REL_INVALID_ARG;
  (void)hipStreamSynchronize(b->ctx->stream);
  free_batch(b);
  return REL_OK;
}

}  // extern "C"
