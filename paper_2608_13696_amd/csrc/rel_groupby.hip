// Stand-alone group-by over many groups: the rows are partitioned by a hash of
// their key, so that a partition's groups fit a workgroup's LDS.
//
// Updating a table in device memory costs three or four atomics per row, and
// those run at about 27 G/s for the whole chip: 20M rows into 2M groups took
// 2.7 ms. Partitioning reads and writes every row once more, but in runs, and
// then all updates are LDS operations: 0.41 ms (6M rows of 15 groups: 147 -> 41 us).
//
//   k_gb_hist     rows per (tile, bin), one tile per workgroup
//   k_gb_colsum   those summed over chunks of tiles, per bin
//   k_gb_offsets  each tile's place in every bin, relative to the bin's start
//   k_gb_units    bin starts; work units (a bin, or a piece of a large one)
//   k_gb_scatter  a tile's rows sorted by bin in LDS and written as runs
//   k_gb_agg      per unit an LDS table; its groups go straight to the output
//
// The partitioned join's partial sums by group (rel_ops.h, Partials) take the
// same way: their kernel counts them per (chunk, bin) itself, a chunk is a tile.
//
// A key that finds no room in a unit's LDS table, and every group of a bin that
// was cut into pieces (hot keys), goes to the group table in device memory,
// which the caller's finalize kernel appends to the output.
#include <algorithm>
#include <type_traits>

#include "rel_device.h"
#include "rel_host.h"
#include "rel_ops.h"

namespace {

using namespace rel;
using relh::GroupRows;

constexpr int kGbBlock = 1024;
constexpr int kGbRows = 7;  // rows per thread of a tile: 7168 rows of 20 B fill most of a CU's LDS
constexpr int64_t kGbTile = (int64_t)kGbBlock * kGbRows;
constexpr uint32_t kGbMaxBins = 2048;
constexpr int kGbChunks = 32;
constexpr int kGbSubRows = 32768;  // a bin with more rows is cut into pieces of this many
constexpr int kGbProbe = 64;       // LDS probe walk before a row goes to device memory

// Every kernel returns at once when the sample found few groups (`few`, see k_gb_begin).
struct GbArgs {
  GroupRows in;
  const uint32_t* few;
  uint32_t nb, shift;  // bins, 32 - log2(bins)
  int64_t ntiles;
  const uint32_t* more_tiles;  // with partials: beside ntiles (null: none)
  uint32_t max_rows;           // that the memory is laid out for
  uint32_t* status;
  relh::Partials part;
  uint32_t* hist;      // [ntiles][nb], then offsets
  uint32_t* chunk;     // [kGbChunks][nb]
  uint32_t* start;     // [nb]
  uint4* units;        // {first row, end row, piece of a cut bin, 0}
  uint32_t* n_units;
  int64_t* key;        // the rows by bin
  int64_t* price;
  int32_t* qty;
  relh::PartialCols bin;  // the partials by bin
  __device__ __forceinline__ int64_t tiles() const {
    return more_tiles ? min(ntiles + (int64_t)*more_tiles, part.max_chunks) : ntiles;
  }
};

__device__ __forceinline__ int64_t row_of(const GroupRows& in, int64_t i) { return in.sel ? (int64_t)ld_once(in.sel + i) : i; }

// rank of each active lane's row in its bin, lanes sharing the first active lane's bin served by one atomic (hot keys)
__device__ __forceinline__ uint32_t bin_rank(uint32_t* ctr, uint32_t bin, bool active) {
  const uint64_t act = wave_ballot(active);
  if (act == 0) return 0;
  const int leader = __ffsll((long long)act) - 1;
  const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
  const bool mine = active && bin == b0;
  const uint64_t same = wave_ballot(mine);
  if (__popcll(same) < kWaveCombineMin) return active ? atomicAdd(&ctr[bin], 1u) : 0u;
  uint32_t base = 0, rank = 0;
  if ((int)lane_id() == leader) base = atomicAdd(&ctr[b0], (uint32_t)__popcll(same));
  if (active && !mine) rank = atomicAdd(&ctr[bin], 1u);
  base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
  return mine ? base + mask_rank(same) : rank;
}

__global__ __launch_bounds__(kGbBlock) void k_gb_hist(GbArgs a) {
  __shared__ uint32_t cnt[kGbMaxBins];
  if (*a.few) return;
  const uint32_t t = threadIdx.x;
  for (uint32_t b = t; b < a.nb; b += kGbBlock) cnt[b] = 0;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x), i0 = tile * kGbTile + t;
  int64_t row[kGbRows], key[kGbRows];
#pragma unroll
  for (int k = 0; k < kGbRows; ++k) row[k] = i0 + k * kGbBlock < a.in.n ? row_of(a.in, i0 + k * kGbBlock) : -1;
#pragma unroll
  for (int k = 0; k < kGbRows; ++k) key[k] = row[k] >= 0 ? ld_once((const long long*)a.in.key + row[k]) : 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kGbRows; ++k) (void)bin_rank(cnt, group_bin(key[k], a.shift), row[k] >= 0);
  __syncthreads();
  for (uint32_t b = t; b < a.nb; b += kGbBlock) a.hist[tile * a.nb + b] = cnt[b];
}

// Workgroup (x, y): the bins 64 x .. 64 x + 63 of chunk y's tiles; a wave takes every fourth tile.
constexpr int kColBins = 64, kColWaves = 4;

__device__ __forceinline__ void chunk_tiles(const GbArgs& a, int64_t* lo, int64_t* hi) {
  const int64_t ntiles = a.tiles(), per = (ntiles + kGbChunks - 1) / kGbChunks;
  *lo = min(ntiles, (int64_t)blockIdx.y * per);
  *hi = min(ntiles, *lo + per);
}

__global__ __launch_bounds__(kColBins * kColWaves) void k_gb_colsum(GbArgs a) {
  __shared__ uint32_t s[kColWaves][kColBins];
  if (*a.few) return;
  const uint32_t b = blockIdx.x * kColBins + threadIdx.x % kColBins, w = threadIdx.x / kColBins;
  int64_t lo, hi;
  chunk_tiles(a, &lo, &hi);
  uint32_t c = 0;
#pragma unroll 4
  for (int64_t i = lo + w; i < hi; i += kColWaves) c += a.hist[i * a.nb + b];
  s[w][threadIdx.x % kColBins] = c;
  __syncthreads();
  if (w == 0) a.chunk[blockIdx.y * a.nb + b] = s[0][threadIdx.x] + s[1][threadIdx.x] + s[2][threadIdx.x] + s[3][threadIdx.x];
}

// Exclusive offsets down each bin's column, in place: a wave takes a quarter of the chunk's tiles.
__global__ __launch_bounds__(kColBins * kColWaves) void k_gb_offsets(GbArgs a) {
  __shared__ uint32_t s[kColWaves][kColBins];
  if (*a.few) return;
  const uint32_t x = threadIdx.x % kColBins, b = blockIdx.x * kColBins + x, w = threadIdx.x / kColBins;
  int64_t lo, hi;
  chunk_tiles(a, &lo, &hi);
  const int64_t per = (hi - lo + kColWaves - 1) / kColWaves;
  const int64_t l = min(hi, lo + (int64_t)w * per), h = min(hi, l + per);
  uint32_t c = 0;
#pragma unroll 4
  for (int64_t i = l; i < h; ++i) c += a.hist[i * a.nb + b];
  s[w][x] = c;
  uint32_t run = 0;
#pragma unroll
  for (int y = 0; y < kGbChunks; ++y) run += y < (int)blockIdx.y ? a.chunk[y * a.nb + b] : 0u;
  __syncthreads();
  for (uint32_t v = 0; v < w; ++v) run += s[v][x];
  constexpr int kAhead = 8;
  for (int64_t i = l; i < h; i += kAhead) {
    uint32_t v[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) v[k] = i + k < h ? a.hist[(i + k) * a.nb + b] : 0u;
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
      if (i + k < h) {
        a.hist[(i + k) * a.nb + b] = run;
        run += v[k];
      }
  }
}

// One workgroup; two consecutive bins per thread.
__global__ __launch_bounds__(kGbBlock) void k_gb_units(GbArgs a) {
  __shared__ uint32_t scr[kGbBlock / kWave];
  if (*a.few) return;
  constexpr int kPer = kGbMaxBins / kGbBlock;
  uint32_t c[kPer], rows = 0, pieces = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t b = threadIdx.x * kPer + k;
    c[k] = 0;
    if (b < a.nb)
      for (int y = 0; y < kGbChunks; ++y) c[k] += a.chunk[y * a.nb + b];
    rows += c[k];
    pieces += (c[k] + kGbSubRows - 1) / kGbSubRows;
  }
  uint32_t total, n_units;
  uint32_t lo = block_excl_scan<kGbBlock>(rows, scr, &total);
  uint32_t u = block_excl_scan<kGbBlock>(pieces, scr, &n_units);
  if (total > a.max_rows) {  // (partials, and only of a repeated dim key: see k_part_join_eager)
    if (threadIdx.x == 0) {
      *a.n_units = 0;
      set_status(a.status, kDevDupKey);
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t b = threadIdx.x * kPer + k;
    if (b < a.nb) a.start[b] = lo;
    const uint32_t hi = lo + c[k];
    for (uint32_t r = lo; r < hi; r += kGbSubRows) a.units[u++] = make_uint4(r, min(hi, r + kGbSubRows), c[k] > kGbSubRows, 0u);
    lo = hi;
  }
  if (threadIdx.x == 0) *a.n_units = n_units;
}

// One row of the sorted tile: a fact row, or (P) a partial.
template <bool P>
struct GbRow {
  using Key = std::conditional_t<P, int32_t, int64_t>;
  using Qty = std::conditional_t<P, uint64_t, int32_t>;
  static constexpr int kRows = P ? relh::kPartialTile / kGbBlock : kGbRows;
  Key key[kRows * kGbBlock];
  int64_t price[kRows * kGbBlock];
  Qty qty[kRows * kGbBlock];
  uint32_t count[P ? kRows * kGbBlock : 1];
};

template <bool P>
__global__ __launch_bounds__(kGbBlock) void k_gb_scatter(GbArgs a) {
  __shared__ uint32_t cnt[kGbMaxBins];    // rows per bin, then the bin's first LDS row
  __shared__ uint32_t delta[kGbMaxBins];  // output position minus LDS row (mod 2^32)
  __shared__ GbRow<P> lds;
  __shared__ uint32_t scr[kGbBlock / kWave];
  constexpr int kRows = GbRow<P>::kRows;
  if (*a.few) return;
  const int64_t ntiles = P ? a.tiles() : (int64_t)gridDim.x;
  if (blockIdx.x >= ntiles || (P && *a.n_units == 0)) return;
  const uint32_t t = threadIdx.x;
  constexpr int kPer = kGbMaxBins / kGbBlock;
#pragma unroll
  for (int k = 0; k < kPer; ++k) cnt[t + k * kGbBlock] = 0;
  const int64_t tile = xcd_tile(blockIdx.x, (uint32_t)ntiles), i0 = tile * (kRows * kGbBlock) + t;
  int64_t row[kRows], price[kRows];
  typename GbRow<P>::Key key[kRows];
  typename GbRow<P>::Qty qty[kRows];
  uint32_t count[P ? kRows : 1];
  if constexpr (P) {
    const int64_t end = tile * (kRows * kGbBlock) + a.part.fill[tile];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      row[k] = i0 + k * kGbBlock < end ? i0 + k * kGbBlock : -1;
      const int64_t r = row[k] >= 0 ? row[k] : tile * (kRows * kGbBlock);
      key[k] = ld_once(a.part.cols.key + r);
      price[k] = ld_once((const long long*)a.part.cols.price + r);
      qty[k] = (uint64_t)ld_once((const long long*)a.part.cols.qty + r);
      count[k] = (uint32_t)ld_once((const int32_t*)a.part.cols.count + r);
    }
  } else {
#pragma unroll
    for (int k = 0; k < kRows; ++k) row[k] = i0 + k * kGbBlock < a.in.n ? row_of(a.in, i0 + k * kGbBlock) : -1;
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int64_t r = row[k] >= 0 ? row[k] : 0;
      key[k] = ld_once((const long long*)a.in.key + r);
      price[k] = ld_once((const long long*)a.in.price + r);
      qty[k] = ld_once(a.in.qty + r);
    }
  }
  uint32_t at[kPer];  // where this tile's run of the thread's bins starts
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t b = t * kPer + k;
    at[k] = b < a.nb ? a.start[b] + a.hist[tile * a.nb + b] : 0u;
  }
  __syncthreads();
  uint32_t rank[kRows];
#pragma unroll
  for (int k = 0; k < kRows; ++k) rank[k] = bin_rank(cnt, group_bin(key[k], a.shift), row[k] >= 0);
  __syncthreads();
  uint32_t c[kPer], sum = 0, total;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    c[k] = cnt[t * kPer + k];
    sum += c[k];
  }
  uint32_t run = block_excl_scan<kGbBlock>(sum, scr, &total);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    cnt[t * kPer + k] = run;
    delta[t * kPer + k] = at[k] - run;
    run += c[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRows; ++k)
    if (row[k] >= 0) {
      const uint32_t slot = cnt[group_bin(key[k], a.shift)] + rank[k];
      lds.key[slot] = key[k];
      lds.price[slot] = price[k];
      lds.qty[slot] = qty[k];
      if constexpr (P) lds.count[slot] = count[k];
    }
  __syncthreads();
  for (uint32_t j = t; j < total; j += kGbBlock) {
    const typename GbRow<P>::Key kv = lds.key[j];
    const uint32_t pos = delta[group_bin(kv, a.shift)] + j;
    if constexpr (P) {
      a.bin.key[pos] = kv;
      a.bin.price[pos] = (uint64_t)lds.price[j];
      a.bin.qty[pos] = lds.qty[j];
      a.bin.count[pos] = lds.count[j];
    } else {
      a.key[pos] = kv;
      a.price[pos] = lds.price[j];
      a.qty[pos] = lds.qty[j];
    }
  }
}

template <int SLOTS>
struct GbTable {
  int64_t key[SLOTS];
  uint64_t price[SLOTS];
  uint64_t qty[SLOTS];
  uint32_t count[SLOTS];
  __device__ __forceinline__ void clear(int s) {
    key[s] = kGroupEmpty;
    price[s] = 0;
    qty[s] = 0;
    count[s] = 0;
  }
  __device__ __forceinline__ int find(int64_t k) {
    // (the finalizer of MurmurHash3: one multiplication fewer left consecutive keys of a bin in runs of over 64 slots)
    uint32_t f = group_fold(k);
    f = (f ^ (f >> 16)) * 0x85EBCA6Bu;
    f = (f ^ (f >> 13)) * 0xC2B2AE35u;
    uint32_t h = f >> (32 - __builtin_ctz(SLOTS));
    for (int step = 0; step < kGbProbe; ++step) {
      const int64_t cur = key[h];
      if (cur == k) return (int)h;
      if (cur == kGroupEmpty) {
        const int64_t old = (int64_t)atomicCAS((unsigned long long*)&key[h], (unsigned long long)kGroupEmpty, (unsigned long long)k);
        if (old == kGroupEmpty || old == k) return (int)h;
      }
      h = (h + 1) & (SLOTS - 1);
    }
    return -1;
  }
  __device__ __forceinline__ void add(int s, uint64_t sp, uint64_t sq, uint32_t c) {
    atomicAdd((unsigned long long*)&price[s], (unsigned long long)sp);
    atomicAdd((unsigned long long*)&qty[s], (unsigned long long)sq);
    atomicAdd(&count[s], c);
  }
};

// Workgroup b takes units b, b + G, ... A table key is found by its first row,
// so a key is either in the unit's LDS table for all its rows or (64 occupied
// slots after its home one, which stay occupied) in device memory for all.
template <bool P, int SLOTS, int NT>
__global__ __launch_bounds__(NT) void k_gb_agg(GbArgs a, GroupView g, relh::DirectOut o) {
  __shared__ GbTable<SLOTS> tab;
  __shared__ uint32_t scr[NT / kWave];
  __shared__ int64_t s_pos;
  if (*a.few) return;
  const uint32_t t = threadIdx.x;
  constexpr int kPer = SLOTS / NT, kAhead = 2;
#pragma unroll
  for (int k = 0; k < kPer; ++k) tab.clear(t + k * NT);
  const uint32_t n_units = *a.n_units;
  bool device = false;  // this thread sent a row or a group to device memory
  // One step's rows of a thread. The next step's, or the next unit's first, are
  // on their way while a step's go into the table: there is no second workgroup
  // on the CU to fill the wait (20M rows of 2M groups: 172 us without, 159 with 2
  // rows ahead, 163 with 4, 195 with 6). What is left is the table: walks side by
  // side instead of one after the other took 178, so it is its LDS operations.
  typename GbRow<P>::Key nkey[kAhead];
  uint64_t nsp[kAhead];
  typename GbRow<P>::Qty nqty[kAhead];
  uint32_t nct[kAhead];
  auto load = [&](uint32_t r0, uint32_t end) {
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const uint32_t r = min(r0 + k * NT, end - 1);
      if constexpr (P) {
        nkey[k] = a.bin.key[r];
        nsp[k] = a.bin.price[r];
        nqty[k] = a.bin.qty[r];
        nct[k] = a.bin.count[r];
      } else {
        nkey[k] = a.key[r];
        nsp[k] = (uint64_t)a.price[r];
        nqty[k] = a.qty[r];
        nct[k] = 1;
      }
    }
  };
  uint4 next = make_uint4(0, 0, 0, 0);
  if (blockIdx.x < n_units) {
    next = a.units[blockIdx.x];
    load(next.x + t, next.y);
  }
  for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
    const uint4 d = next;
    const bool cut = d.z != 0;
    if (u + gridDim.x < n_units) next = a.units[u + gridDim.x];
    __syncthreads();  // the table is clear
    for (uint32_t r0 = d.x + t; r0 - t < d.y; r0 += NT * kAhead) {
      int64_t key[kAhead];
      uint64_t sp[kAhead], sq[kAhead];
      uint32_t ct[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        key[k] = (int64_t)nkey[k];
        sp[k] = nsp[k];
        sq[k] = (uint64_t)(int64_t)nqty[k];
        ct[k] = nct[k];
      }
      if (r0 - t + NT * kAhead < d.y) load(r0 + NT * kAhead, d.y);
      else if (u + gridDim.x < n_units) load(next.x + t, next.y);
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        bool mine = r0 + k * NT < d.y;
        uint32_t c = ct[k];
        if (cut) {
          // a hot key's rows sit side by side: the lanes that share the first lane's key are summed first
          const uint64_t act = wave_ballot(mine);
          if (act == 0) continue;
          const int first = __ffsll((long long)act) - 1;
          const int64_t k0 = wave_at(key[k], first);
          const bool same = mine && key[k] == k0;
          const uint64_t ball = wave_ballot(same);
          if (__popcll(ball) >= kWaveCombineMin) {
            const uint64_t p = wave_sum_u64(same ? sp[k] : 0), q = wave_sum_u64(same ? sq[k] : 0);
            const uint32_t all = P ? (uint32_t)wave_sum_u64(same ? c : 0u) : (uint32_t)__popcll(ball);
            if ((int)lane_id() == first) {
              sp[k] = p;
              sq[k] = q;
              c = all;
            } else {
              mine = mine && !same;
            }
          }
        }
        if (!mine) continue;
        const int s = key[k] != kGroupEmpty ? tab.find(key[k]) : -1;
        if (s >= 0) {
          tab.add(s, sp[k], sq[k], c);
        } else {
          group_add(g, key[k], sp[k], sq[k], c);
          device = true;
        }
      }
    }
    __syncthreads();
    uint32_t mine = 0, total;
#pragma unroll
    for (int k = 0; k < kPer; ++k) mine += tab.count[t + k * NT] != 0;
    uint32_t pos = block_excl_scan<NT>(mine, scr, &total);
    if (!cut) {
      if (t == 0) s_pos = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)o.n_direct, (unsigned long long)total);
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int s = (int)t + k * NT;
      if (tab.count[s] == 0) continue;
      if (cut) {
        group_add(g, tab.key[s], tab.price[s], tab.qty[s], tab.count[s]);
        device = true;
      } else {
        const int64_t at = s_pos + pos++;
        if (at < o.cap) {
          o.key[at] = tab.key[s];
          o.sum_price[at] = (int64_t)tab.price[s];
          o.sum_qty[at] = (int64_t)tab.qty[s];
          o.count[at] = (int64_t)tab.count[s];
        } else {
          set_status(g.status, kDevOverflow);
        }
      }
      tab.clear(s);
    }
  }
  if (device) *o.touched = 1u;
}

// First kernel of a group-by: clears the call's words and, when asked, decides
// from a sample whether there are few groups: a key per thread, spread over the
// input, goes into an LDS table, and at most kFewGroups distinct ones among
// them mean that LDS tables over the unpartitioned rows serve almost every row.
// (The decision is one of speed; either way counts every row.)
constexpr int kSampleSlots = 2 * kGbBlock;
constexpr uint32_t kFewGroups = 320;
__global__ __launch_bounds__(kGbBlock) void k_gb_begin(GroupRows in, int32_t mode, uint32_t* __restrict__ few,
                                                       uint64_t* __restrict__ words, int32_t n_words,
                                                       uint64_t* __restrict__ state, int64_t n_state) {
  __shared__ int64_t tab[kSampleSlots];
  __shared__ uint32_t scr[kGbBlock / kWave];
  const uint32_t t = threadIdx.x;
  const int64_t id = (int64_t)blockIdx.x * kGbBlock + t;
  if (id < n_words) words[id] = 0;
  for (int64_t i = id; i < n_state; i += (int64_t)gridDim.x * kGbBlock) state[i] = 0;
  if (blockIdx.x != 0) return;
  if (mode != relh::GB_SAMPLE) {
    if (t == 0) *few = mode == relh::GB_FEW;
    return;
  }
  tab[t] = kGroupEmpty;
  tab[t + kGbBlock] = kGroupEmpty;
  const int64_t i = (int64_t)(((unsigned __int128)t * (uint64_t)in.n) / kGbBlock);
  const int64_t key = in.key[in.sel ? (int64_t)in.sel[i] : i];
  __syncthreads();
  bool first = false;  // the thread brought a new key (one that finds no slot counts as new)
  if (key != kGroupEmpty) {
    uint32_t h = hash64(key, 32 - __builtin_ctz(kSampleSlots));
    first = true;
    for (int step = 0; step < 32; ++step) {
      const int64_t old = (int64_t)atomicCAS((unsigned long long*)&tab[h], (unsigned long long)kGroupEmpty, (unsigned long long)key);
      if (old == kGroupEmpty) break;
      if (old == key) {
        first = false;
        break;
      }
      h = (h + 1) & (kSampleSlots - 1);
    }
  }
  uint32_t distinct;
  (void)block_excl_scan<kGbBlock>(first, scr, &distinct);
  if (t == 0) *few = distinct <= kFewGroups;
}

}  // namespace

namespace relh {

rel_status groupby_begin(rel_ctx* ctx, const GroupRows& in, int mode, uint32_t* few, uint64_t* words, int32_t n_words,
                         uint64_t* state, int64_t n_state) {
  hipLaunchKernelGGL(k_gb_begin, dim3(grid_for(ctx, n_state, kGbBlock * 8, 1)), dim3(kGbBlock), 0, ctx->stream, in, (int32_t)mode,
                     few, words, n_words, state, n_state);
  REL_LAUNCH_CHECK(ctx, "groupby_begin");
  return REL_OK;
}

// Memory of a partitioned group-by of n rows and about `expected` groups.
//
// Bins: a unit's groups should take at most half of the larger LDS table
// (4096 slots, one workgroup per CU), or of the smaller one (2048 slots, two)
// while 64 bins and more allow it. More bins cost the scatter its runs.
static rel_status take_rows(rel_ctx* ctx, int64_t rows, int64_t expected, GbArgs* out) {
  uint32_t bits = 6;
  while (bits < 11 && (expected >> bits) > 2048) ++bits;
  GbArgs a{};
  a.nb = 1u << bits;
  a.shift = 32 - bits;
  a.ntiles = (rows + kGbTile - 1) / kGbTile;
  const size_t n = (size_t)rows, max_units = a.nb + n / kGbSubRows + 1;
  const size_t hist = (size_t)a.ntiles * a.nb * 4, chunk = (size_t)kGbChunks * a.nb * 4;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  void* mem;
  rel_status s = scratch(ctx, SCR_GROUPBY, 2 * up(n * 8) + up(n * 4) + up(hist) + up(chunk) + up(a.nb * 4) + up(max_units * 16) + 256, &mem);
  if (s != REL_OK) return s;
  char* p = (char*)mem;
  auto take = [&](size_t bytes) {
    char* q = p;
    p += up(bytes);
    return q;
  };
  a.key = (int64_t*)take(n * 8);
  a.price = (int64_t*)take(n * 8);
  a.qty = (int32_t*)take(n * 4);
  a.hist = (uint32_t*)take(hist);
  a.chunk = (uint32_t*)take(chunk);
  a.start = (uint32_t*)take(a.nb * 4);
  a.units = (uint4*)take(max_units * 16);
  a.n_units = (uint32_t*)take(4);
  *out = a;
  return REL_OK;
}

rel_status groupby_memory(rel_ctx* ctx, int64_t rows, int64_t expected) {
  GbArgs a;
  return take_rows(ctx, rows, expected, &a);
}

rel_status groupby_partitioned(rel_ctx* ctx, const GroupRows& in, int64_t expected, const uint32_t* few,
                               const rel::GroupView& g, const DirectOut& o) {
  GbArgs a;
  rel_status s = take_rows(ctx, in.n, expected, &a);
  if (s != REL_OK) return s;
  a.in = in;
  a.few = few;
  a.max_rows = (uint32_t)in.n;
  a.status = g.status;
  const bool small = (expected >> (32 - a.shift)) <= 1024;
  KernelTimer kt(ctx, "groupby");
  const dim3 tiles((unsigned)a.ntiles), cols(a.nb / kColBins, kGbChunks);
  hipLaunchKernelGGL(k_gb_hist, tiles, dim3(kGbBlock), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_colsum, cols, dim3(kColBins * kColWaves), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_offsets, cols, dim3(kColBins * kColWaves), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_units, dim3(1), dim3(kGbBlock), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_scatter<false>, tiles, dim3(kGbBlock), 0, ctx->stream, a);
  if (small)
    hipLaunchKernelGGL((k_gb_agg<false, 2048, 512>), dim3(2 * ctx->num_cus), dim3(512), 0, ctx->stream, a, g, o);
  else
    hipLaunchKernelGGL((k_gb_agg<false, 4096, 1024>), dim3(ctx->num_cus), dim3(1024), 0, ctx->stream, a, g, o);
  REL_LAUNCH_CHECK(ctx, "groupby");
  return REL_OK;
}

rel_status partials_take(rel_ctx* ctx, int64_t max_rows, unsigned workgroups, int64_t expected, size_t at_least,
                         uint32_t* n_chunks, Partials* p) {
  // Bins: as above by the groups, and so many that a bin's partials make about
  // one unit.
  uint32_t bits = 6;
  while (bits < 11 && ((expected >> bits) > 2048 || (max_rows >> bits) > kGbSubRows / 2)) ++bits;
  p->nb = 1u << bits;
  p->shift = 32 - bits;
  p->max_rows = max_rows;
  p->first_chunks = workgroups;
  p->max_chunks = max_rows / (kPartialTile - kPartialMost) + workgroups;  // (a chunk ends when the next unit's might not fit)
  p->n_chunks = n_chunks;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  auto cols = [&](int id, size_t n, PartialCols* c) {
    void* mem;
    rel_status s = scratch(ctx, id, std::max(at_least, 2 * up(n * 8) + 2 * up(n * 4)), &mem);
    if (s != REL_OK) return s;
    char* q = (char*)mem;
    c->price = (uint64_t*)q;
    c->qty = (uint64_t*)(q + up(n * 8));
    c->key = (int32_t*)(q + 2 * up(n * 8));
    c->count = (uint32_t*)(q + 2 * up(n * 8) + up(n * 4));
    return s;
  };
  rel_status s = cols(SCR_PART_A, (size_t)p->max_chunks * kPartialTile, &p->cols);
  if (s == REL_OK) s = cols(SCR_PART_B, (size_t)max_rows, &p->binned);
  const size_t fill = up((size_t)p->max_chunks * 4), hist = up((size_t)p->max_chunks * p->nb * 4);
  const size_t chunk = up((size_t)kGbChunks * p->nb * 4), max_units = p->nb + (size_t)max_rows / kGbSubRows + 1;
  void* mem = nullptr;
  if (s == REL_OK) s = scratch(ctx, SCR_GROUPBY, fill + hist + chunk + up(p->nb * 4) + up(max_units * 16) + 256, &mem);
  char* q = (char*)mem;
  p->fill = (uint32_t*)q;
  p->hist = (uint32_t*)(q + fill);
  p->work = q + fill + hist;
  return s;
}

rel_status partials_reduce(rel_ctx* ctx, const Partials& p, int64_t expected, const uint32_t* zero, const rel::GroupView& g,
                           const DirectOut& o) {
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  GbArgs a{};
  a.few = zero;
  a.max_rows = (uint32_t)p.max_rows;
  a.status = g.status;
  a.nb = p.nb;
  a.shift = p.shift;
  a.ntiles = p.first_chunks;
  a.more_tiles = p.n_chunks;
  a.part = p;
  a.hist = p.hist;
  char* q = p.work;
  a.chunk = (uint32_t*)q;
  q += up((size_t)kGbChunks * p.nb * 4);
  a.start = (uint32_t*)q;
  q += up(p.nb * 4);
  a.units = (uint4*)q;
  q += up((p.nb + (size_t)p.max_rows / kGbSubRows + 1) * 16);
  a.n_units = (uint32_t*)q;
  a.bin = p.binned;
  KernelTimer kt(ctx, "partials");
  const dim3 cols(a.nb / kColBins, kGbChunks);
  hipLaunchKernelGGL(k_gb_colsum, cols, dim3(kColBins * kColWaves), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_offsets, cols, dim3(kColBins * kColWaves), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_units, dim3(1), dim3(kGbBlock), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_scatter<true>, dim3((unsigned)p.max_chunks), dim3(kGbBlock), 0, ctx->stream, a);
  if ((expected >> (32 - p.shift)) <= 1024)
    hipLaunchKernelGGL((k_gb_agg<true, 2048, 512>), dim3(2 * ctx->num_cus), dim3(512), 0, ctx->stream, a, g, o);
  else
    hipLaunchKernelGGL((k_gb_agg<true, 4096, 1024>), dim3(ctx->num_cus), dim3(1024), 0, ctx->stream, a, g, o);
  REL_LAUNCH_CHECK(ctx, "partials");
  return REL_OK;
}

}  // namespace relh
