// Stand-alone group-by over many groups: the rows are partitioned by a hash of
// their key, so that a partition's groups fit a workgroup's LDS.
//
// Updating a table in device memory costs three or four atomics per row, and
// those run at about 27 G/s for the whole chip: 20M rows into 2M groups took
// 2.7 ms. Partitioning reads and writes every row once more, but in runs, and
// then all updates are LDS operations: 0.43 ms (6M rows of 15 groups: 147 -> 41 us).
//
//   k_gb_hist     rows per (tile, bin), one tile per workgroup
//   k_gb_colsum   those summed over chunks of tiles, per bin
//   k_gb_offsets  each tile's place in every bin, relative to the bin's start
//   k_gb_units    bin starts; work units (a bin, or a piece of a large one)
//   k_gb_scatter  a tile's rows sorted by bin in LDS and written as runs
//   k_gb_agg      per unit an LDS table; its groups go straight to the output
//
// A key that finds no room in a unit's LDS table, and every group of a bin that
// was cut into pieces (hot keys), goes to the group table in device memory,
// which the caller's finalize kernel appends to the output.
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

// The key folded to 32 bits; the bin and the LDS slot are taken from different products of it.
__device__ __forceinline__ uint32_t fold(int64_t key) {
  return (uint32_t)key ^ ((uint32_t)((uint64_t)key >> 32) * 0x85EBCA6Bu);
}
__device__ __forceinline__ uint32_t bin_of(int64_t key, uint32_t shift) { return (fold(key) * 2654435769u) >> shift; }

// Every kernel returns at once when the sample found few groups (`few`, see k_gb_begin).
struct GbArgs {
  GroupRows in;
  const uint32_t* few;
  uint32_t nb, shift;  // bins, 32 - log2(bins)
  int64_t ntiles;
  uint32_t* hist;      // [ntiles][nb], then offsets
  uint32_t* chunk;     // [kGbChunks][nb]
  uint32_t* start;     // [nb]
  uint4* units;        // {first row, end row, piece of a cut bin, 0}
  uint32_t* n_units;
  int64_t* key;        // the rows by bin
  int64_t* price;
  int32_t* qty;
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
  for (int k = 0; k < kGbRows; ++k) (void)bin_rank(cnt, bin_of(key[k], a.shift), row[k] >= 0);
  __syncthreads();
  for (uint32_t b = t; b < a.nb; b += kGbBlock) a.hist[tile * a.nb + b] = cnt[b];
}

// Workgroup (x, y): the bins 64 x .. 64 x + 63 of chunk y's tiles; a wave takes every fourth tile.
constexpr int kColBins = 64, kColWaves = 4;

__device__ __forceinline__ void chunk_tiles(const GbArgs& a, int64_t* lo, int64_t* hi) {
  const int64_t per = (a.ntiles + kGbChunks - 1) / kGbChunks;
  *lo = min(a.ntiles, (int64_t)blockIdx.y * per);
  *hi = min(a.ntiles, *lo + per);
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

__global__ __launch_bounds__(kGbBlock) void k_gb_scatter(GbArgs a) {
  __shared__ uint32_t cnt[kGbMaxBins];    // rows per bin, then the bin's first LDS row
  __shared__ uint32_t delta[kGbMaxBins];  // output position minus LDS row (mod 2^32)
  __shared__ int64_t s_key[kGbTile];
  __shared__ int64_t s_price[kGbTile];
  __shared__ int32_t s_qty[kGbTile];
  __shared__ uint32_t scr[kGbBlock / kWave];
  if (*a.few) return;
  const uint32_t t = threadIdx.x;
  constexpr int kPer = kGbMaxBins / kGbBlock;
#pragma unroll
  for (int k = 0; k < kPer; ++k) cnt[t + k * kGbBlock] = 0;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x), i0 = tile * kGbTile + t;
  int64_t row[kGbRows], key[kGbRows], price[kGbRows];
  int32_t qty[kGbRows];
#pragma unroll
  for (int k = 0; k < kGbRows; ++k) row[k] = i0 + k * kGbBlock < a.in.n ? row_of(a.in, i0 + k * kGbBlock) : -1;
#pragma unroll
  for (int k = 0; k < kGbRows; ++k) {
    const int64_t r = row[k] >= 0 ? row[k] : 0;
    key[k] = ld_once((const long long*)a.in.key + r);
    price[k] = ld_once((const long long*)a.in.price + r);
    qty[k] = ld_once(a.in.qty + r);
  }
  uint32_t at[kPer];  // where this tile's run of the thread's bins starts
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t b = t * kPer + k;
    at[k] = b < a.nb ? a.start[b] + a.hist[tile * a.nb + b] : 0u;
  }
  __syncthreads();
  uint32_t rank[kGbRows];
#pragma unroll
  for (int k = 0; k < kGbRows; ++k) rank[k] = bin_rank(cnt, bin_of(key[k], a.shift), row[k] >= 0);
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
  for (int k = 0; k < kGbRows; ++k)
    if (row[k] >= 0) {
      const uint32_t slot = cnt[bin_of(key[k], a.shift)] + rank[k];
      s_key[slot] = key[k];
      s_price[slot] = price[k];
      s_qty[slot] = qty[k];
    }
  __syncthreads();
  for (uint32_t j = t; j < total; j += kGbBlock) {
    const int64_t kv = s_key[j];
    const uint32_t pos = delta[bin_of(kv, a.shift)] + j;
    a.key[pos] = kv;
    a.price[pos] = s_price[j];
    a.qty[pos] = s_qty[j];
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
    uint32_t f = fold(k);
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
template <int SLOTS, int NT>
__global__ __launch_bounds__(NT) void k_gb_agg(GbArgs a, GroupView g, relh::DirectOut o) {
  __shared__ GbTable<SLOTS> tab;
  __shared__ uint32_t scr[NT / kWave];
  __shared__ int64_t s_pos;
  if (*a.few) return;
  const uint32_t t = threadIdx.x;
  constexpr int kPer = SLOTS / NT, kAhead = 4;
#pragma unroll
  for (int k = 0; k < kPer; ++k) tab.clear(t + k * NT);
  const uint32_t n_units = *a.n_units;
  bool device = false;  // this thread sent a row or a group to device memory
  for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
    const uint4 d = a.units[u];
    const bool cut = d.z != 0;
    __syncthreads();  // the table is clear
    for (uint32_t r0 = d.x + t; r0 - t < d.y; r0 += NT * kAhead) {
      int64_t key[kAhead];
      uint64_t sp[kAhead], sq[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const uint32_t r = min(r0 + k * NT, d.y - 1);
        key[k] = a.key[r];
        sp[k] = (uint64_t)a.price[r];
        sq[k] = (uint64_t)(int64_t)a.qty[r];
      }
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        bool mine = r0 + k * NT < d.y;
        uint32_t c = 1;
        if (cut) {
          // a hot key's rows sit side by side: the lanes that share the first lane's key are summed first
          const uint64_t act = wave_ballot(mine);
          if (act == 0) continue;
          const int first = __ffsll((long long)act) - 1;
          const int64_t k0 = __shfl(key[k], first, kWave);
          const bool same = mine && key[k] == k0;
          const uint64_t ball = wave_ballot(same);
          if (__popcll(ball) >= kWaveCombineMin) {
            const uint64_t p = wave_sum_u64(same ? sp[k] : 0), q = wave_sum_u64(same ? sq[k] : 0);
            if ((int)lane_id() == first) {
              sp[k] = p;
              sq[k] = q;
              c = (uint32_t)__popcll(ball);
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

rel_status groupby_partitioned(rel_ctx* ctx, const GroupRows& in, int64_t expected, const uint32_t* few,
                               const rel::GroupView& g, const DirectOut& o) {
  // Bins: a unit's groups should take at most half of the larger LDS table
  // (4096 slots, one workgroup per CU), or of the smaller one (2048 slots, two)
  // while 64 bins and more allow it. More bins cost the scatter its runs.
  uint32_t bits = 6;
  while (bits < 11 && (expected >> bits) > 2048) ++bits;
  const bool small = (expected >> bits) <= 1024;
  GbArgs a{};
  a.in = in;
  a.few = few;
  a.nb = 1u << bits;
  a.shift = 32 - bits;
  a.ntiles = (in.n + kGbTile - 1) / kGbTile;
  const size_t n = (size_t)in.n, max_units = a.nb + n / kGbSubRows + 1;
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
  KernelTimer kt(ctx, "groupby");
  const dim3 tiles((unsigned)a.ntiles), cols(a.nb / kColBins, kGbChunks);
  hipLaunchKernelGGL(k_gb_hist, tiles, dim3(kGbBlock), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_colsum, cols, dim3(kColBins * kColWaves), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_offsets, cols, dim3(kColBins * kColWaves), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_units, dim3(1), dim3(kGbBlock), 0, ctx->stream, a);
  hipLaunchKernelGGL(k_gb_scatter, tiles, dim3(kGbBlock), 0, ctx->stream, a);
  if (small)
    hipLaunchKernelGGL((k_gb_agg<2048, 512>), dim3(2 * ctx->num_cus), dim3(512), 0, ctx->stream, a, g, o);
  else
    hipLaunchKernelGGL((k_gb_agg<4096, 1024>), dim3(ctx->num_cus), dim3(1024), 0, ctx->stream, a, g, o);
  REL_LAUNCH_CHECK(ctx, "groupby");
  return REL_OK;
}

}  // namespace relh
