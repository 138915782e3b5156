// Selection vectors in two passes: the rows' outcomes as one bit each, then
// the bits as ascending row ids.
//
// The first pass (one kernel per kind of predicate) reads the columns once
// and writes a bit per row and a count per tile. The second (k_select_expand)
// reads the bits only: every workgroup sums the counts of the tiles before
// its own, so nothing is zeroed beforehand, no workgroup waits on another and
// no ticket or look-back state exists. The bits are 1/32 of an int32 column,
// so the second pass costs little besides the output it writes.
//
// A wave takes 2048 consecutive rows at a time, as 8 chunks of 256: lane l
// holds rows 4 l .. 4 l + 3 of each chunk, so every load of a wave covers
// consecutive 16-byte words (4-byte elements). Its eight 4-bit outcomes,
// chunk c in bits 4 c .. 4 c + 3, are transposed between the eight lanes of a
// group, after which each lane holds 32 consecutive rows' bits.
#pragma once

#include "rel_device.h"
#include "rel_host.h"

namespace rel {

constexpr int kSelBlock = 256;
constexpr int kSelWaveRows = 2048;                          // rows of a wave's step
constexpr int kSelChunk = 256;                              // rows of one chunk (4 per lane)
constexpr int kSelStep = kSelBlock / kWave * kSelWaveRows;  // rows of a workgroup's step
constexpr int kSelSub = kSelBlock * 64;                     // rows of a workgroup's step in the second pass
constexpr int kSelSparse = kSelSub / 4;                     // ids of one such step that are staged in LDS
// A tile is a whole number of second-pass steps, as few as keep the number of
// tiles (and so the counts that each workgroup adds up) at most this.
constexpr int64_t kSelMaxTiles = 4096;
static_assert(kSelSub % kSelStep == 0, "a tile is whole steps of both passes");

// 8 x 8 transpose of 4-bit fields between the eight lanes of a group: field j
// of lane i becomes field i of lane j.
__device__ __forceinline__ uint32_t transpose_nibbles(uint32_t x) {
  const uint32_t lane = lane_id();
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) {
    const uint32_t keep = d == 1 ? 0x0F0F0F0Fu : d == 2 ? 0x00FF00FFu : 0x0000FFFFu;
    const uint32_t y = (uint32_t)__shfl_xor((int)x, d, kWave);
    x = (lane & d) ? (x & ~keep) | ((y & ~keep) >> (4 * d)) : (x & keep) | ((y & keep) << (4 * d));
  }
  return x;
}

// One lane's outcomes of a wave's step starting at row `base` into the bit
// array (row r is bit r % 32 of word r / 32); returns how many of the word's
// rows pass.
__device__ __forceinline__ uint32_t store_bits(uint32_t* __restrict__ bits, int64_t base, uint32_t nibbles) {
  const uint32_t word = transpose_nibbles(nibbles);
  const uint32_t lane = lane_id();
  bits[base / 32 + (lane & 7u) * 8 + (lane >> 3)] = word;
  return (uint32_t)__popc(word);
}

// The end of the first pass: the tile's count, one 32-bit sum per workgroup.
__device__ __forceinline__ void store_tile_count(uint32_t* __restrict__ counts, uint32_t c) {
  __shared__ uint32_t s_cnt[kSelBlock / kWave];
  c = wave_sum(c);
  if (lane_id() == 0) s_cnt[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < kSelBlock / kWave; ++w) t += s_cnt[w];
    counts[blockIdx.x] = t;
  }
}

}  // namespace rel

namespace relh {

// Sizes and scratch of one selection over n rows.
struct SelectPlan {
  int64_t n = 0;
  int64_t tile_rows = 0;  // a multiple of rel::kSelSub
  int64_t ntiles = 0;     // workgroups of either pass
  uint32_t* bits = nullptr;
  uint32_t* counts = nullptr;
};
// n > 0. The bit array has whole tiles; the first pass writes all of it.
rel_status select_plan(rel_ctx* ctx, int64_t n, SelectPlan* out);
// The second pass: the ascending ids of the rows whose bits are set, and their number.
rel_status select_expand(rel_ctx* ctx, const SelectPlan& p, int32_t* out_idx, int64_t* d_out_count);

}  // namespace relh
