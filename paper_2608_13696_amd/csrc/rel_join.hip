// Hash join: build (insert_if_n analogue) and probe (count + retrieve
// analogue, fused into one pass because a PK-FK probe emits at most one pair
// per probe row, so no counting pass is needed to size the output).
#include <algorithm>
#include <mutex>
#include <utility>

#include "rel_device.h"
#include "rel_host.h"
#include "rel_ops.h"

namespace {

using namespace rel;
using relh::PAY_I32;
using relh::PAY_I8;
using relh::PAY_ROW_ID;

// Insert (pk[j], payload) with one 64-bit CAS per attempted slot. Consecutive
// threads take consecutive rows, so the key and payload reads are coalesced
// and each thread keeps its CAS independent of the others. Also zeroes the
// caller's spans of words.
__device__ __forceinline__ void zero_spans(const relh::ZeroSpans& z) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
#pragma unroll
  for (int k = 0; k < 2; ++k)
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < z.n[k]; i += stride) z.p[k][i] = 0;
}

template <int PK>
__global__ __launch_bounds__(256) void k_join_build(const int32_t* __restrict__ pk, const void* __restrict__ payload,
                                                    int64_t m, uint64_t* __restrict__ slots, uint32_t mask,
                                                    uint32_t shift, uint32_t* __restrict__ status, relh::ZeroSpans z) {
  zero_spans(z);
  int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; j < m; j += stride) {
    const int32_t key = pk[j];
    const int32_t pl = PK == PAY_ROW_ID ? (int32_t)j
                       : PK == PAY_I32  ? ((const int32_t*)payload)[j]
                                        : (int32_t)((const int8_t*)payload)[j];
    join_insert(slots, mask, shift, key, pl, status);
  }
}

// ---- join index (dense array or hash table) ----------------------------------------------------------------------------

// Minimum and maximum of the build keys, order-encoded so that both are
// maxima over unsigned words that start at 0 (see JoinIndex::mm). Few, large
// workgroups with two 16-byte loads in flight per thread; each writes its pair
// to part[2b], part[2b + 1], and a kernel that follows combines them (the
// clearing kernel of a stand-alone table, the build where the table was left
// empty): no atomics, and no word to zero first.
constexpr int kIdxBlock = 256;
constexpr int kMinMaxBlock = 512;
constexpr int kMinMaxGrid = relh::kKeyMinMaxParts;
__device__ __forceinline__ void minmax_add(int32_t k, uint32_t& lo, uint32_t& hi) {
  const uint32_t o = (uint32_t)k ^ 0x80000000u;
  lo = max(lo, ~o);
  hi = max(hi, o);
}

__global__ __launch_bounds__(kMinMaxBlock) void k_key_minmax(const int32_t* __restrict__ pk, int64_t m, uint32_t* part,
                                                             relh::ZeroSpans z) {
  zero_spans(z);
  __shared__ uint32_t s_lo[kMinMaxBlock / kWave], s_hi[kMinMaxBlock / kWave];
  uint32_t lo = 0, hi = 0;  // max of ~(key ^ 2^31), max of (key ^ 2^31)
  const int64_t nq = m / 4;  // whole 16-byte quads (pk is 16-byte aligned)
  const int4* q = reinterpret_cast<const int4*>(pk);
  constexpr int kQ = 4;  // quads in flight per thread
  const int64_t stride = (int64_t)gridDim.x * kMinMaxBlock * kQ;
  for (int64_t i = blockIdx.x * (int64_t)kMinMaxBlock * kQ + threadIdx.x; i < nq; i += stride) {
    int4 v[kQ];
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
      const int64_t j = i + (int64_t)k * kMinMaxBlock;
      v[k] = q[j < nq ? j : i];
    }
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
      minmax_add(v[k].x, lo, hi); minmax_add(v[k].y, lo, hi); minmax_add(v[k].z, lo, hi); minmax_add(v[k].w, lo, hi);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < (m & 3)) minmax_add(pk[nq * 4 + threadIdx.x], lo, hi);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    lo = max(lo, (uint32_t)__shfl_xor((int)lo, d, kWave));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, kWave));
  }
  if (lane_id() == 0) {
    s_lo[threadIdx.x / kWave] = lo;
    s_hi[threadIdx.x / kWave] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kMinMaxBlock / kWave; ++w) {
      lo = max(lo, s_lo[w]);
      hi = max(hi, s_hi[w]);
    }
    part[2 * blockIdx.x] = lo;
    part[2 * blockIdx.x + 1] = hi;
  }
}

// The keys' range from the min/max pairs of k_key_minmax, which every workgroup
// combines for itself; workgroup 0 also stores it in x.mm for the kernels that
// follow. Synchronises the workgroup.
__device__ __forceinline__ DenseRange combine_minmax(const JoinIndex& x, const uint32_t* __restrict__ part, int32_t nparts) {
  __shared__ uint32_t s_mm[2];
  if (threadIdx.x < kWave) {
    uint32_t lo = 0, hi = 0;
    for (int i = threadIdx.x; i < nparts; i += kWave) {
      lo = max(lo, part[2 * i]);
      hi = max(hi, part[2 * i + 1]);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      lo = max(lo, (uint32_t)__shfl_xor((int)lo, d, kWave));
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, kWave));
    }
    if (threadIdx.x == 0) {
      s_mm[0] = lo;
      s_mm[1] = hi;
      if (blockIdx.x == 0) {
        uint32_t* mm = const_cast<uint32_t*>(x.mm);
        mm[0] = lo;
        mm[1] = hi;
      }
    }
  }
  __syncthreads();
  return dense_range_of(x, s_mm[0], s_mm[1]);
}

// Clears whichever structure the keys' range selects: the 16-byte words that
// hold the dense entries in use, or the whole hash table; and zeroes the
// caller's spans of 64-bit words. (Stand-alone tables; the fused path's index
// is emptied by the kernel after the one that probes it.)
__global__ __launch_bounds__(kIdxBlock) void k_index_clear(JoinIndex x, const uint32_t* __restrict__ part, int32_t nparts,
                                                           relh::ZeroSpans z) {
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  const DenseRange r = combine_minmax(x, part, nparts);
  const int64_t stride = (int64_t)gridDim.x * kIdxBlock;
  int64_t i = blockIdx.x * (int64_t)kIdxBlock + threadIdx.x;
  zero_spans(z);
  if (r.dense) {
    const int64_t words = dense_words(x, r);
    for (; i < words; i += stride) reinterpret_cast<v4u*>(x.dense)[i] = v4u{0u, 0u, 0u, 0u};
  } else {
    uint64_t* slots = const_cast<uint64_t*>(x.hash.slots);
    for (; i < (int64_t)x.hash.mask + 2; i += stride) slots[i] = kJoinEmpty;
  }
}

// Dense: plain stores (a repeated key is found by counting the entries, which
// the probing kernel does). A thread loads kBuildQuads 16-byte quads of keys
// (and their payloads) before it stores any entry, so its random stores do
// not wait on one load at a time. (Cutting the key range into one slice per
// XCD, so that each L2 takes the stores of its own slice only, measured
// slower on 1.5M keys: 26 us against 17, each XCD then reading every key.)
// Hash: one 64-bit CAS per attempted slot.
constexpr int kBuildQuads = 4;

template <int PK>
__global__ __launch_bounds__(kIdxBlock) void k_index_build(const int32_t* __restrict__ pk, int64_t m, JoinIndex x,
                                                           const uint32_t* __restrict__ part, int32_t nparts,
                                                           uint32_t* __restrict__ status) {
  const DenseRange r = nparts > 0 ? combine_minmax(x, part, nparts) : dense_range(x);
  if (r.dense) {
    const int64_t nq = (m + 3) / 4;
    const int4* q = reinterpret_cast<const int4*>(pk);
    const int64_t step = (int64_t)gridDim.x * kIdxBlock;
    for (int64_t i0 = blockIdx.x * (int64_t)kIdxBlock + threadIdx.x; i0 < nq; i0 += step * kBuildQuads) {
      int32_t key[kBuildQuads * 4];
#pragma unroll
      for (int u = 0; u < kBuildQuads; ++u) {
        const int64_t i = i0 + u * step;
        if (4 * i + 4 <= m) {
          const int4 v = q[i];
          key[4 * u] = v.x; key[4 * u + 1] = v.y; key[4 * u + 2] = v.z; key[4 * u + 3] = v.w;
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) key[4 * u + c] = 4 * i + c < m ? pk[4 * i + c] : 0;
        }
      }
      uint32_t e[kBuildQuads * 4];
#pragma unroll
      for (int u = 0; u < kBuildQuads; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int64_t j = 4 * (i0 + u * step) + c;
          e[4 * u + c] = j < m ? dense_encode(x, j) : 0u;
        }
#pragma unroll
      for (int u = 0; u < kBuildQuads; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int64_t j = 4 * (i0 + u * step) + c;
          if (j < m) dense_store(x, (int64_t)key[4 * u + c] - r.kmin, e[4 * u + c]);
        }
    }
    return;
  }
  const int64_t stride = (int64_t)gridDim.x * kIdxBlock;
  for (int64_t j = blockIdx.x * (int64_t)kIdxBlock + threadIdx.x; j < m; j += stride) {
    const int32_t key = pk[j];
    const int32_t pl = PK == PAY_ROW_ID ? (int32_t)j
                       : PK == PAY_I32  ? ((const int32_t*)x.payload)[j]
                                        : (int32_t)((const int8_t*)x.payload)[j];
    join_insert(const_cast<uint64_t*>(x.hash.slots), x.hash.mask, x.hash.shift, key, pl, status);
  }
}

// The dense index's duplicate check on its own, for calls whose probing
// kernel does not run (no probe rows): one workgroup counts the entries. A
// no-op for a hash table.
constexpr int kVerifyBlock = 1024;
__global__ __launch_bounds__(kVerifyBlock) void k_index_verify(JoinIndex x, uint32_t* __restrict__ status) {
  __shared__ uint64_t s_red[kVerifyBlock / kWave];
  const DenseRange r = dense_range(x);
  if (!r.dense) return;
  const uint64_t c = block_sum_u64<kVerifyBlock>(dense_count_entries<kVerifyBlock>(x, 0, dense_words(x, r)), s_red);
  if (threadIdx.x == 0 && c != (uint64_t)x.m) set_status(status, kDevDupKey);
}

// The same check by many workgroups, for a stand-alone table, whose build
// must report a repeated key itself: every workgroup adds its entries to
// tail[0], and the last one to arrive (tail[1]) compares the sum with m.
__global__ __launch_bounds__(kVerifyBlock) void k_index_count(JoinIndex x, uint64_t* __restrict__ tail,
                                                              uint32_t* __restrict__ status) {
  __shared__ uint64_t s_red[kVerifyBlock / kWave];
  const DenseRange r = dense_range(x);
  if (!r.dense) return;
  const int64_t words = dense_words(x, r), per = (words + gridDim.x - 1) / gridDim.x;
  const int64_t w0 = (int64_t)blockIdx.x * per;
  const uint64_t c = block_sum_u64<kVerifyBlock>(dense_count_entries<kVerifyBlock>(x, w0, min(words, w0 + per)), s_red);
  if (threadIdx.x != 0) return;
  __hip_atomic_fetch_add(&tail[0], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (__hip_atomic_fetch_add(&tail[1], 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != gridDim.x - 1) return;
  if (__hip_atomic_load(&tail[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (uint64_t)x.m)
    set_status(status, kDevDupKey);
}

// Probe: a wave takes 8 x 64 consecutive probe rows per step, one row of each
// 64 per lane. Every lane issues the first reads of its eight rows (the dense
// entry, or the first hash slot) together (the random table reads are the
// cost, so eight are in flight per lane instead of one), then finishes each
// probe. A wave runs kProbeGroup steps, keeping each row's match in
// registers, and then the workgroup reserves output space for all of them
// with one atomic: the count is one word, and atomics on one cache line
// serialise on this chip at about 12 ns each, so one per step (512 rows)
// bounded the kernel. Matches are compacted with one ballot per row group. Output order is therefore
// unspecified.
// On 28.15M probes into a 15M-key hash table, with one atomic per wave and
// step: 0.78 ms with eight rows per lane, 1.40 ms with four, 5.31 ms with one;
// sixteen spill the ballot masks. 28.15M probes of Zipf(0.8) keys into a dense
// table of 15M keys (60 MB): 0.37 ms with one atomic per workgroup, 0.46 ms
// with one per wave; the table's lines, fetched at 7 TB/s, then bound it (two
// steps or one per reservation, and larger workgroups, measured the same).
constexpr int kProbeBlock = 256;
constexpr int kProbeRows = 8;
constexpr int kProbeGroup = 4;

enum ProbeKind { PROBE_HASH = 0, PROBE_ROW_ID, PROBE_WIDE };

// Output positions for a workgroup's matches, `total` of them in this wave
// (the same on every lane): one atomic per workgroup, then the waves' shares in
// order. Synchronises the workgroup.
template <int NT>
__device__ __forceinline__ int64_t reserve_output(uint32_t total, int64_t* __restrict__ d_count) {
  __shared__ uint32_t s_total[NT / kWave];
  __shared__ int64_t s_off;
  const uint32_t wave = threadIdx.x / kWave;
  __syncthreads();  // (the last reservation has been read)
  if (lane_id() == 0) s_total[wave] = total;
  __syncthreads();
  uint32_t before = 0, sum = 0;
#pragma unroll
  for (uint32_t w = 0; w < NT / kWave; ++w) {
    const uint32_t t = s_total[w];
    before += w < wave ? t : 0u;
    sum += t;
  }
  if (threadIdx.x == 0 && sum != 0)
    s_off = (int64_t)dev_add_ret<unsigned long long>((unsigned long long*)d_count, (unsigned long long)sum);
  __syncthreads();
  return s_off + before;
}

template <int KIND>
__device__ __forceinline__ void probe_rows(const JoinIndex& x, const DenseRange& r, const int32_t* __restrict__ fk,
                                           const int32_t* __restrict__ sel, int64_t n, int32_t* __restrict__ out_fact,
                                           int32_t* __restrict__ out_payload, int64_t* __restrict__ d_count) {
  constexpr int64_t kStep = (int64_t)kWave * kProbeRows;
  const JoinView& t = x.hash;
  constexpr int64_t kBlockRows = kStep * kProbeGroup * (kProbeBlock / kWave);
  const uint32_t lane = lane_id();
  for (int64_t block0 = blockIdx.x * kBlockRows; block0 < n; block0 += gridDim.x * kBlockRows) {
    const int64_t base0 = block0 + (int64_t)(threadIdx.x / kWave) * kStep * kProbeGroup;
    int32_t hrow[kProbeGroup][kProbeRows];  // the matching fact row, or -1
    int32_t hpl[kProbeGroup][kProbeRows];
    uint32_t total = 0;
#pragma unroll
    for (int g = 0; g < kProbeGroup; ++g) {
      const int64_t base = base0 + g * kStep;
      int32_t row[kProbeRows], key[kProbeRows];
      uint64_t first[kProbeRows];
#pragma unroll
      for (int k = 0; k < kProbeRows; ++k) {
        const int64_t i = base + k * kWave + lane;
        row[k] = i < n ? (sel ? ld_once(sel + i) : (int32_t)i) : -1;
      }
#pragma unroll
      for (int k = 0; k < kProbeRows; ++k) key[k] = row[k] >= 0 ? ld_once(fk + row[k]) : 0;
#pragma unroll
      for (int k = 0; k < kProbeRows; ++k) {
        if (KIND == PROBE_HASH) {
          first[k] = row[k] >= 0 ? t.slots[join_first_index(t, key[k])] : kJoinEmpty;
        } else {
          const uint32_t off = (uint32_t)key[k] - (uint32_t)r.kmin;
          const bool in = row[k] >= 0 && (int64_t)off < r.range;
          if (KIND == PROBE_WIDE) first[k] = in ? ((const uint64_t*)x.dense)[off] : 0ull;
          else first[k] = in ? ((const uint32_t*)x.dense)[off] : 0u;
        }
      }
#pragma unroll
      for (int k = 0; k < kProbeRows; ++k) {
        hpl[g][k] = 0;
        bool hit;
        if (KIND == PROBE_HASH) {
          hit = row[k] >= 0 && join_finish(t, key[k], first[k], &hpl[g][k]);
        } else {
          hit = first[k] != 0;
          hpl[g][k] = KIND == PROBE_WIDE ? (int32_t)(uint32_t)first[k] : (int32_t)((uint32_t)first[k] - 1u);
        }
        hrow[g][k] = hit ? row[k] : -1;
        total += (uint32_t)__popcll(wave_ballot(hit));
      }
    }
    int64_t off = reserve_output<kProbeBlock>(total, d_count);
#pragma unroll
    for (int g = 0; g < kProbeGroup; ++g) {
#pragma unroll
      for (int k = 0; k < kProbeRows; ++k) {
        const uint64_t b = wave_ballot(hrow[g][k] >= 0);
        if (hrow[g][k] >= 0) {
          const int64_t o = off + mask_rank(b);
          out_fact[o] = hrow[g][k];
          out_payload[o] = hpl[g][k];
        }
        off += __popcll(b);
      }
    }
  }
}

__global__ __launch_bounds__(kProbeBlock) void k_join_probe(JoinIndex x, const int32_t* __restrict__ fk,
                                                    const int32_t* __restrict__ sel, int64_t n,
                                                    int32_t* __restrict__ out_fact, int32_t* __restrict__ out_payload,
                                                    int64_t* __restrict__ d_count) {
  probe_rows<PROBE_HASH>(x, DenseRange{}, fk, sel, n, out_fact, out_payload, d_count);
}

// A table that may be dense: the keys' range on the device says whether it is.
template <bool WIDE>
__global__ __launch_bounds__(kProbeBlock) void k_join_probe_index(JoinIndex x, const int32_t* __restrict__ fk,
                                                                  const int32_t* __restrict__ sel, int64_t n,
                                                                  int32_t* __restrict__ out_fact,
                                                                  int32_t* __restrict__ out_payload,
                                                                  int64_t* __restrict__ d_count) {
  const DenseRange r = dense_range(x);
  if (r.dense) probe_rows<WIDE ? PROBE_WIDE : PROBE_ROW_ID>(x, r, fk, sel, n, out_fact, out_payload, d_count);
  else probe_rows<PROBE_HASH>(x, r, fk, sel, n, out_fact, out_payload, d_count);
}

}  // namespace

namespace relh {

// The entries of an index that is empty. nparts > 0: the keys' range is still
// to be combined from `part`.
static rel_status index_entries(rel_ctx* ctx, const int32_t* pk, int payload_kind, const rel::JoinIndex& x,
                                const uint32_t* part, int32_t nparts) {
  if (x.m == 0) return REL_OK;
  KernelTimer kt(ctx, "join_build");
  auto* kernel = payload_kind == PAY_I32  ? &k_index_build<PAY_I32>
                 : payload_kind == PAY_I8 ? &k_index_build<PAY_I8>
                                          : &k_index_build<PAY_ROW_ID>;
  hipLaunchKernelGGL(kernel, dim3(grid_for(ctx, x.m, kIdxBlock * 4, 8)), dim3(kIdxBlock), 0, ctx->stream, pk, x.m, x, part,
                     nparts, ctx->d_status);
  REL_LAUNCH_CHECK(ctx, "join index build");
  return REL_OK;
}

static int32_t key_minmax(rel_ctx* ctx, const int32_t* pk, int64_t m, uint32_t* part, const ZeroSpans& zero) {
  int64_t gm = (m + kMinMaxBlock * 16 - 1) / (kMinMaxBlock * 16);
  if (gm > kMinMaxGrid) gm = kMinMaxGrid;
  if (m > 0) {
    KernelTimer kt(ctx, "key_minmax");
    hipLaunchKernelGGL(k_key_minmax, dim3((unsigned)gm), dim3(kMinMaxBlock), 0, ctx->stream, pk, m, part, zero);
  }
  return (int32_t)gm;
}

int32_t key_minmax_partials(rel_ctx* ctx, const int32_t* pk, int64_t m, uint32_t* part) {
  return key_minmax(ctx, pk, m, part, ZeroSpans{});
}

static rel_status hash_entries(rel_ctx* ctx, const int32_t* pk, const void* payload, int payload_kind, int64_t m,
                               const rel::JoinView& v, const ZeroSpans& zero) {
  KernelTimer kt(ctx, "join_build");
  auto* kernel = payload_kind == PAY_I32  ? &k_join_build<PAY_I32>
                 : payload_kind == PAY_I8 ? &k_join_build<PAY_I8>
                                          : &k_join_build<PAY_ROW_ID>;
  hipLaunchKernelGGL(kernel, dim3(grid_for(ctx, m, 256, 8)), dim3(256), 0, ctx->stream, pk, payload, m,
                     const_cast<uint64_t*>(v.slots), v.mask, v.shift, ctx->d_status, zero);
  REL_LAUNCH_CHECK(ctx, "join_build");
  return REL_OK;
}

// Up to this many keys, and for at most so many probe rows, the fused path's
// index is a hash table whatever the keys' range: its 2 MB stay in L2, and one
// launch builds it, where a dense array takes two (the keys' range first) of about
// 3 us each. A probe of it costs more: it reads 8 bytes of a table of up to 2 MB
// and walks on where keys collide or match nothing, against 2 or 4 bytes of at
// most 128 or 256 KB. Measured, (prio, flag) of 16K keys, hash table and dense
// array in us: 60K rows 17.4 and 21.5, 1M 20.7 and 26.3, 6M 45.5 and 51.4, 30M 208
// and 171; a quarter of the rows with a match: 1M 23.2 and 25.9, 6M 56.4 and 48.4,
// 30M 234 and 154.
constexpr int64_t kHashMaxKeys = 1 << 16, kHashMaxRows = 1 << 21;

rel_status join_index_build(rel_ctx* ctx, const int32_t* pk, const void* payload, int payload_kind, int64_t m,
                            int64_t probes, uint32_t* mm, const ZeroSpans& zero, rel::JoinIndex* out) {
  const uint32_t jl = join_log2cap(m, nullptr);
  const size_t hash_bytes = ((size_t)8 << jl) + 8;
  rel_status s;
  // both structures are empty between calls (join_index_wipe)
  auto empty = [&](int id, size_t bytes, uint64_t word, void** p) {
    return scratch_empty(ctx, id, bytes, p, [&](void* q) { return fill_u64(ctx, q, (bytes + 7) / 8, word); });
  };
  void *jt, *dt = nullptr, *part = nullptr;
  if ((s = empty(SCR_JOIN_TABLE, hash_bytes, rel::kJoinEmpty, &jt)) != REL_OK) return s;
  rel::JoinIndex x{};
  x.hash = rel::JoinView{(const uint64_t*)jt, (uint32_t)((1ull << jl) - 1), 32u - jl};
  x.payload = payload;
  x.pkind = payload_kind;
  x.narrow = payload_kind == PAY_I8;
  x.m = m;
  if (m == 0 || (m <= kHashMaxKeys && probes <= kHashMaxRows)) {
    s = hash_entries(ctx, pk, payload, payload_kind, m, x.hash, zero);
  } else {
    x.dense_cap = 2 * m;
    x.mm = mm;
    if ((s = empty(SCR_DENSE, (size_t)x.dense_cap * 4 + 16, 0, &dt)) != REL_OK) return s;
    x.dense = dt;
    if ((s = scratch(ctx, SCR_MINMAX, (size_t)kMinMaxGrid * 8, &part)) != REL_OK) return s;
    const int32_t parts = key_minmax(ctx, pk, m, (uint32_t*)part, zero);
    s = index_entries(ctx, pk, payload_kind, x, (const uint32_t*)part, parts);
  }
  *out = x;
  return s;
}

void join_index_wiped(rel_ctx* ctx, const rel::JoinIndex& x) {
  scratch_emptied(ctx, SCR_JOIN_TABLE);
  if (x.dense) scratch_emptied(ctx, SCR_DENSE);
}

rel_status join_index_verify(rel_ctx* ctx, const rel::JoinIndex& x) {
  if (x.m == 0) return REL_OK;
  KernelTimer kt(ctx, "join_index_verify");
  hipLaunchKernelGGL(k_index_verify, dim3(1), dim3(kVerifyBlock), 0, ctx->stream, x, ctx->d_status);
  REL_LAUNCH_CHECK(ctx, "join index verify");
  return REL_OK;
}

uint32_t join_log2cap(int64_t m, const rel_table_opts* opts) {
  double load = (opts && opts->max_load > 0.f) ? (double)opts->max_load : 0.5;
  if (load > 0.9) load = 0.9;
  int64_t want = (int64_t)((double)(m > 0 ? m : 1) / load) + 1;
  if (opts && opts->capacity_hint > want) want = opts->capacity_hint;
  uint32_t l = log2_ceil((uint64_t)want);
  if (l < 4) l = 4;
  return l;
}

}  // namespace relh

namespace {

// A stand-alone table's memory: 2^log2cap + 1 slots, of which a dense array
// uses as much as its range needs, then the tail: the keys' order-encoded
// minimum and maximum, the entry count and the count's arrivals.
constexpr size_t kTailBytes = 32;
// From this many keys a table may be dense. Below it the hash table (at most
// 2 MB) stays in L2 and the two kernels more cost as much as they save.
constexpr int64_t kDenseMinKeys = 1 << 16;

uint64_t* table_tail(const rel_join_table* t) { return (uint64_t*)((char*)t->slots + t->bytes - kTailBytes); }

rel::JoinIndex table_index(const rel_join_table* t, const int32_t* payload) {
  rel::JoinIndex x{};
  x.hash = rel::JoinView{t->slots, (uint32_t)((1ull << t->log2cap) - 1), 32u - t->log2cap};
  x.dense = t->slots;
  x.mm = (const uint32_t*)table_tail(t);
  // at most twice the keys, and what the slots hold
  x.dense_cap = std::min<int64_t>(2 * t->m, (int64_t)1 << (t->log2cap + (t->wide ? 0 : 1)));
  x.payload = payload;
  x.pkind = t->wide ? PAY_I32 : PAY_ROW_ID;
  x.wide = t->wide;
  x.m = t->m;
  return x;
}

// Table memory: a context keeps the last table's memory that was given back
// (one buffer, freed with the context, when another one takes its place or
// when any of the library's allocations for the context fails), because
// allocating and freeing the 256 MB of a 15M-key table for each query took 0.3
// ms, as long as building and probing it. The memory of a table whose work all
// went to one stream is kept, for a table on the same stream, whose kernels
// follow the old ones'; any other goes back through hipFree, which waits for the
// device. The stream is the caller's and may be gone by now, so it is told by the
// context's turns, not by its address, and not asked. Of recorded work nothing is
// kept or reused, so that no graph holds memory that another table gets.
rel_status take_table(rel_ctx* ctx, size_t bytes, uint64_t** out) {
  if (!relh::capturing(ctx->stream)) {
    std::lock_guard<std::mutex> lock(ctx->table_mu);
    ScratchBuf& b = ctx->spare;
    if (b.ptr && b.bytes == bytes && ctx->spare_turn == ctx->stream_turn) {
      *out = (uint64_t*)b.ptr;
      b = ScratchBuf{};
      return REL_OK;
    }
  }
  void* p = nullptr;
  const rel_status s = relh::device_alloc(ctx, bytes, &p);
  if (s != REL_OK) return relh::fail(ctx, REL_OOM, "rel_join_build: table allocation failed");
  *out = (uint64_t*)p;
  return REL_OK;
}

// Kernels of the context's stream are about to use the table.
void note_use(const rel_join_table* t) {
  if (t->turn != t->ctx->stream_turn || relh::capturing(t->ctx->stream)) t->keep = false;
}

rel_status build_table(rel_ctx* ctx, const int32_t* pk, const int32_t* payload, const rel_join_table* t) {
  const int64_t m = t->m;
  const int64_t words = (int64_t)(1ull << t->log2cap) + 1;
  const rel::JoinIndex x = table_index(t, payload);
  const int kind = payload ? PAY_I32 : PAY_ROW_ID;
  rel_status s;
  if (!t->may_be_dense) {
    {
      relh::KernelTimer kt(ctx, "join_table_init");
      s = relh::fill_u64(ctx, t->slots, (size_t)words, rel::kJoinEmpty);
    }
    if (s != REL_OK || m == 0) return s;
    return relh::hash_entries(ctx, pk, payload, kind, m, x.hash, relh::ZeroSpans{});
  }
  void* part;
  if ((s = relh::scratch(ctx, SCR_MINMAX, (size_t)kMinMaxGrid * 8, &part)) != REL_OK) return s;
  uint64_t* tail = table_tail(t);
  const relh::ZeroSpans zero{{tail + 1, nullptr}, {2, 0}};
  const int32_t parts = relh::key_minmax(ctx, pk, m, (uint32_t*)part, relh::ZeroSpans{});
  {
    relh::KernelTimer kt(ctx, "join_table_init");
    hipLaunchKernelGGL(k_index_clear, dim3(relh::grid_for(ctx, std::max(x.dense_cap, words), kIdxBlock * 8, 4)), dim3(kIdxBlock), 0,
                       ctx->stream, x, (const uint32_t*)part, parts, zero);
    REL_LAUNCH_CHECK(ctx, "join index clear");
  }
  if ((s = relh::index_entries(ctx, pk, kind, x, nullptr, 0)) != REL_OK) return s;
  relh::KernelTimer kt(ctx, "join_index_verify");
  hipLaunchKernelGGL(k_index_count, dim3((unsigned)ctx->num_cus), dim3(kVerifyBlock), 0, ctx->stream, x, tail + 1, ctx->d_status);
  REL_LAUNCH_CHECK(ctx, "join_index_verify");
  return REL_OK;
}

}  // namespace

extern "C" {

rel_status rel_join_build(rel_ctx* ctx, const int32_t* pk, const int32_t* payload, int64_t m,
                          const rel_table_opts* opts, rel_join_table** out) {
  if (!ctx || !out || m < 0 || (m > 0 && !pk)) return relh::fail(ctx, REL_INVALID_ARG, "rel_join_build: bad argument");
  if (m >= (1ll << 30)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_join_build: m >= 2^30");
  if (opts && opts->placement != REL_PLACE_AUTO && opts->placement != REL_PLACE_GLOBAL)
    return relh::fail(ctx, REL_UNSUPPORTED, "rel_join_build: standalone tables live in device memory");
  const uint32_t l = relh::join_log2cap(m, opts);
  if (l > 31) return relh::fail(ctx, REL_UNSUPPORTED, "rel_join_build: capacity above 2^31");
  rel_join_table* t = new rel_join_table();
  t->ctx = ctx;
  t->log2cap = l;
  t->m = m;
  t->may_be_dense = m >= kDenseMinKeys && relh::aligned16(pk);  // (the range is found by 16-byte loads)
  t->turn = ctx->stream_turn;
  t->wide = payload != nullptr;
  const size_t bytes = ((size_t)8 << l) + 8;
  t->bytes = (bytes + 15) / 16 * 16 + kTailBytes;
  rel_status s = take_table(ctx, t->bytes, &t->slots);
  if (s == REL_OK) {
    note_use(t);
    s = build_table(ctx, pk, payload, t);
    if (s != REL_OK) (void)hipFree(t->slots);
  }
  if (s != REL_OK) {
    delete t;
    return s;
  }
  {
    std::lock_guard<std::mutex> lock(ctx->table_mu);
    ++ctx->tables;
  }
  *out = t;
  return REL_OK;
}

rel_status rel_join_table_destroy(rel_join_table* t) {
  if (!t) return REL_INVALID_ARG;
  rel_ctx* ctx = t->ctx;
  void* give = t->slots;
  bool last = false;
  {
    std::lock_guard<std::mutex> lock(ctx->table_mu);
    if (!ctx->closed && t->keep) {
      std::swap(give, ctx->spare.ptr);
      ctx->spare.bytes = t->bytes;
      ctx->spare_turn = t->turn;
    }
    last = --ctx->tables == 0 && ctx->closed;
  }
  if (give) (void)hipFree(give);
  if (last) delete ctx;
  delete t;
  return REL_OK;
}

rel_status rel_join_probe(rel_ctx* ctx, const rel_join_table* t, const int32_t* fk, const int32_t* sel, int64_t n,
                          int32_t* out_fact_idx, int32_t* out_payload, int64_t out_cap, int64_t* d_out_count) {
  if (!ctx || !t || n < 0 || !d_out_count || (n > 0 && (!fk || !out_fact_idx || !out_payload)))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_join_probe: bad argument");
  if (t->ctx != ctx) return relh::fail(ctx, REL_INVALID_ARG, "rel_join_probe: table belongs to another context");
  if (n >= (1ll << 31)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_join_probe: n >= 2^31");
  if (out_cap < n) return relh::fail(ctx, REL_CAPACITY, "rel_join_probe: out_cap %lld < n %lld", (long long)out_cap, (long long)n);
  rel_status s = relh::fill_u64(ctx, d_out_count, 1, 0);
  if (s != REL_OK || n == 0) return s;
  const rel::JoinIndex x = table_index(t, nullptr);
  note_use(t);
  const unsigned grid = relh::grid_for(ctx, n, kProbeBlock * kProbeRows, 8);
  relh::KernelTimer kt(ctx, "join_probe");
  auto* kernel = !t->may_be_dense ? &k_join_probe : t->wide ? &k_join_probe_index<true> : &k_join_probe_index<false>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kProbeBlock), 0, ctx->stream, x, fk, sel, n, out_fact_idx, out_payload,
                     d_out_count);
  REL_LAUNCH_CHECK(ctx, "join_probe");
  return REL_OK;
}

}  // extern "C"
