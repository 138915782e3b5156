// Internal entry points shared between librel's translation units.
#pragma once

#include "rel_device.h"
#include "rel_host.h"

namespace relh {

// Source of a join-table payload.
enum PayloadKind : int { PAY_ROW_ID = 0, PAY_I32 = 1, PAY_I8 = 2, PAY_NONE = 3 };

// Largest group count the fused pipeline keeps in its per-workgroup LDS table
// (1024 slots, load <= 0.5).
constexpr int64_t kLdsGroupCap = 512;

// log2 of the join-table capacity for m keys under opts (plain: 2m rounded up).
uint32_t join_log2cap(int64_t m, const rel_table_opts* opts);
// The join index over pk[0..m) in the context's scratch: for few keys and not too
// many rows that probe it a hash table, else a dense array when the keys' range is at most 2m wide, or the
// plain-sized hash table (decided on the device). mm: two device words that
// receive the keys' order-encoded minimum and maximum. The first kernel also
// zeroes `zero`'s spans (words later kernels of the call start from). A dense
// index is not yet checked for repeated keys: the kernel that probes it counts
// its entries (dense_count_entries, compared with m), or the caller runs
// join_index_verify. The memory is taken to be empty and has to be left empty:
// a kernel after the probing one runs join_index_wipe, and once that is
// enqueued the caller says so with join_index_wiped.
struct ZeroSpans {
  uint64_t* p[2];
  int64_t n[2];
};
rel_status join_index_build(rel_ctx* ctx, const int32_t* pk, const void* payload, int payload_kind, int64_t m,
                            int64_t probes, uint32_t* mm, const ZeroSpans& zero, rel::JoinIndex* out);
void join_index_wiped(rel_ctx* ctx, const rel::JoinIndex& x);
rel_status join_index_verify(rel_ctx* ctx, const rel::JoinIndex& x);
// Order-encoded minimum and maximum of pk[0..m) per workgroup: pair i is
// {max of ~(key ^ 2^31), max of (key ^ 2^31)} over workgroup i's keys, so the
// maxima over all pairs encode the keys' minimum and maximum. part holds
// kKeyMinMaxParts pairs; returns the number written (0 when m == 0).
constexpr int32_t kKeyMinMaxParts = 256;
int32_t key_minmax_partials(rel_ctx* ctx, const int32_t* pk, int64_t m, uint32_t* part);

// GROUP BY fk of fact JOIN dim ON fk = pk WHERE day < day_lt through radix
// partitioning of both sides and LDS-resident per-partition tables. Adds the
// passing-row and join-match counts to counters[CNT_ROWS_PASSED] and
// counters[CNT_JOIN_MATCHES]; writes groups and *d_n_groups.
rel_status partitioned_groupjoin(rel_ctx* ctx, const rel_fact* fact, const rel_dim* dim, int32_t day_lt,
                                 rel_groups_out* out, int64_t* counters);
// GROUP BY (dim.prio, fact.flag) or dim.grp over the same partitioned join:
// aggregates into the device-memory group table group_slots (2^group_log2cap
// slots plus the side slot, initialised by the caller; probe walks bounded by
// max_probe) through per-workgroup LDS tables (probe budget lds_probe), or,
// with eager (dim.grp only), through per-unit partials per dim key, which go to
// `partials` instead when that is given. Adds to the same two counters.
rel_status partitioned_join_agg(rel_ctx* ctx, const rel_fact* fact, const rel_dim* dim, int32_t day_lt, int group_by,
                                void* group_slots, uint32_t group_log2cap, uint32_t max_probe, int32_t lds_probe,
                                bool eager, const struct Partials* partials, int64_t* counters);
// Takes the memory that partitioned_join_agg needs (without partials).
rel_status partitioned_memory(rel_ctx* ctx, int64_t n, int64_t m);
// The most partials that the eager form yields, its workgroups, and the bytes of
// the buffers SCR_PART_A and SCR_PART_B that the partitioning itself needs.
void partials_bounds(rel_ctx* ctx, int64_t n, int64_t m, int64_t* max_rows, unsigned* workgroups, size_t* fact_bytes);

// Rows of a stand-alone group-by: row = sel ? sel[k] : k for k in [0, n).
struct GroupRows {
  const int64_t* key;
  const int64_t* price;
  const int32_t* qty;
  const int32_t* sel;
  int64_t n;
};

// Where units of the partitioned group-by write finished groups.
struct DirectOut {
  int64_t* key;
  int64_t* sum_price;
  int64_t* sum_qty;
  int64_t* count;
  int64_t cap;
  uint64_t* n_direct;  // groups written so far (may exceed cap)
  uint32_t* touched;   // set when a group went to the device table instead
};

// How a group-by decides between LDS tables over its rows as they come (few
// groups) and partitioning them.
enum GroupbyMode : int { GB_FEW = 0, GB_MANY, GB_SAMPLE };
// Writes the decision (1: few groups) to *few and clears words[0, n_words) and state[0, n_state).
rel_status groupby_begin(rel_ctx* ctx, const GroupRows& in, int mode, uint32_t* few, uint64_t* words, int32_t n_words,
                         uint64_t* state, int64_t n_state);
// Takes the memory that groupby_partitioned needs.
rel_status groupby_memory(rel_ctx* ctx, int64_t rows, int64_t expected);
// Groups of the rows, unless *few: straight to `o`, or to the device table g
// (set *o.touched), about `expected` of them.
rel_status groupby_partitioned(rel_ctx* ctx, const GroupRows& in, int64_t expected, const uint32_t* few,
                               const rel::GroupView& g, const DirectOut& o);

// Partial sums by group that a kernel's workgroups leave in chunks of memory, and
// how many of a chunk's lie in each bin. Workgroup w of the first_chunks fills
// chunk w first and takes more from *n_chunks (on from first_chunks).
constexpr int kPartialTile = 5120;  // of a chunk: a tile that is sorted in LDS
constexpr int kPartialMost = 2048;  // that a workgroup adds at a time
struct PartialCols {
  int32_t* key;
  uint64_t* price;
  uint64_t* qty;
  uint32_t* count;
};
struct Partials {
  PartialCols cols;    // [max_chunks * kPartialTile]
  PartialCols binned;  // [max_rows]
  uint32_t* fill;      // [max_chunks]
  uint32_t* hist;      // [max_chunks][nb]
  char* work;
  uint32_t* n_chunks;
  uint32_t nb, shift;
  int64_t first_chunks, max_chunks, max_rows;
};
// Memory for partials, in SCR_PART_A and _B (at least `at_least` bytes each, for
// what lies there before) and SCR_GROUPBY. *n_chunks is zero at the start.
rel_status partials_take(rel_ctx* ctx, int64_t max_rows, unsigned workgroups, int64_t expected, size_t at_least,
                         uint32_t* n_chunks, Partials* p);
// The partials' groups to `o`, or to the device table g (set *o.touched); *zero is 0.
rel_status partials_reduce(rel_ctx* ctx, const Partials& p, int64_t expected, const uint32_t* zero, const rel::GroupView& g,
                           const DirectOut& o);

}  // namespace relh
