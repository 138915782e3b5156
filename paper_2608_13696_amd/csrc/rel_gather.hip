// Join-output materialisation: out[i] = in[map[i]] for the columns a consumer
// of the join wants, with map = the probe's fact rows or dim rows.
//
// This is the gather the paper finds behind cuDF's most expensive kernel by
// aggregate time (Section 7, the transform kernel): an unrolled loop that
// reads and writes one element per access and so leaves bandwidth unused. Here
// each thread owns four consecutive pairs: it reads their indices with one
// 16-byte load per side, issues the four element reads of a column together,
// and writes the four results with one store of 4 x elem_bytes (16 bytes for
// int32 columns, two for int64). Row indices are checked against the source
// column's length; an index out of range sets REL_DEV_BADARG and writes zero.
#include "rel_device.h"
#include "rel_host.h"
#include "rel_ops.h"

namespace {

using namespace rel;

constexpr int kGBlock = 256;
constexpr int kGMaxCols = 8;

struct GCol {
  const void* src;
  void* dst;
  int64_t src_rows;
  int32_t eb;    // element bytes: 1, 2, 4 or 8
  int32_t side;  // 0: indexed by fact row, 1: by dim row
};

struct GatherArgs {
  const int32_t* fidx;
  const int32_t* didx;
  const int64_t* d_n;
  int64_t max_pairs;
  uint32_t* status;
  int32_t ncols;
  GCol cols[kGMaxCols];
};

// `c.side` 0: fact rows come in ascending runs, so their elements stream and
// are not worth keeping; dim rows come in any order.
template <class T>
__device__ __forceinline__ T gather_one(const GCol& c, int32_t row, uint32_t* status) {
  if ((uint64_t)(uint32_t)row >= (uint64_t)c.src_rows) {
    set_status(status, kDevBadArg);
    return T(0);
  }
  return c.side ? static_cast<const T*>(c.src)[row] : ld_once(static_cast<const T*>(c.src) + row);
}

// Four consecutive results at element i0 (a multiple of four).
template <class T>
__device__ __forceinline__ void store_quad(const GCol& c, int64_t i0, T v0, T v1, T v2, T v3) {
  T* d = static_cast<T*>(c.dst) + i0;
  if constexpr (sizeof(T) == 1) {
    *reinterpret_cast<uint32_t*>(d) = (uint32_t)(uint8_t)v0 | (uint32_t)(uint8_t)v1 << 8 |
                                      (uint32_t)(uint8_t)v2 << 16 | (uint32_t)(uint8_t)v3 << 24;
  } else if constexpr (sizeof(T) == 2) {
    *reinterpret_cast<uint2*>(d) = make_uint2((uint32_t)(uint16_t)v0 | (uint32_t)(uint16_t)v1 << 16,
                                              (uint32_t)(uint16_t)v2 | (uint32_t)(uint16_t)v3 << 16);
  } else if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<uint4*>(d) = make_uint4((uint32_t)v0, (uint32_t)v1, (uint32_t)v2, (uint32_t)v3);
  } else {
    *reinterpret_cast<ulonglong2*>(d) = make_ulonglong2((unsigned long long)v0, (unsigned long long)v1);
    *reinterpret_cast<ulonglong2*>(d + 2) = make_ulonglong2((unsigned long long)v2, (unsigned long long)v3);
  }
}

// Four pairs starting at i0 (all in range): element reads first, then one store.
template <class T>
__device__ __forceinline__ void gather_quad(const GCol& c, const int4& idx, int64_t i0, uint32_t* status) {
  const T v0 = gather_one<T>(c, idx.x, status);
  const T v1 = gather_one<T>(c, idx.y, status);
  const T v2 = gather_one<T>(c, idx.z, status);
  const T v3 = gather_one<T>(c, idx.w, status);
  store_quad<T>(c, i0, v0, v1, v2, v3);
}

template <class T>
__device__ __forceinline__ void gather_tail(const GCol& c, const int32_t* fidx, const int32_t* didx, int64_t i,
                                            uint32_t* status) {
  const int32_t row = c.side ? didx[i] : fidx[i];
  static_cast<T*>(c.dst)[i] = gather_one<T>(c, row, status);
}

__global__ __launch_bounds__(kGBlock) void k_join_gather(GatherArgs a) {
  int64_t n = *a.d_n;
  if (n > a.max_pairs) {
    if (blockIdx.x == 0 && threadIdx.x == 0) set_status(a.status, kDevBadArg);
    n = a.max_pairs;
  }
  if (n < 0) n = 0;
  if (a.ncols == 0) return;
  const int64_t quads = n / 4;
  const int64_t stride = (int64_t)gridDim.x * kGBlock;
  bool need_f = false, need_d = false;
  for (int c = 0; c < a.ncols; ++c) {
    need_f |= a.cols[c].side == 0;
    need_d |= a.cols[c].side != 0;
  }
  for (int64_t q = blockIdx.x * (int64_t)kGBlock + threadIdx.x; q < quads; q += stride) {
    const int64_t i0 = 4 * q;
    const int4 f = need_f ? ld_once(reinterpret_cast<const int4*>(a.fidx + i0)) : make_int4(0, 0, 0, 0);
    const int4 d = need_d ? ld_once(reinterpret_cast<const int4*>(a.didx + i0)) : make_int4(0, 0, 0, 0);
    for (int c = 0; c < a.ncols; ++c) {
      const GCol& col = a.cols[c];
      const int4& idx = col.side ? d : f;
      switch (col.eb) {
        case 1: gather_quad<uint8_t>(col, idx, i0, a.status); break;
        case 2: gather_quad<uint16_t>(col, idx, i0, a.status); break;
        case 4: gather_quad<uint32_t>(col, idx, i0, a.status); break;
        default: gather_quad<uint64_t>(col, idx, i0, a.status); break;
      }
    }
  }
  // the last n mod 4 pairs, one thread each
  const int64_t t = blockIdx.x * (int64_t)kGBlock + threadIdx.x;
  if (t < n - 4 * quads) {
    const int64_t i = 4 * quads + t;
    for (int c = 0; c < a.ncols; ++c) {
      const GCol& col = a.cols[c];
      switch (col.eb) {
        case 1: gather_tail<uint8_t>(col, a.fidx, a.didx, i, a.status); break;
        case 2: gather_tail<uint16_t>(col, a.fidx, a.didx, i, a.status); break;
        case 4: gather_tail<uint32_t>(col, a.fidx, a.didx, i, a.status); break;
        default: gather_tail<uint64_t>(col, a.fidx, a.didx, i, a.status); break;
      }
    }
  }
}

// A dim column larger than an XCD's L2, read by slices (sliced_read): a thread
// takes four quads of pairs.
constexpr int kSliceQuads = kSliceReads / 4;

template <class T>
__global__ __launch_bounds__(kGBlock, 8) void k_join_gather_sliced(GCol c, const int32_t* __restrict__ idx,
                                                                   const int64_t* __restrict__ d_n, int64_t max_pairs,
                                                                   uint32_t* __restrict__ status) {
  const int64_t n = max(min(*d_n, max_pairs), (int64_t)0);
  const int64_t quads = n / 4;
  const int64_t b0 = (int64_t)blockIdx.x * kGBlock * kSliceQuads;
  if (b0 > quads) return;
  const int64_t q0 = b0 + threadIdx.x;
  const uint32_t rows = (uint32_t)c.src_rows, bytes = rows * (uint32_t)sizeof(T);
  uint32_t o[kSliceReads];
  typename SliceReg<T>::type v[kSliceReads];
#pragma unroll
  for (int u = 0; u < kSliceQuads; ++u) {
    const int64_t q = q0 + u * kGBlock;
    const int4 t = q < quads ? ld_once(reinterpret_cast<const int4*>(idx) + q) : make_int4(0, 0, 0, 0);
    o[4 * u] = t.x;
    o[4 * u + 1] = t.y;
    o[4 * u + 2] = t.z;
    o[4 * u + 3] = t.w;
  }
  bool bad = false;
#pragma unroll
  for (int k = 0; k < kSliceReads; ++k) {
    v[k] = 0;
    bad |= o[k] >= rows;
    o[k] = o[k] < rows ? o[k] * (uint32_t)sizeof(T) : ~0u;
  }
  if (bad) set_status(status, kDevBadArg);
  sliced_read<T>(c.src, bytes, o, v);
#pragma unroll
  for (int u = 0; u < kSliceQuads; ++u) {
    const int64_t q = q0 + u * kGBlock;
    if (q < quads) store_quad<T>(c, 4 * q, (T)v[4 * u], (T)v[4 * u + 1], (T)v[4 * u + 2], (T)v[4 * u + 3]);
  }
  // the last n mod 4 pairs
  if (blockIdx.x == 0 && threadIdx.x < n - 4 * quads) gather_tail<T>(c, nullptr, idx, 4 * quads + threadIdx.x, status);
}

// Fact rows come in ascending runs, which need no slices.
bool take_sliced(const GCol& c, int64_t max_pairs) {
  return c.side == REL_SIDE_DIM && sliced_size(c.src_rows * c.eb) && max_pairs >= kSliceMinReads;
}

template <class T>
void launch_sliced(rel_ctx* ctx, const GCol& c, const int32_t* idx, const int64_t* d_n, int64_t max_pairs) {
  const int64_t per = (int64_t)kGBlock * kSliceQuads;
  const unsigned grid = (unsigned)((max_pairs / 4 + per - 1) / per + (max_pairs < 4));
  hipLaunchKernelGGL(k_join_gather_sliced<T>, dim3(grid), dim3(kGBlock), 0, ctx->stream, c, idx, d_n, max_pairs,
                     ctx->d_status);
}

}  // namespace

extern "C" {

rel_status rel_join_gather(rel_ctx* ctx, const int32_t* fact_idx, const int32_t* dim_idx, const int64_t* d_n_pairs,
                           int64_t max_pairs, const rel_gather_col* cols, int32_t n_cols) {
  if (!ctx || !cols || !d_n_pairs || n_cols < 1 || n_cols > kGMaxCols || max_pairs < 0)
    return relh::fail(ctx, REL_INVALID_ARG, "rel_join_gather: bad argument");
  if (max_pairs >= (1ll << 31)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_join_gather: max_pairs >= 2^31");
  GatherArgs a{};
  GCol sliced[kGMaxCols];
  int n_sliced = 0;
  bool need_f = false, need_d = false;
  for (int32_t c = 0; c < n_cols; ++c) {
    const rel_gather_col& g = cols[c];
    const int eb = g.elem_bytes;
    if ((eb != 1 && eb != 2 && eb != 4 && eb != 8) || (g.side != REL_SIDE_FACT && g.side != REL_SIDE_DIM) ||
        g.src_rows < 0 || (g.src_rows > 0 && !g.src) || (max_pairs > 0 && !g.dst))
      return relh::fail(ctx, REL_INVALID_ARG, "rel_join_gather: column %d invalid", c);
    if (((uintptr_t)g.src % (uintptr_t)eb) != 0 || !relh::aligned16(g.dst))
      return relh::fail(ctx, REL_INVALID_ARG, "rel_join_gather: column %d misaligned (src to its element, dst to 16 B)", c);
    const GCol col{g.src, g.dst, g.src_rows, eb, g.side};
    if (take_sliced(col, max_pairs)) sliced[n_sliced++] = col;
    else a.cols[a.ncols++] = col;
    need_f |= g.side == REL_SIDE_FACT;
    need_d |= g.side == REL_SIDE_DIM;
  }
  if (max_pairs > 0 && ((need_f && (!fact_idx || !relh::aligned16(fact_idx))) || (need_d && (!dim_idx || !relh::aligned16(dim_idx)))))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_join_gather: index arrays must be non-null and 16-byte aligned");
  if (max_pairs == 0) return REL_OK;
  a.fidx = fact_idx;
  a.didx = dim_idx;
  a.d_n = d_n_pairs;
  a.max_pairs = max_pairs;
  a.status = ctx->d_status;
  const unsigned grid = relh::grid_for(ctx, (max_pairs + 3) / 4, kGBlock, 8);
  relh::KernelTimer kt(ctx, "join_gather");
  // (also with no column left: it checks the count)
  hipLaunchKernelGGL(k_join_gather, dim3(a.ncols ? grid : 1), dim3(kGBlock), 0, ctx->stream, a);
  for (int c = 0; c < n_sliced; ++c) {
    const GCol& col = sliced[c];
    switch (col.eb) {
      case 1: launch_sliced<uint8_t>(ctx, col, dim_idx, d_n_pairs, max_pairs); break;
      case 2: launch_sliced<uint16_t>(ctx, col, dim_idx, d_n_pairs, max_pairs); break;
      case 4: launch_sliced<uint32_t>(ctx, col, dim_idx, d_n_pairs, max_pairs); break;
      default: launch_sliced<uint64_t>(ctx, col, dim_idx, d_n_pairs, max_pairs); break;
    }
  }
  REL_LAUNCH_CHECK(ctx, "join_gather");
  return REL_OK;
}

}  // extern "C"
