// General selection predicates: a conjunction of typed terms, compiled or
// interpreted (declared in rel.h).
//
// Both modes are the first pass of a selection (rel_select.h): a bit per row,
// which k_select_expand turns into row ids. A term is first brought to one of
// three exact tests (Test): a closed range, membership by a 64-bit map of
// small integers, or a list; the range's complement serves NE. Integer tests
// on columns of at most 32 bits are done in 32 bits, float tests in float,
// with bounds moved to the nearest value of the column's type inside them.
//   * compiled: the pass is generated for the predicate and built with hipRTC
//     for the device it runs on: the tests' constants are in the code, and a
//     lane issues the loads of all columns for several chunks before any
//     test.
//   * interpreted: one kernel of the library walks the tests, each for a
//     lane's 32 rows at a time, so that one dispatch on type and test serves
//     2048 rows of a wave and its eight or sixteen loads are in flight
//     together. A wave none of whose rows is left stops.
// Either is bound by HBM. A 4-term predicate over 60M rows of 17 B, 4.8M of
// them selected: 0.178 ms compiled (5.8 TB/s), 0.194 ms interpreted (5.3
// TB/s). Testing 16 consecutive rows per lane, so that a wave's loads were 64
// B or more apart, in a single pass with a look-back took 0.32 ms compiled;
// walking the terms row by row took 1.92 ms.
#include <hip/hiprtc.h>

#include <cinttypes>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <string>
#include <vector>

#include "rel_device.h"
#include "rel_host.h"
#include "rel_select.h"

namespace {

using namespace rel;

// Bytes of one element of a rel_dtype (I8, I16, I32, I64, F32, F64).
int dtype_bytes(int dt) {
  static const int kBytes[] = {1, 2, 4, 8, 4, 8};
  return kBytes[dt];
}

enum TestKind : int32_t {
  T_RANGE = 0,  // lo <= x <= hi
  T_MAP,        // x - lo in [0, 63] and that bit of `map` set (integers)
  T_LIST        // x equals one of v[0 .. nv)
};

// Values are bit patterns of the type the column is tested in: int32 for I8,
// I16 and I32, else the column's own.
struct Test {
  int32_t column, dtype, kind, negate, nv;
  uint64_t lo, hi, map;
  uint64_t v[REL_PRED_MAX_VALUES];
};

struct Program {
  int32_t n;
  Test t[REL_PRED_MAX_TERMS];
};

struct Columns {
  const void* c[8];
};

template <class V>
uint64_t to_bits(V v) {
  uint64_t b = 0;
  std::memcpy(&b, &v, sizeof v);
  return b;
}

template <class V>
__host__ __device__ __forceinline__ V from_bits(uint64_t b) {
  V v;
  __builtin_memcpy(&v, &b, sizeof v);
  return v;
}

// The closed range of doubles that a comparison keeps; empty as [NaN, NaN].
void fp_range(const rel_pred_term& t, double* lo, double* hi) {
  const double inf = std::numeric_limits<double>::infinity(), v = t.fvalues[0];
  *lo = -inf;
  *hi = inf;
  switch (t.op) {
    case REL_OP_LT: *hi = v == -inf ? NAN : std::nextafter(v, -inf); break;
    case REL_OP_LE: *hi = v; break;
    case REL_OP_GT: *lo = v == inf ? NAN : std::nextafter(v, inf); break;
    case REL_OP_GE: *lo = v; break;
    case REL_OP_BETWEEN: *lo = v; *hi = t.fvalues[1]; break;
    default: *lo = *hi = v; break;  // EQ, and NE negated
  }
}

// The closed range of integers that a comparison keeps; empty as lo > hi.
void int_range(const rel_pred_term& t, int64_t* lo, int64_t* hi) {
  const int64_t v = t.ivalues[0];
  *lo = INT64_MIN;
  *hi = INT64_MAX;
  switch (t.op) {
    case REL_OP_LT: if (v == INT64_MIN) { *lo = 1; *hi = 0; } else *hi = v - 1; break;
    case REL_OP_LE: *hi = v; break;
    case REL_OP_GT: if (v == INT64_MAX) { *lo = 1; *hi = 0; } else *lo = v + 1; break;
    case REL_OP_GE: *lo = v; break;
    case REL_OP_BETWEEN: *lo = v; *hi = t.ivalues[1]; break;
    default: *lo = *hi = v; break;
  }
}

Test make_test(const rel_pred_term& t) {
  Test r{};
  r.column = t.column;
  r.dtype = t.dtype;
  r.kind = t.op == REL_OP_IN ? T_LIST : T_RANGE;
  r.negate = t.op == REL_OP_NE;
  if (t.dtype >= REL_DT_F32) {
    const bool f32 = t.dtype == REL_DT_F32;
    if (t.op == REL_OP_IN) {
      // a float column equals only literals that are floats; NaN equals nothing
      for (int j = 0; j < t.n_values; ++j) {
        const double v = t.fvalues[j];
        if (v != v || (f32 && (double)(float)v != v)) continue;
        r.v[r.nv++] = f32 ? to_bits((float)v) : to_bits(v);
      }
      return r;
    }
    double lo, hi;
    fp_range(t, &lo, &hi);
    if (!f32) {
      r.lo = to_bits(lo);
      r.hi = to_bits(hi);
      return r;
    }
    const float inf = std::numeric_limits<float>::infinity();
    float a = (float)lo, b = (float)hi;
    if ((double)a < lo) a = std::nextafter(a, inf);
    if ((double)b > hi) b = std::nextafter(b, -inf);
    r.lo = to_bits(a);
    r.hi = to_bits(b);
    return r;
  }
  const bool wide = t.dtype == REL_DT_I64;
  const int64_t tmin = wide ? INT64_MIN : INT32_MIN, tmax = wide ? INT64_MAX : INT32_MAX;
  auto put = [&](int64_t v) { return wide ? (uint64_t)v : (uint64_t)(uint32_t)(int32_t)v; };
  if (t.op == REL_OP_IN) {
    int64_t lo = INT64_MAX, hi = INT64_MIN;
    for (int j = 0; j < t.n_values; ++j) {
      const int64_t v = t.ivalues[j];
      if (v < tmin || v > tmax) continue;
      r.v[r.nv++] = put(v);
      lo = v < lo ? v : lo;
      hi = v > hi ? v : hi;
    }
    if (r.nv > 0 && (uint64_t)hi - (uint64_t)lo < 64) {
      r.kind = T_MAP;
      r.lo = put(lo);
      for (int j = 0; j < t.n_values; ++j) {
        const int64_t v = t.ivalues[j];
        if (v >= tmin && v <= tmax) r.map |= 1ull << ((uint64_t)v - (uint64_t)lo);
      }
    }
    return r;
  }
  int64_t lo, hi;
  int_range(t, &lo, &hi);
  lo = lo < tmin ? tmin : lo;
  hi = hi > tmax ? tmax : hi;
  if (lo > hi) lo = 1, hi = 0;  // empty, and both bounds within the type
  r.lo = put(lo);
  r.hi = put(hi);
  return r;
}

// ---- interpreted -------------------------------------------------------------------------------------------------------

// Four consecutive elements (4-row aligned) as values to test. 8-byte types
// take two loads, the others one.
template <class T, class V>
__device__ __forceinline__ void load4(const T* p, V (&v)[4]) {
  T e[4];
  if (sizeof(T) == 1) {
    const uint32_t w = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
    __builtin_memcpy(e, &w, sizeof e);
  } else if (sizeof(T) == 2) {
    const uint64_t w = __builtin_nontemporal_load(reinterpret_cast<const uint64_t*>(p));
    __builtin_memcpy(e, &w, sizeof e);
  } else {
#pragma unroll
    for (int h = 0; h < (int)sizeof(T) / 4; ++h) {
      const v4i_t w = __builtin_nontemporal_load(reinterpret_cast<const v4i_t*>(p) + h);
      __builtin_memcpy(reinterpret_cast<char*>(e) + 16 * h, &w, 16);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (V)e[j];
}

template <class V>
__device__ __forceinline__ uint32_t in_map(V x, const Test& t) {
  if constexpr (sizeof(V) == 4) {
    const uint32_t d = (uint32_t)x - (uint32_t)t.lo;
    return d < 64u ? (uint32_t)(t.map >> d) & 1u : 0u;
  } else {
    const uint64_t d = (uint64_t)x - t.lo;
    return d < 64u ? (uint32_t)(t.map >> d) & 1u : 0u;
  }
}

// The test's outcome for K rows, bit k for x[k].
template <class V, bool INT, int K>
__device__ __forceinline__ uint32_t test_rows(const Test& t, const V (&x)[K]) {
  uint32_t m = 0;
  if (t.kind == T_RANGE) {
    const V lo = from_bits<V>(t.lo), hi = from_bits<V>(t.hi);
#pragma unroll
    for (int k = 0; k < K; ++k) m |= (uint32_t)((x[k] >= lo) & (x[k] <= hi)) << k;
    return t.negate ? ~m : m;
  }
  if constexpr (INT) {
    if (t.kind == T_MAP) {
#pragma unroll
      for (int k = 0; k < K; ++k) m |= in_map<V>(x[k], t) << k;
      return m;
    }
  }
  for (int j = 0; j < t.nv; ++j) {
    const V v = from_bits<V>(t.v[j]);
#pragma unroll
    for (int k = 0; k < K; ++k) m |= (uint32_t)(x[k] == v) << k;
  }
  return m;
}

// One term for the lane's 32 rows of a step, G chunks' loads in flight.
template <class T, class V, bool INT, int G>
__device__ __forceinline__ uint32_t test_step(const Test& t, const void* col, int64_t r0) {
  const T* p = (const T*)col + r0;
  uint32_t m = 0;
#pragma unroll 1
  for (int c = 0; c < 8; c += G) {
    V x[4 * G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      V q[4];
      load4<T, V>(p + (c + g) * kSelChunk, q);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * g + j] = q[j];
    }
    const uint32_t part = test_rows<V, INT, 4 * G>(t, x);
    m |= (4 * G == 32 ? part : part & ((1u << (4 * G % 32)) - 1u)) << (4 * c);
  }
  return m;
}

__device__ uint32_t test_one(const Test& t, const void* col, int64_t r) {
  switch (t.dtype) {
    case REL_DT_I8: { const int32_t x[1] = {((const int8_t*)col)[r]}; return test_rows<int32_t, true, 1>(t, x) & 1u; }
    case REL_DT_I16: { const int32_t x[1] = {((const int16_t*)col)[r]}; return test_rows<int32_t, true, 1>(t, x) & 1u; }
    case REL_DT_I32: { const int32_t x[1] = {((const int32_t*)col)[r]}; return test_rows<int32_t, true, 1>(t, x) & 1u; }
    case REL_DT_I64: { const int64_t x[1] = {((const int64_t*)col)[r]}; return test_rows<int64_t, true, 1>(t, x) & 1u; }
    case REL_DT_F32: { const float x[1] = {((const float*)col)[r]}; return test_rows<float, false, 1>(t, x) & 1u; }
    default: { const double x[1] = {((const double*)col)[r]}; return test_rows<double, false, 1>(t, x) & 1u; }
  }
}

__global__ __launch_bounds__(kSelBlock) void k_pred_interpreted(Program prog, Columns cols, int64_t n, int64_t tile_rows,
                                                                uint32_t* __restrict__ bits,
                                                                uint32_t* __restrict__ counts) {
  const int64_t t0 = (int64_t)blockIdx.x * tile_rows;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
  uint32_t c = 0;
  for (int64_t s = 0; s < tile_rows; s += kSelStep) {
    const int64_t base = t0 + s + (int64_t)wave * kSelWaveRows;
    const int64_t r0 = base + 4 * lane;
    uint32_t nib = 0;
    if (base + kSelWaveRows <= n) {
      nib = ~0u;
      for (int i = 0; i < prog.n; ++i) {
        const Test& t = prog.t[i];
        const void* col = cols.c[t.column];
        switch (t.dtype) {
          case REL_DT_I8: nib &= test_step<int8_t, int32_t, true, 8>(t, col, r0); break;
          case REL_DT_I16: nib &= test_step<int16_t, int32_t, true, 8>(t, col, r0); break;
          case REL_DT_I32: nib &= test_step<int32_t, int32_t, true, 8>(t, col, r0); break;
          case REL_DT_I64: nib &= test_step<int64_t, int64_t, true, 4>(t, col, r0); break;
          case REL_DT_F32: nib &= test_step<float, float, false, 8>(t, col, r0); break;
          default: nib &= test_step<double, double, false, 4>(t, col, r0); break;
        }
        if (wave_ballot(nib != 0) == 0) break;
      }
    } else if (base < n) {  // the last rows, one by one
      for (int k = 0; k < 32; ++k) {
        const int64_t r = r0 + (k / 4) * kSelChunk + k % 4;
        uint32_t ok = r < n;
        for (int i = 0; i < prog.n && ok; ++i) ok = test_one(prog.t[i], cols.c[prog.t[i].column], r);
        nib |= ok << k;
      }
    }
    c += store_bits(bits, base, nib);
  }
  store_tile_count(counts, c);
}

// ---- compiled ----------------------------------------------------------------------------------------------------------

// The pass around the generated functions `step_bits` (a lane's 32 rows of a
// whole step, U chunks' loads at a time) and `row_ok` (one row): the layout of
// rel_select.h.
const char* kSkeleton = R"SKEL(
typedef struct { const void* c[8]; } Cols;
typedef int v4i __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ void load4(const T* p, T* e) {
  if (sizeof(T) == 1) {
    const unsigned w = __builtin_nontemporal_load(reinterpret_cast<const unsigned*>(p));
    __builtin_memcpy(e, &w, 4);
  } else if (sizeof(T) == 2) {
    const unsigned long long w = __builtin_nontemporal_load(reinterpret_cast<const unsigned long long*>(p));
    __builtin_memcpy(e, &w, 8);
  } else {
#pragma unroll
    for (int h = 0; h < (int)sizeof(T) / 4; ++h) {
      const v4i w = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p) + h);
      __builtin_memcpy(reinterpret_cast<char*>(e) + 16 * h, &w, 16);
    }
  }
}

__device__ __forceinline__ unsigned step_bits(const Cols& cols, long long r0);
__device__ __forceinline__ bool row_ok(const Cols& cols, long long r);

extern "C" __global__ __launch_bounds__(256) void k_pred_compiled(Cols cols, long long n, long long tile_rows,
                                                                  unsigned* bits, unsigned* counts) {
  __shared__ unsigned s_cnt[4];
  const unsigned lane = __lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const long long t0 = (long long)blockIdx.x * tile_rows;
  unsigned c = 0;
  for (long long s = 0; s < tile_rows; s += 8192) {
    const long long base = t0 + s + (long long)wave * 2048;
    const long long r0 = base + 4 * lane;
    unsigned x = 0;
    if (base + 2048 <= n) {
      x = step_bits(cols, r0);
    } else if (base < n) {
      for (int k = 0; k < 32; ++k) {
        const long long r = r0 + (k / 4) * 256 + k % 4;
        if (r < n) x |= (unsigned)row_ok(cols, r) << k;
      }
    }
#pragma unroll
    for (int d = 1; d < 8; d <<= 1) {
      const unsigned keep = d == 1 ? 0x0F0F0F0Fu : d == 2 ? 0x00FF00FFu : 0x0000FFFFu;
      const unsigned y = (unsigned)__shfl_xor((int)x, d, 64);
      x = (lane & d) ? (x & ~keep) | ((y & ~keep) >> (4 * d)) : (x & keep) | ((y & keep) << (4 * d));
    }
    bits[base / 32 + (lane & 7u) * 8 + (lane >> 3)] = x;
    c += __popc(x);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor((int)c, o, 64);
  if (lane == 0) s_cnt[wave] = c;
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
}
)SKEL";

const char* kTypeName[6] = {"signed char", "short", "int", "long long", "float", "double"};

std::string int_literal(int64_t v) {
  if (v == INT64_MIN) return "(-9223372036854775807LL - 1)";
  char b[32];
  std::snprintf(b, sizeof b, "%" PRId64 "LL", v);
  return b;
}

std::string fp_literal(double v) {
  if (std::isnan(v)) return "__builtin_nan(\"\")";
  if (std::isinf(v)) return v > 0 ? "__builtin_inf()" : "(-__builtin_inf())";
  char b[64];
  std::snprintf(b, sizeof b, "%a", v);  // hexadecimal: the exact double
  return b;
}

// A test's value as text of the type it is tested in.
std::string literal(const Test& t, uint64_t bits) {
  switch (t.dtype) {
    case REL_DT_F32: return "(float)" + fp_literal((double)from_bits<float>(bits));
    case REL_DT_F64: return fp_literal(from_bits<double>(bits));
    case REL_DT_I64: return int_literal((int64_t)bits);
    default: return "(int)" + int_literal((int64_t)(int32_t)(uint32_t)bits);
  }
}

// The test of element expression `x` (of the type it is tested in).
std::string test_expr(const Test& t, const std::string& x) {
  if (t.kind == T_RANGE) {
    const std::string e = "((" + x + " >= " + literal(t, t.lo) + ") & (" + x + " <= " + literal(t, t.hi) + "))";
    return t.negate ? "!" + e : e;
  }
  if (t.kind == T_MAP) {
    char map[32];
    std::snprintf(map, sizeof map, "0x%" PRIx64 "ull", t.map);
    const std::string u = t.dtype == REL_DT_I64 ? "(unsigned long long)" : "(unsigned)";
    const std::string d = "(" + u + x + " - " + u + literal(t, t.lo) + ")";
    return "((" + d + " < 64u) & (bool)((" + map + " >> (" + d + " & 63u)) & 1ull))";
  }
  std::string e = "(false";
  for (int j = 0; j < t.nv; ++j) e += " | (" + x + " == " + literal(t, t.v[j]) + ")";
  return e + ")";
}

// Chunks whose loads a lane has in flight together: as many as keep them at
// 256 B per lane (64 registers), so that wide rows cost no occupancy.
int chunks_in_flight(int bytes_per_row) {
  int u = 8;
  while (u > 1 && u * bytes_per_row > 64) u /= 2;
  return u;
}

std::string generate(const Program& prog, const std::vector<int>& col_dtype, int bytes_per_row) {
  const std::string U = std::to_string(chunks_in_flight(bytes_per_row));
  std::string s = "#define U " + U + "\n";
  s += kSkeleton;
  s += "__device__ __forceinline__ unsigned step_bits(const Cols& cols, long long r0) {\n  unsigned bits = 0;\n"
       "#pragma unroll 1\n  for (int c = 0; c < 8; c += U) {\n";
  for (size_t k = 0; k < col_dtype.size(); ++k) {
    if (col_dtype[k] < 0) continue;
    const std::string T = kTypeName[col_dtype[k]], i = std::to_string(k);
    s += "    " + T + " e" + i + "[4 * U];\n    const " + T + "* p" + i + " = (const " + T + "*)cols.c[" + i + "] + r0 + c * 256;\n";
    s += "#pragma unroll\n    for (int g = 0; g < U; ++g) load4<" + T + ">(p" + i + " + g * 256, e" + i + " + 4 * g);\n";
  }
  s += "    unsigned m = 0;\n#pragma unroll\n    for (int k = 0; k < 4 * U; ++k) {\n      bool ok = true;\n";
  auto value = [&](const Test& t, const std::string& e) {
    const std::string V = t.dtype < REL_DT_I32 ? "int" : kTypeName[t.dtype];
    return "{ const " + V + " x = (" + V + ")" + e + "; ok = ok & " + test_expr(t, "x") + "; }\n";
  };
  for (int i = 0; i < prog.n; ++i) s += "      " + value(prog.t[i], "e" + std::to_string(prog.t[i].column) + "[k]");
  s += "      m |= (unsigned)ok << k;\n    }\n    bits |= m << (4 * c);\n  }\n  return bits;\n}\n";
  s += "__device__ __forceinline__ bool row_ok(const Cols& cols, long long r) {\n  bool ok = true;\n";
  for (int i = 0; i < prog.n; ++i)
    s += "  " + value(prog.t[i], std::string("((const ") + kTypeName[prog.t[i].dtype] + "*)cols.c[" + std::to_string(prog.t[i].column) + "])[r]");
  s += "  return ok;\n}\n";
  return s;
}

}  // namespace

struct rel_pred {
  rel_ctx* ctx = nullptr;
  int mode = 0;
  int max_column = -1;
  std::vector<int> col_dtype;  // dtype each used column must have (-1: unused)
  hipModule_t module = nullptr;
  hipFunction_t fn = nullptr;
  Program prog{};              // the tests, for the interpreter
};

namespace {

void free_pred(rel_pred* p) {
  if (!p) return;
  if (p->module) (void)hipModuleUnload(p->module);
  delete p;
}

rel_status compile(rel_ctx* ctx, const std::string& src, const char* kernel, hipModule_t* mod, hipFunction_t* fn) {
  hipDeviceProp_t prop;
  REL_HIP_CHECK(ctx, hipGetDeviceProperties(&prop, ctx->device));
  const std::string arch = std::string("--offload-arch=") + prop.gcnArchName;
  const char* opts[] = {arch.c_str(), "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};
  hiprtcProgram prog;
  if (hiprtcCreateProgram(&prog, src.c_str(), "rel_pred.hip", 0, nullptr, nullptr) != HIPRTC_SUCCESS)
    return relh::fail(ctx, REL_HIP, "rel_pred_create: hiprtcCreateProgram failed");
  const hiprtcResult r = hiprtcCompileProgram(prog, (int)(sizeof opts / sizeof opts[0]), opts);
  if (r != HIPRTC_SUCCESS) {
    size_t n = 0;
    hiprtcGetProgramLogSize(prog, &n);
    std::string log(n, '\0');
    if (n) hiprtcGetProgramLog(prog, &log[0]);
    hiprtcDestroyProgram(&prog);
    return relh::fail(ctx, REL_HIP, "rel_pred_create: compilation failed: %.900s", log.c_str());
  }
  size_t size = 0;
  hiprtcGetCodeSize(prog, &size);
  std::vector<char> code(size);
  hiprtcGetCode(prog, code.data());
  hiprtcDestroyProgram(&prog);
  REL_HIP_CHECK(ctx, hipModuleLoadData(mod, code.data()));
  REL_HIP_CHECK(ctx, hipModuleGetFunction(fn, *mod, kernel));
  return REL_OK;
}

}  // namespace

extern "C" {

rel_status rel_pred_create(rel_ctx* ctx, const rel_pred_term* terms, int32_t n_terms, int32_t mode, rel_pred** out) {
  if (!ctx || !terms || !out || n_terms < 1 || n_terms > REL_PRED_MAX_TERMS ||
      (mode != REL_PRED_COMPILED && mode != REL_PRED_INTERPRETED))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_pred_create: bad argument");
  std::vector<int> col_dtype;
  for (int32_t i = 0; i < n_terms; ++i) {
    const rel_pred_term& t = terms[i];
    const bool ok_n = t.op <= REL_OP_NE ? t.n_values == 1 : t.op == REL_OP_BETWEEN ? t.n_values == 2
                                                                                 : t.n_values >= 1 && t.n_values <= REL_PRED_MAX_VALUES;
    if (t.column < 0 || t.column >= 8 || t.dtype < REL_DT_I8 || t.dtype > REL_DT_F64 || t.op < REL_OP_LT ||
        t.op > REL_OP_IN || !ok_n)
      return relh::fail(ctx, REL_INVALID_ARG, "rel_pred_create: term %d invalid", i);
    if ((int)col_dtype.size() <= t.column) col_dtype.resize(t.column + 1, -1);
    if (col_dtype[t.column] != -1 && col_dtype[t.column] != t.dtype)
      return relh::fail(ctx, REL_INVALID_ARG, "rel_pred_create: column %d given two types", t.column);
    col_dtype[t.column] = t.dtype;
  }
  rel_pred* p = new rel_pred();
  p->ctx = ctx;
  p->mode = mode;
  p->col_dtype = col_dtype;
  p->max_column = (int)col_dtype.size() - 1;
  p->prog.n = n_terms;
  for (int32_t i = 0; i < n_terms; ++i) p->prog.t[i] = make_test(terms[i]);
  rel_status s = REL_OK;
  if (mode == REL_PRED_COMPILED) {
    int bytes_per_row = 0;
    for (int dt : col_dtype)
      if (dt >= 0) bytes_per_row += dtype_bytes(dt);
    s = compile(ctx, generate(p->prog, col_dtype, bytes_per_row), "k_pred_compiled", &p->module, &p->fn);
  }
  if (s != REL_OK) {
    free_pred(p);
    return s;
  }
  *out = p;
  return REL_OK;
}

rel_status rel_pred_filter(rel_pred* p, const void* const* columns, int32_t n_columns, int64_t n, int32_t* out_idx,
                           int64_t out_cap, int64_t* d_out_count) {
  if (!p) return REL_INVALID_ARG;
  rel_ctx* ctx = p->ctx;
  if (!columns || n < 0 || !d_out_count || (n > 0 && !out_idx) || n_columns <= p->max_column || n_columns > 8)
    return relh::fail(ctx, REL_INVALID_ARG, "rel_pred_filter: bad argument");
  if (n >= (1ll << 31)) return relh::fail(ctx, REL_UNSUPPORTED, "rel_pred_filter: n >= 2^31");
  if (out_cap < n) return relh::fail(ctx, REL_CAPACITY, "rel_pred_filter: out_cap < n");
  Columns cols{};
  for (int c = 0; c < n_columns; ++c) {
    const bool used = c < (int)p->col_dtype.size() && p->col_dtype[c] >= 0;
    if (used && n > 0 && (!columns[c] || !relh::aligned16(columns[c])))
      return relh::fail(ctx, REL_INVALID_ARG, "rel_pred_filter: column %d null or not 16-byte aligned", c);
    cols.c[c] = columns[c];
  }
  if (n == 0) return relh::fill_u64(ctx, d_out_count, 1, 0);
  relh::SelectPlan sp;
  const rel_status s = relh::select_plan(ctx, n, &sp);
  if (s != REL_OK) return s;
  relh::KernelTimer kt(ctx, p->mode == REL_PRED_COMPILED ? "pred_compiled" : "pred_interpreted");
  if (p->mode == REL_PRED_COMPILED) {
    void* args[] = {&cols, &sp.n, &sp.tile_rows, &sp.bits, &sp.counts};
    REL_HIP_CHECK(ctx, hipModuleLaunchKernel(p->fn, (unsigned)sp.ntiles, 1, 1, kSelBlock, 1, 1, 0, ctx->stream, args, nullptr));
  } else {
    hipLaunchKernelGGL(k_pred_interpreted, dim3((unsigned)sp.ntiles), dim3(kSelBlock), 0, ctx->stream, p->prog, cols, n,
                       sp.tile_rows, sp.bits, sp.counts);
    REL_LAUNCH_CHECK(ctx, "pred_interpreted");
  }
  return relh::select_expand(ctx, sp, out_idx, d_out_count);
}

rel_status rel_pred_destroy(rel_pred* p) {
  if (!p) return REL_INVALID_ARG;
  (void)hipStreamSynchronize(p->ctx->stream);
  free_pred(p);
  return REL_OK;
}

}  // extern "C"
