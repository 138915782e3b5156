// Learned planner: the input sketch (HyperLogLog of fact.fk and dim.grp,
// statistics of sampled rows), the MLP's forward / backward / Adam kernels,
// and the sizing rule that turns a prediction into a plan.
//
// HyperLogLog follows Flajolet, Fusy, Gandouet and Meunier (2007): m = 64
// registers indexed by the top 6 bits of a 64-bit hash; each keeps the
// largest rho = 1 + leading zeros of the remaining 58 bits (59 if all zero).
// The hash of an int32 key is the first SplitMix64 output (Steele, Lea and
// Flood 2014) with the key as the state.
#include <algorithm>
#include <cmath>

#include "rel_device.h"
#include "rel_host.h"
#include "rel_ops.h"

namespace {

using namespace rel;

constexpr int kFeat = REL_SKETCH_FEATURES;
constexpr int kIn = 40, kH = 64, kOut = 2;
constexpr int kW1 = 0, kB1 = kW1 + kIn * kH, kW2 = kB1 + kH, kB2 = kW2 + kH * kH, kW3 = kB2 + kH, kB3 = kW3 + kH * kOut;
constexpr int kParams = kB3 + kOut;
static_assert(kParams == REL_MLP_PARAMS, "parameter layout");
constexpr int kMaxSample = 256;

// The sketch reads every key of both columns once (300 MB at 60M fact and 15M dim
// rows, 59 us at the rate of a copy); the hash's 64-bit products cost as much
// again where they do not overlap with the loads, since 32-bit multiplies run at
// a quarter of the rate and a 64-bit product is three of them. So only the hash's
// high word is computed, where it decides the row, and the first product's part
// of the constant high word is picked, not multiplied: five multiplies per key.
// One launch for both columns takes 80 us, two with the whole hash took 109;
// without the lookups of the registers in LDS it would be 65, but a hot key
// passes any common threshold (88).
constexpr uint64_t kHllAdd = 0x9E3779B97F4A7C15ull, kHllMul1 = 0xBF58476D1CE4E5B9ull, kHllMul2 = 0x94D049BB133111EBull;

__device__ __forceinline__ uint64_t hll_hash(int32_t v) {
  uint64_t z = (uint64_t)(uint32_t)v + kHllAdd;
  z = (z ^ (z >> 30)) * kHllMul1;
  z = (z ^ (z >> 27)) * kHllMul2;
  return z ^ (z >> 31);
}

// The high word of hll_hash(v).
__device__ __forceinline__ uint32_t hll_hash_high(int32_t v) {
  constexpr uint32_t kHi0 = (uint32_t)(kHllAdd >> 32), kHi1 = kHi0 + 1;  // the sum's high word, without and with a carry
  constexpr uint32_t kX0 = kHi0 ^ (kHi0 >> 30), kX1 = kHi1 ^ (kHi1 >> 30);
  const uint32_t lo = (uint32_t)v + (uint32_t)kHllAdd;
  const bool carry = lo < (uint32_t)kHllAdd;
  const uint32_t x = lo ^ __builtin_amdgcn_alignbit(carry ? kHi1 : kHi0, lo, 30);
  const uint64_t p0 = (uint64_t)x * (uint32_t)kHllMul1;
  const uint32_t pl = (uint32_t)p0;
  const uint32_t ph = (uint32_t)(p0 >> 32) + x * (uint32_t)(kHllMul1 >> 32) + (carry ? kX1 * (uint32_t)kHllMul1 : kX0 * (uint32_t)kHllMul1);
  const uint32_t yl = pl ^ __builtin_amdgcn_alignbit(ph, pl, 27), yh = ph ^ (ph >> 27);
  const uint32_t q = __umulhi(yl, (uint32_t)kHllMul2) + yl * (uint32_t)(kHllMul2 >> 32) + yh * (uint32_t)kHllMul2;
  return q ^ (q >> 31);
}

__device__ __forceinline__ void hll_add(uint32_t* regs, int32_t v) {
  const uint64_t h = hll_hash(v), w = h << 6;
  atomicMax(&regs[h >> 58], w ? (uint32_t)__clzll((long long)w) + 1u : 59u);
}

// Four keys. Reading the registers first skips most atomics once they settle; a
// row past the hash's high word (27 and more) always takes the long way.
__device__ __forceinline__ void hll_add4(uint32_t* regs, int4 v) {
  const int32_t k[4] = {v.x, v.y, v.z, v.w};
  bool more = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t h = hll_hash_high(k[i]);
    more = more || (uint32_t)__clz((int)(h << 6 | 32u)) >= min(regs[h >> 26], 26u);
  }
  if (more) {
#pragma unroll
    for (int i = 0; i < 4; ++i) hll_add(regs, k[i]);
  }
}

constexpr int kHllLoads = 2;  // 16-byte loads in flight per thread

constexpr int kHllBlock = 1024;  // two workgroups per CU: few registers to settle
constexpr int kHllCopies = 16;   // of the device's registers: atomics on one line take turns

// Registers of two columns over all rows, each with its share of the
// workgroups; regs (device, kHllCopies x 2 x 64 words) must start at zero.

__global__ __launch_bounds__(kHllBlock) void k_hll(const int32_t* __restrict__ keys0, int64_t n0, uint32_t grid0,
                                             const int32_t* __restrict__ keys1, int64_t n1, uint32_t* __restrict__ regs) {
  __shared__ uint32_t r[64];
  if (threadIdx.x < 64) r[threadIdx.x] = 0;
  __syncthreads();
  const bool second = blockIdx.x >= grid0;
  const int32_t* const keys = second ? keys1 : keys0;
  const int64_t n = second ? n1 : n0, n4 = n / 4;
  const int64_t at = (second ? blockIdx.x - grid0 : blockIdx.x) * (int64_t)blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)(second ? gridDim.x - grid0 : grid0) * blockDim.x;
  const int4* const k4 = reinterpret_cast<const int4*>(keys);
  uint32_t* const mine = regs + blockIdx.x % kHllCopies * 128 + (second ? 64 : 0);
  // A register that has seen few keys is raised often. The first keys of all
  // workgroups are therefore shared (n4 is the same for all of a column's).
  if (n4 > stride) {
    if (at < n4) hll_add4(r, k4[at]);
    __syncthreads();
    if (threadIdx.x < 64) {
      uint32_t best = r[threadIdx.x];
      __hip_atomic_fetch_max(&mine[threadIdx.x], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int c = 0; c < kHllCopies; ++c)
        best = max(best, __hip_atomic_load(&regs[c * 128 + (second ? 64 : 0) + threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      r[threadIdx.x] = best;
    }
    __syncthreads();
  }
  const int64_t start = at + (n4 > stride ? stride : 0);
  int4 v[kHllLoads], next[kHllLoads];
  auto load = [&](int64_t i, int4 (&to)[kHllLoads]) {  // (a key twice changes nothing)
#pragma unroll
    for (int k = 0; k < kHllLoads; ++k) to[k] = k4[min(i + k * stride, n4 - 1)];
  };
  if (start < n4) load(start, v);
  for (int64_t i = start; i < n4; i += stride * kHllLoads) {
    if (i + stride * kHllLoads < n4) load(i + stride * kHllLoads, next);
#pragma unroll
    for (int k = 0; k < kHllLoads; ++k) hll_add4(r, v[k]);
#pragma unroll
    for (int k = 0; k < kHllLoads; ++k) v[k] = next[k];
  }
  for (int64_t i = 4 * n4 + at; i < n; i += stride) hll_add(r, keys[i]);
  __syncthreads();
  if (threadIdx.x < 64 && r[threadIdx.x])
    __hip_atomic_fetch_max(&mine[threadIdx.x], r[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct SketchArgs {
  const int32_t* fk;
  const int32_t* day;
  const int32_t* pk;
  const int32_t* grp;
  int64_t n, m;
  int32_t day_lt, group_by;
  const int64_t* fsample;
  const int64_t* dsample;
  int32_t k;
  const uint32_t* regs;  // kHllCopies x (fk, then grp)
  float* features;
  uint8_t* hll_out;
};

// One workgroup computes the features, so its chain of dependent steps is all
// that counts: sums and extremes go over LDS only across the waves and by
// shuffles inside one, counts of conditions are ballots, several values share
// one pass over LDS, the registers' sums take a wave, a register per lane, and
// the logarithms a lane each: 17 us, where thread 0 and trees of barriers took 40.

// Sums over the 256 threads, always in the same order (thread t's with t + 128's,
// then t + 64's, ... t + 1's). Every thread calls it and gets the sums.
template <int N>
__device__ void block_sum_d(double (&v)[N], double (*buf)[256]) {
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < N; ++i) buf[i][t] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int l = t & 63;
    double x = (buf[i][l] + buf[i][l + 128]) + (buf[i][l + 64] + buf[i][l + 192]);
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) x += __shfl_down(x, s, kWave);
    v[i] = __shfl(x, 0, kWave);
  }
  __syncthreads();
}

// Threads of the 256 for which each of N conditions holds.
template <int N>
__device__ void block_counts(const bool (&c)[N], int (&n)[N], int (*buf)[4]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint64_t b = __ballot(c[i]);
    if ((threadIdx.x & 63) == 0) buf[i][threadIdx.x / kWave] = __popcll(b);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) n[i] = buf[i][0] + buf[i][1] + buf[i][2] + buf[i][3];
  __syncthreads();
}

// Maxima of N values over the 256 threads (a minimum is the maximum of ~v).
template <int N>
__device__ void block_max(int32_t (&v)[N], int (*buf)[4]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v[i] = max(v[i], __shfl_xor(v[i], s, kWave));
    if ((threadIdx.x & 63) == 0) buf[i][threadIdx.x / kWave] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = max(max(buf[i][0], buf[i][1]), max(buf[i][2], buf[i][3]));
  __syncthreads();
}

// How often a thread's sample occurs among the k, and whether it is the first
// of them. vals[j] is the same word for all lanes; from k on the array holds
// zeros, which are taken off again. Two instructions per comparison, and two
// more for the samples of the thread's own wave, where it matters which come
// before it.
__device__ __forceinline__ void sample_freq(const int32_t* vals, int k, int* count, bool* first) {
  const int t = threadIdx.x, wave = t / kWave, lane = t % kWave;
  const int32_t v = vals[t];
  const int4* const v4 = reinterpret_cast<const int4*>(vals);
  int c = 0, before = 0;
  for (int w = 0; w < kMaxSample / kWave; ++w) {
    if (w == wave) before += c;
#pragma unroll
    for (int j = 0; j < kWave / 4; ++j) {
      const int4 x = v4[w * (kWave / 4) + j];
      c += (x.x == v) + (x.y == v) + (x.z == v) + (x.w == v);
    }
  }
#pragma unroll
  for (int j = 0; j < kWave / 4; ++j) {
    const int4 x = v4[wave * (kWave / 4) + j];
    before += (x.x == v && 4 * j < lane) + (x.y == v && 4 * j + 1 < lane) + (x.z == v && 4 * j + 2 < lane) + (x.w == v && 4 * j + 3 < lane);
  }
  *count = c - (v == 0 ? kMaxSample - k : 0);
  *first = before == 0;
}

// A column's 64 registers, one per lane: estimate, zero registers, sum, largest.
__device__ double hll_estimate(uint32_t reg, int* zeros, double* sum, uint32_t* most) {
  double z = ldexp(1.0, -(int)reg), t = (double)reg;
  uint32_t mx = reg;
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
    z += __shfl_xor(z, s, kWave);
    t += __shfl_xor(t, s, kWave);
    mx = max(mx, (uint32_t)__shfl_xor((int)mx, s, kWave));
  }
  const int zr = __popcll(__ballot(reg == 0));
  double e = 0.709 * 64.0 * 64.0 / z;
  if (e <= 2.5 * 64.0 && zr > 0) e = 64.0 * log(64.0 / (double)zr);
  *zeros = zr;
  *sum = t;
  *most = mx;
  return e;
}

// The 40 features (one workgroup of 256 threads, k <= 256 samples):
//  0 log2(1+N)  1 log2(1+M)  2 log2((1+N)/(1+M))  3 sampled selectivity
//  4..6 one-hot group mode (fk, dim.grp, (prio, flag))
//  7..10 sampled fk: distinct, singletons, doubletons, max frequency (each / k)
//  11 fraction of sampled fk inside [min, max] of sampled pk
//  12 log2(1 + range of sampled fk)  13 log2(1 + range of sampled pk)
//  14..16 sampled grp: distinct / k, singletons / k, log2(1 + range)
//  17..20 HLL(fk): log2(1 + estimate), zero registers / 64, mean register / 16, max register / 64
//  21..36 histogram of the fk registers (value v in bin min(v, 15)) / 64
//  37..38 HLL(grp): log2(1 + estimate), zero registers / 64
//  39 Pearson correlation of sampled (day, fk), 0 when degenerate
__global__ __launch_bounds__(256) void k_sketch_features(SketchArgs a) {
  static_assert(kMaxSample == 256, "a sample per thread");
  __shared__ alignas(16) int32_t s_fk[kMaxSample], s_grp[kMaxSample];
  __shared__ double dbuf[3][256];
  __shared__ int ibuf[8][4];
  __shared__ int hist[16];
  __shared__ double f[kFeat];
  const int t = threadIdx.x, k = a.k;
  const double kk = (double)k;
  const bool in = t < k, hn = a.n > 0, hm = a.m > 0, hg = hm && a.grp != nullptr;
  uint32_t reg = 0;
#pragma unroll
  for (int c = 0; c < kHllCopies; ++c) reg = max(reg, a.regs[c * 128 + (t & 127)]);
  const int64_t fs = in && hn ? a.fsample[t] : 0, ds = in && hm ? a.dsample[t] : 0;
  const int32_t fk = in && hn ? a.fk[fs] : 0, day = in && hn ? a.day[fs] : 0;
  const int32_t pk = in && hm ? a.pk[ds] : 0, grp = in && hg ? a.grp[ds] : 0;
  s_fk[t] = fk;
  s_grp[t] = grp;
  if (t < kFeat) f[t] = 0.0;
  if (t < 16) hist[t] = 0;
  if (t < 128) a.hll_out[t] = (uint8_t)reg;
  __syncthreads();
  // every thread takes part in all of these, also where a side has no rows
  int32_t ext[6] = {in ? fk : INT32_MIN, in ? ~fk : INT32_MIN, in ? pk : INT32_MIN, in ? ~pk : INT32_MIN,
                    in ? grp : INT32_MIN, in ? ~grp : INT32_MIN};
  int fc, gc;
  bool ffirst, gfirst;
  sample_freq(s_fk, k, &fc, &ffirst);
  sample_freq(s_grp, k, &gc, &gfirst);
  block_max(ext, ibuf);
  const int32_t fmax = ext[0], fmin = ~ext[1], pmax = ext[2], pmin = ~ext[3], gmax = ext[4], gmin = ~ext[5];
  int32_t freq[1] = {in ? fc : 0};
  block_max(freq, ibuf);
  int cnt[7];  // rows passed, keys inside; distinct, single and double keys; distinct and single groups
  const bool cond[7] = {in && day < a.day_lt, in && fk >= pmin && fk <= pmax, in && ffirst, in && fc == 1,
                        in && ffirst && fc == 2, in && gfirst, in && gc == 1};
  block_counts(cond, cnt, ibuf);
  double mean[2] = {in ? (double)day : 0.0, in ? (double)fk : 0.0};
  block_sum_d(mean, dbuf);
  const double da = in ? (double)day - mean[0] / kk : 0.0, db = in ? (double)fk - mean[1] / kk : 0.0;
  double mom[3] = {da * da, db * db, da * db};
  block_sum_d(mom, dbuf);
  if (t < kWave) {  // the fk registers
    int zeros;
    double sum;
    uint32_t mx;
    const double e = hll_estimate(reg, &zeros, &sum, &mx);
    atomicAdd(&hist[min(reg, 15u)], 1);
    if (t == 0) {
      f[17] = log2(1.0 + e);
      f[18] = zeros / 64.0;
      f[19] = sum / 64.0 / 16.0;
      f[20] = mx / 64.0;
    }
  } else if (t < 2 * kWave) {  // the grp registers
    int zeros;
    double sum;
    uint32_t mx;
    const double e = hll_estimate(reg, &zeros, &sum, &mx);
    if (t == kWave && a.grp != nullptr) {
      f[37] = log2(1.0 + e);
      f[38] = zeros / 64.0;
    }
  } else if (t < 3 * kWave) {  // the logarithms, one per lane
    const int l = t - 2 * kWave;
    const double n1 = 1.0 + (double)a.n, m1 = 1.0 + (double)a.m;
    const double x = l == 0   ? n1
                     : l == 1 ? m1
                     : l == 2 ? n1 / m1
                     : l == 3 ? (hn ? 1.0 + ((double)fmax - (double)fmin) : 1.0)
                     : l == 4 ? (hn && hm ? 1.0 + ((double)pmax - (double)pmin) : 1.0)
                     : l == 5 ? (hg ? 1.0 + ((double)gmax - (double)gmin) : 1.0)
                              : 1.0;
    const double y = log2(x);
    const int at = l < 3 ? l : l == 3 ? 12 : l == 4 ? 13 : 16;
    if (l < 6) f[at] = y;
  } else if (t == 3 * kWave) {
    f[4] = a.group_by == REL_GROUP_FK;
    f[5] = a.group_by == REL_GROUP_DIM_GRP;
    f[6] = a.group_by == REL_GROUP_PRIO_FLAG;
    if (hn) {
      f[3] = cnt[0] / kk;
      f[7] = cnt[2] / kk;
      f[8] = cnt[3] / kk;
      f[9] = cnt[4] / kk;
      f[10] = freq[0] / kk;
      if (hm) f[11] = cnt[1] / kk;
      f[39] = (mom[0] > 0 && mom[1] > 0) ? mom[2] / sqrt(mom[0] * mom[1]) : 0.0;
    }
    if (hg) {
      f[14] = cnt[5] / kk;
      f[15] = cnt[6] / kk;
    }
  }
  __syncthreads();
  if (t < 16) f[21 + t] = hist[t] / 64.0;
  __syncthreads();
  if (t < kFeat) a.features[t] = (float)f[t];
}

// ---- MLP ----------------------------------------------------------------------------------------------------------------

// The network's kernels are bound by latency, not by arithmetic (a training
// step of 256 samples is 14 MFLOP): what counts is how few dependent steps a
// workgroup takes. A workgroup of four waves stages the parameters into LDS
// and takes 16 samples at a time; lane j of wave q holds hidden unit j of the
// samples 4 q .. 4 q + 3, so a weight is read from LDS once for four samples
// and the samples' inputs, stored unit by unit, come as one broadcast 16-byte
// read. At 256 samples: forward 6.5 us, backward 11.3 us and the reduction 3.1
// us; one wave per workgroup and one sample at a time took 29.6, 61.9 and 5.5.
constexpr int kSPB = 16;           // samples of a workgroup's step
constexpr int kMlpBlock = 256;
constexpr int kSPT = 4;            // samples per thread
constexpr int kSRow = kSPB + 4;    // row of a [unit][sample] array: lanes' 16-byte accesses spread over the banks
constexpr int kW2Row = kH + 1;     // W2's rows, padded so that a lane may also walk its own row
constexpr int kMaxGradParts = 256; // workgroups (and partial gradients) of a backward pass

struct alignas(16) MlpLds {
  float w1[kIn * kH], w2[kH * kW2Row], w3[kH * kOut], b1[kH], b2[kH], b3[kOut];
  alignas(16) float x[kIn * kSRow];
  alignas(16) float h1[kH * kSRow];
  alignas(16) float h2[kH * kSRow];
  float y[kSPB * kOut];

  __device__ __forceinline__ float* param(int i) {
    if (i < kB1) return &w1[i];
    if (i < kW2) return &b1[i - kB1];
    if (i < kB2) return &w2[(i - kW2) / kH * kW2Row + (i - kW2) % kH];
    if (i < kW3) return &b2[i - kB2];
    if (i < kB3) return &w3[i - kW3];
    return &b3[i - kB3];
  }
  // All loads of a thread in flight before the first is stored.
  __device__ __forceinline__ void load_params(const float* __restrict__ p) {
    constexpr int kN = (kParams + kMlpBlock - 1) / kMlpBlock;
    float v[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      const int i = k * kMlpBlock + (int)threadIdx.x;
      v[k] = i < kParams ? p[i] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      const int i = k * kMlpBlock + (int)threadIdx.x;
      if (i < kParams) *param(i) = v[k];
    }
  }
  // The samples s0 .. s0 + 15 (those past B as zeros).
  __device__ __forceinline__ void load_x(const float* __restrict__ xg, int s0, int B) {
    for (int e = threadIdx.x; e < kSPB * kIn; e += kMlpBlock) {
      const int s = e / kIn, i = e % kIn;
      x[i * kSRow + s] = s0 + s < B ? xg[(size_t)(s0 + s) * kIn + i] : 0.f;
    }
  }
  // One hidden layer for the thread's four samples: out[j] = relu(b[j] + sum_i in[i] w[i][j]),
  // summed in the order of i; the units of samples past B are zero.
  template <int N, int ROW>
  __device__ __forceinline__ void layer(const float* in, const float* w, const float* b, float* out, int valid) {
    const int j = threadIdx.x & (kWave - 1), q = threadIdx.x / kWave;
    const float bj = b[j];
    float z[kSPT] = {bj, bj, bj, bj};
#pragma unroll 8
    for (int i = 0; i < N; ++i) {
      const float wi = w[i * ROW + j];
      const float4 v = *reinterpret_cast<const float4*>(in + i * kSRow + kSPT * q);
      z[0] += v.x * wi;
      z[1] += v.y * wi;
      z[2] += v.z * wi;
      z[3] += v.w * wi;
    }
#pragma unroll
    for (int k = 0; k < kSPT; ++k) z[k] = z[k] > 0.f && kSPT * q + k < valid ? z[k] : 0.f;
    *reinterpret_cast<float4*>(out + j * kSRow + kSPT * q) = make_float4(z[0], z[1], z[2], z[3]);
  }
  // Both hidden layers and the outputs of a step of `valid` samples; ends with a barrier.
  __device__ __forceinline__ void forward(int valid) {
    layer<kIn, kH>(x, w1, b1, h1, valid);
    __syncthreads();
    layer<kH, kW2Row>(h1, w2, b2, h2, valid);
    __syncthreads();
    if (threadIdx.x < kSPB * kOut) {
      const int s = threadIdx.x / kOut, o = threadIdx.x % kOut;
      float v = b3[o];
#pragma unroll 8
      for (int i = 0; i < kH; ++i) v += h2[i * kSRow + s] * w3[i * kOut + o];
      y[threadIdx.x] = v;
    }
    __syncthreads();
  }
};

__global__ __launch_bounds__(kMlpBlock) void k_mlp_forward(const float* __restrict__ params, const float* __restrict__ x,
                                                           int32_t B, float* __restrict__ y) {
  __shared__ MlpLds m;
  const int s0 = blockIdx.x * kSPB, valid = min(kSPB, B - s0);
  m.load_x(x, s0, B);
  m.load_params(params);
  __syncthreads();
  m.forward(valid);
  if ((int)threadIdx.x < valid * kOut) y[(size_t)s0 * kOut + threadIdx.x] = m.y[threadIdx.x];
}

// sum_s a[s] b[s] over a step's samples, added to `acc` in the order of s.
__device__ __forceinline__ float dot_samples(const float* a, const float (&b)[kSPB], float acc) {
#pragma unroll
  for (int k = 0; k < kSPB / 4; ++k) {
    const float4 v = *reinterpret_cast<const float4*>(a + 4 * k);
    acc += v.x * b[4 * k];
    acc += v.y * b[4 * k + 1];
    acc += v.z * b[4 * k + 2];
    acc += v.w * b[4 * k + 3];
  }
  return acc;
}

__device__ __forceinline__ void read_samples(const float* a, float (&b)[kSPB]) {
#pragma unroll
  for (int k = 0; k < kSPB / 4; ++k) {
    const float4 v = *reinterpret_cast<const float4*>(a + 4 * k);
    b[4 * k] = v.x;
    b[4 * k + 1] = v.y;
    b[4 * k + 2] = v.z;
    b[4 * k + 3] = v.w;
  }
}

// Per-workgroup partial gradients over steps blockIdx.x, blockIdx.x + G, ...
// Lane j of wave q owns rows 10 q .. 10 q + 9 of W1's column j and rows 16 q ..
// 16 q + 15 of W2's; waves 0 and 1 also W3, the biases and the loss. Every
// entry has one owner, which keeps it in a register over all steps, so
// nothing needs an atomic and the sums have a fixed order.
__global__ __launch_bounds__(kMlpBlock) void k_mlp_backward(const float* __restrict__ params, const float* __restrict__ x,
                                                            const float* __restrict__ tgt, int32_t B,
                                                            float* __restrict__ partial, float* __restrict__ partial_loss) {
  __shared__ MlpLds m;
  __shared__ alignas(16) float dz1[kH * kSRow];
  __shared__ alignas(16) float dz2[kH * kSRow];
  __shared__ float dy[kSPB * kOut];
  __shared__ float s_loss[kSPB * kOut];
  const int t = threadIdx.x, j = t & (kWave - 1), q = t / kWave;
  constexpr int kR1 = kIn / 4, kR2 = kH / 4;
  float g1[kR1] = {}, g2[kR2] = {}, g3 = 0.f, gb1 = 0.f, gb2 = 0.f, gb3 = 0.f, loss = 0.f;
  const float invB = 1.0f / (float)B;
  m.load_params(params);
  for (int s0 = blockIdx.x * kSPB; s0 < B; s0 += gridDim.x * kSPB) {
    const int valid = min(kSPB, B - s0);
    m.load_x(x, s0, B);
    __syncthreads();
    m.forward(valid);
    if (t < kSPB * kOut) {
      const float d = t < valid * kOut ? m.y[t] - tgt[(size_t)s0 * kOut + t] : 0.f;
      dy[t] = d * invB;
      s_loss[t] = d * d;
    }
    __syncthreads();
    // output layer: W3 and b3 (entry t), and the second layer's deltas
    float4 d2;
    {
      const float wa = m.w3[j * kOut], wb = m.w3[j * kOut + 1];
      const float4 h = *reinterpret_cast<const float4*>(m.h2 + j * kSRow + kSPT * q);
      const float* e = dy + kSPT * q * kOut;
      d2.x = h.x > 0.f ? e[0] * wa + e[1] * wb : 0.f;
      d2.y = h.y > 0.f ? e[2] * wa + e[3] * wb : 0.f;
      d2.z = h.z > 0.f ? e[4] * wa + e[5] * wb : 0.f;
      d2.w = h.w > 0.f ? e[6] * wa + e[7] * wb : 0.f;
      *reinterpret_cast<float4*>(dz2 + j * kSRow + kSPT * q) = d2;
    }
    if (t < kH * kOut) {
      const int i = t / kOut, o = t % kOut;
      for (int s = 0; s < kSPB; ++s) g3 += m.h2[i * kSRow + s] * dy[s * kOut + o];
    } else if (t < kH * kOut + kOut) {
      for (int s = 0; s < kSPB; ++s) gb3 += dy[s * kOut + (t - kH * kOut)];
    } else if (t == kMlpBlock - 1) {
      for (int s = 0; s < kSPB; ++s) loss += s_loss[s * kOut] + s_loss[s * kOut + 1];
    }
    __syncthreads();
    // second layer: W2's column j, and the first layer's deltas (unit j)
    float d[kSPB];
    read_samples(dz2 + j * kSRow, d);
#pragma unroll
    for (int r = 0; r < kR2; ++r) g2[r] = dot_samples(m.h1 + (kR2 * q + r) * kSRow, d, g2[r]);
    if (q == 1) {
#pragma unroll
      for (int s = 0; s < kSPB; ++s) gb2 += d[s];
    }
    float e[kSPT] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int c = 0; c < kH; ++c) {
      const float w = m.w2[j * kW2Row + c];
      const float4 v = *reinterpret_cast<const float4*>(dz2 + c * kSRow + kSPT * q);
      e[0] += v.x * w;
      e[1] += v.y * w;
      e[2] += v.z * w;
      e[3] += v.w * w;
    }
    const float4 h = *reinterpret_cast<const float4*>(m.h1 + j * kSRow + kSPT * q);
    *reinterpret_cast<float4*>(dz1 + j * kSRow + kSPT * q) =
        make_float4(h.x > 0.f ? e[0] : 0.f, h.y > 0.f ? e[1] : 0.f, h.z > 0.f ? e[2] : 0.f, h.w > 0.f ? e[3] : 0.f);
    __syncthreads();
    // first layer: W1's column j
    read_samples(dz1 + j * kSRow, d);
#pragma unroll
    for (int r = 0; r < kR1; ++r) g1[r] = dot_samples(m.x + (kR1 * q + r) * kSRow, d, g1[r]);
    if (q == 0) {
#pragma unroll
      for (int s = 0; s < kSPB; ++s) gb1 += d[s];
    }
    __syncthreads();  // the next step writes x
  }
  float* out = partial + (size_t)blockIdx.x * kParams;
#pragma unroll
  for (int r = 0; r < kR1; ++r) out[kW1 + (kR1 * q + r) * kH + j] = g1[r];
#pragma unroll
  for (int r = 0; r < kR2; ++r) out[kW2 + (kR2 * q + r) * kH + j] = g2[r];
  if (q == 0) out[kB1 + j] = gb1;
  if (q == 1) out[kB2 + j] = gb2;
  if (t < kH * kOut) out[kW3 + t] = g3;
  else if (t < kH * kOut + kOut) out[kB3 + t - kH * kOut] = gb3;
  if (t == kMlpBlock - 1) partial_loss[blockIdx.x] = loss;
}

// Sum the per-workgroup partials: a thread adds every fourth one, in order,
// and the four sums are added in order (deterministic).
constexpr int kReduceCols = 64;
constexpr int kReduceBurst = 8;
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* __restrict__ partial, const float* __restrict__ partial_loss,
                                                    int32_t nparts, int32_t B, float* __restrict__ grad,
                                                    float* __restrict__ loss) {
  __shared__ float s_part[4][kReduceCols];
  const int c = threadIdx.x % kReduceCols, g = threadIdx.x / kReduceCols;
  const int i = blockIdx.x * kReduceCols + c;
  float s = 0.f;
  if (i < kParams) {
    for (int b0 = g; b0 < nparts; b0 += 4 * kReduceBurst) {
      float v[kReduceBurst];
#pragma unroll
      for (int k = 0; k < kReduceBurst; ++k) {
        const int b = b0 + 4 * k;
        v[k] = b < nparts ? partial[(size_t)b * kParams + i] : 0.f;
      }
#pragma unroll
      for (int k = 0; k < kReduceBurst; ++k) s += v[k];
    }
  }
  s_part[g][c] = s;
  __syncthreads();
  if (g == 0 && i < kParams) grad[i] = s_part[0][c] + s_part[1][c] + s_part[2][c] + s_part[3][c];
  if (blockIdx.x == 0 && g == 1 && loss) {
    float l = 0.f;
    for (int b = c; b < nparts; b += kWave) l += partial_loss[b];
    l = wave_sum(l);
    if (c == 0) *loss = l / (2.0f * (float)B);
  }
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                                              const float* __restrict__ g, float lr, float b1, float b2, float eps,
                                              float bc1, float bc2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kParams) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / bc1, vh = vi / bc2;
  p[i] -= lr * mh / (sqrtf(vh) + eps);
}

// The network's input. Features that grow with the input size enter relative
// to a reference scale r, the log2 HyperLogLog estimate of the group key
// (fk; dim.grp; for (prio, flag) the smaller of the fk estimate and
// log2(1 + M)): log2 N, log2 M, the sampled key ranges and both estimates
// become differences from r, and the register-level HLL features (their
// level moves with the size) are left out. The network's group output is
// likewise log2(1 + groups) - r and its join output log2(1 + join rows) -
// log2(1 + N). A model trained on small instances then carries over to much
// larger ones. The result is standardised with the training mean and scale.
// aux[0] = raw sampled max frequency (feature 10, the sizing rule's skew
// signal), aux[1] = r, aux[2] = log2(1 + N).
constexpr int kRelFeat[] = {0, 1, 12, 13, 16, 17, 37};

__global__ void k_prepare_input(float* __restrict__ x, const float* __restrict__ mean, const float* __restrict__ scale,
                                float* __restrict__ aux) {
  __shared__ float s_r;
  const int i = threadIdx.x;
  if (i == 0) {
    const float r = x[4] > 0.5f ? x[17] : x[5] > 0.5f ? x[37] : fminf(x[17], x[1]);
    s_r = r;
    aux[0] = x[10];
    aux[1] = r;
    aux[2] = x[0];
  }
  __syncthreads();
  if (i < kFeat) {
    float v = x[i];
    bool rel = false;
#pragma unroll
    for (int j = 0; j < 7; ++j) rel |= i == kRelFeat[j];
    if (rel) v -= s_r;
    else if (i >= 19 && i <= 36) v = 0.f;
    x[i] = (v - mean[i]) / scale[i];
  }
}

// A key seen this often among the sampled rows marks a heavy hitter (about
// 1.5% of the rows or more).
constexpr float kSkewMaxFreq = 4.0f / 256.0f;
// Under such a heavy hitter, with at most so many groups from a dim attribute,
// the plain join (device-memory table) beats the partitioned one: the hot keys'
// probes stay in cache and the groups in LDS, while partitioning still pays its
// passes. How many groups that is depends on how hot the hottest key is and on the
// rows: what LDS cannot hold is updates of few slots in device memory. Measured,
// partitioned time over plain at 1350 / 1700 / 2048 groups and 5M dim keys, f the
// hottest key's share of the rows:
//    2M rows, f 0.03   1.19 1.08 1.07
//    4M rows, f 0.03   0.93 0.76 0.77    f 0.14   1.29 1.17 1.13
//    8M                0.73 0.56 0.58             1.19 1.04 1.04
//   16M                0.57 0.41 0.43             1.04 0.79 0.65    f 0.24   1.43 1.33 1.09
//   60M                0.39 0.27 0.28             0.84 0.63 0.60             1.35 1.16 1.13
// (15M keys alike; 1000 groups at f 0.14 and more 1.17 to 1.80.) The partitioned
// path also wins for every group count when no key is hot.
int64_t plain_join_groups(int64_t n, float max_freq) {
  return (double)max_freq >= 0.05 * std::log2((double)n / (1 << 21)) ? 2048 : 1280;
}

#define TRY(e)                   \
  do {                           \
    rel_status s_ = (e);         \
    if (s_ != REL_OK) return s_; \
  } while (0)

}  // namespace

struct rel_planner {
  rel_ctx* ctx = nullptr;
  float* mem = nullptr;  // params, mean, scale, features, prediction
  float margin = 0.f;
};

extern "C" {

rel_status rel_sketch(rel_ctx* ctx, const rel_fact* fact, const rel_dim* dim, const rel_query* q,
                      const int64_t* d_fact_sample, const int64_t* d_dim_sample, int32_t k, float* d_features,
                      uint8_t* d_hll) {
  if (!ctx || !fact || !dim || !q || !d_features || !d_hll || k < 1 || k > kMaxSample || fact->n < 0 || dim->m < 0 ||
      (fact->n > 0 && (!fact->fk || !fact->day || !d_fact_sample)) || (dim->m > 0 && (!dim->pk || !d_dim_sample)))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_sketch: bad argument");
  if ((fact->fk && !relh::aligned16(fact->fk)) || (dim->grp && !relh::aligned16(dim->grp)))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_sketch: column not 16-byte aligned");
  void* regs;
  TRY(relh::scratch(ctx, SCR_SKETCH, kHllCopies * 128 * sizeof(uint32_t), &regs));
  TRY(relh::fill_u32(ctx, regs, kHllCopies * 128, 0));
  {
    relh::KernelTimer kt(ctx, "sketch_hll");
    const int64_t gm = dim->grp ? dim->m : 0;
    auto grid = [&](int64_t rows) { return rows > 0 ? (unsigned)relh::grid_for(ctx, rows / 4 + 1, kHllBlock * kHllLoads, 2) : 0u; };
    const unsigned g0 = grid(fact->n), g1 = grid(gm);
    if (g0 + g1 > 0)
      hipLaunchKernelGGL(k_hll, dim3(g0 + g1), dim3(kHllBlock), 0, ctx->stream, fact->fk, fact->n, g0, dim->grp, gm, (uint32_t*)regs);
  }
  SketchArgs a{};
  a.fk = fact->fk;
  a.day = fact->day;
  a.pk = dim->pk;
  a.grp = dim->grp;
  a.n = fact->n;
  a.m = dim->m;
  a.day_lt = q->day_lt;
  a.group_by = q->group_by;
  a.fsample = d_fact_sample;
  a.dsample = d_dim_sample;
  a.k = k;
  a.regs = (const uint32_t*)regs;
  a.features = d_features;
  a.hll_out = d_hll;
  relh::KernelTimer kt(ctx, "sketch_features");
  hipLaunchKernelGGL(k_sketch_features, dim3(1), dim3(256), 0, ctx->stream, a);
  REL_LAUNCH_CHECK(ctx, "sketch");
  return REL_OK;
}

rel_status rel_mlp_forward(rel_ctx* ctx, const float* d_params, const float* d_x, int32_t B, float* d_y) {
  if (!ctx || !d_params || !d_x || !d_y || B < 0) return relh::fail(ctx, REL_INVALID_ARG, "rel_mlp_forward: bad argument");
  if (B == 0) return REL_OK;
  relh::KernelTimer kt(ctx, "mlp_forward");
  hipLaunchKernelGGL(k_mlp_forward, dim3((B + kSPB - 1) / kSPB), dim3(kMlpBlock), 0, ctx->stream, d_params, d_x, B, d_y);
  REL_LAUNCH_CHECK(ctx, "mlp_forward");
  return REL_OK;
}

rel_status rel_mlp_backward(rel_ctx* ctx, const float* d_params, const float* d_x, const float* d_t, int32_t B,
                            float* d_grad, float* d_loss) {
  if (!ctx || !d_params || !d_x || !d_t || !d_grad || B < 1)
    return relh::fail(ctx, REL_INVALID_ARG, "rel_mlp_backward: bad argument");
  const int32_t nb = std::min((B + kSPB - 1) / kSPB, kMaxGradParts);
  void* part;
  TRY(relh::scratch(ctx, SCR_MLP, ((size_t)nb * kParams + nb) * sizeof(float), &part));
  float* pl = (float*)part + (size_t)nb * kParams;
  relh::KernelTimer kt(ctx, "mlp_backward");
  hipLaunchKernelGGL(k_mlp_backward, dim3(nb), dim3(kMlpBlock), 0, ctx->stream, d_params, d_x, d_t, B, (float*)part, pl);
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kParams + kReduceCols - 1) / kReduceCols), dim3(256), 0, ctx->stream, (const float*)part,
                     (const float*)pl, nb, B, d_grad, d_loss);
  REL_LAUNCH_CHECK(ctx, "mlp_backward");
  return REL_OK;
}

rel_status rel_mlp_adam_step(rel_ctx* ctx, float* d_params, float* d_m, float* d_v, const float* d_grad, int32_t t,
                             float lr, float beta1, float beta2, float eps) {
  if (!ctx || !d_params || !d_m || !d_v || !d_grad || t < 1) return relh::fail(ctx, REL_INVALID_ARG, "rel_mlp_adam_step: bad argument");
  const float bc1 = (float)(1.0 - std::pow((double)beta1, (double)t));
  const float bc2 = (float)(1.0 - std::pow((double)beta2, (double)t));
  relh::KernelTimer kt(ctx, "mlp_adam");
  hipLaunchKernelGGL(k_adam, dim3((kParams + 255) / 256), dim3(256), 0, ctx->stream, d_params, d_m, d_v, d_grad, lr, beta1,
                     beta2, eps, bc1, bc2);
  REL_LAUNCH_CHECK(ctx, "mlp_adam");
  return REL_OK;
}

rel_status rel_planner_create(rel_ctx* ctx, const float* params, const float* mean, const float* scale,
                              float margin_log2, rel_planner** out) {
  if (!ctx || !params || !mean || !scale || !out || !(margin_log2 >= 0.f))
    return relh::fail(ctx, REL_INVALID_ARG, "rel_planner_create: bad argument");
  for (int i = 0; i < kFeat; ++i)
    if (!(scale[i] > 0.f)) return relh::fail(ctx, REL_INVALID_ARG, "rel_planner_create: scale[%d] must be > 0", i);
  rel_planner* p = new rel_planner();
  p->ctx = ctx;
  p->margin = margin_log2;
  const size_t floats = kParams + 3 * kFeat + 8 + 64;  // params, mean, scale, features, prediction + aux, HLL bytes
  void* mem;
  const rel_status s = relh::device_alloc(ctx, floats * sizeof(float), &mem);
  p->mem = (float*)mem;
  if (s != REL_OK) {
    delete p;
    return relh::fail(ctx, REL_OOM, "rel_planner_create: allocation failed");
  }
  if (hipMemcpy(p->mem, params, kParams * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(p->mem + kParams, mean, kFeat * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(p->mem + kParams + kFeat, scale, kFeat * sizeof(float), hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipFree(p->mem);
    delete p;
    return relh::fail(ctx, REL_HIP, "rel_planner_create: copy failed");
  }
  *out = p;
  return REL_OK;
}

rel_status rel_planner_plan(rel_planner* p, const rel_fact* fact, const rel_dim* dim, const rel_query* q,
                            const int64_t* d_fact_sample, const int64_t* d_dim_sample, int32_t k, rel_plan* plan,
                            float* pred) {
  if (!p || !plan) return REL_INVALID_ARG;
  rel_ctx* ctx = p->ctx;
  float* params = p->mem;
  float* mean = params + kParams;
  float* scale = mean + kFeat;
  float* feat = scale + kFeat;
  float* y = feat + kFeat;  // y[0], y[1]: network outputs; y[2..4]: aux of k_prepare_input
  uint8_t* hll = (uint8_t*)(y + 8);
  TRY(rel_sketch(ctx, fact, dim, q, d_fact_sample, d_dim_sample, k, feat, hll));
  {
    relh::KernelTimer kt(ctx, "planner_input");
    hipLaunchKernelGGL(k_prepare_input, dim3(1), dim3(64), 0, ctx->stream, feat, (const float*)mean,
                       (const float*)scale, y + 2);
  }
  REL_LAUNCH_CHECK(ctx, "prepare_input");
  TRY(rel_mlp_forward(ctx, params, feat, 1, y));
  float hy[5];
  REL_HIP_CHECK(ctx, hipMemcpyAsync(hy, y, sizeof hy, hipMemcpyDeviceToHost, ctx->stream));
  REL_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
  const double log2_join = (double)hy[0] + hy[4], log2_groups = (double)hy[1] + hy[3];
  if (pred) {
    pred[0] = (float)log2_join;
    pred[1] = (float)log2_groups;
  }
  // sizing rule: expected groups = 2^(prediction + margin), never above the plain bound
  const int64_t n = fact->n, m = dim->m;
  const int64_t ub = q->group_by == REL_GROUP_PRIO_FLAG ? std::min<int64_t>(n, 65536) : std::min(n, m);
  double e = std::exp2(log2_groups + (double)p->margin);
  if (!std::isfinite(e) || e > (double)ub) e = (double)ub;
  int64_t expected = (int64_t)std::ceil(e);
  if (expected < 1) expected = 1;
  plan->group_capacity = expected;
  // LDS holds every group when they are few; under a heavy hitter it also pays
  // as a cache in front of a larger device-memory table
  const bool skewed = hy[2] >= kSkewMaxFreq;
  plan->group_placement = (expected <= relh::kLdsGroupCap || skewed) ? REL_PLACE_LDS : REL_PLACE_GLOBAL;
  plan->join_placement = (skewed && q->group_by != REL_GROUP_FK && expected <= plain_join_groups(n, hy[2]))
                             ? REL_PLACE_GLOBAL
                             : REL_PLACE_AUTO;
  plan->allow_fallback = 1;
  plan->reserved = 0;
  return REL_OK;
}

rel_status rel_planner_destroy(rel_planner* p) {
  if (!p) return REL_INVALID_ARG;
  (void)hipStreamSynchronize(p->ctx->stream);
  if (p->mem) (void)hipFree(p->mem);
  delete p;
  return REL_OK;
}

}  // extern "C"
