// Sparsity-path summaries of a weighted particle set (Section 5): weighted quantiles
// F^-1(alpha) per coefficient (absolute medians, credible intervals) and concentrations
// V(Delta) = 1 - Pr(|beta_j| < Delta), on the GPU.
//
// Exactness: the weights are quantised to integers q_i = floor((w_i / max w) 2^K),
// K = 63 - ceil(log2 M), so every partial sum is an exact 64-bit integer and no result
// depends on summation order.  The alpha-quantile is the smallest value whose cumulative
// q reaches ceil(alpha * C) (C = sum q, the product taken exactly in 128 bits).
//
// Selection is a most-significant-digit radix select on order-preserving integer keys of
// the values: each pass builds, per
// coefficient and level, the weighted histogram of the next digit over the values that
// still match the level's prefix, then picks the bucket where the cumulative weight
// crosses the threshold.  Two forms:
//  - sq_column_kernel (M up to 32768 FP32 or 16384 FP64 values): one workgroup per
//    coefficient holds its column and the quantised weights in registers and does the
//    whole selection in one launch;
//  - the multi-pass form for larger sets (the c-marginal mixture over T x N particles): the
//    values are transposed into per-coefficient key columns so that every pass reads
//    contiguous memory, and every pass spreads a column over many workgroups.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "spa_common.hpp"
#include "spa_internal.hpp"
#include "spa_summary.hpp"

namespace spa {

namespace {

constexpr int kPrepThreads = 1024;
constexpr int kHistThreads = 256;
constexpr int kChunk = 4096;         // values per histogram workgroup
constexpr int kBuckets = 256;

__device__ __forceinline__ uint32_t key_of(float v) {
  uint32_t u = __float_as_uint(v);
  if (u == 0x80000000u) u = 0u;      // -0 and +0 are one value
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ uint64_t key_of(double v) {
  uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
  if (u == 0x8000000000000000ull) u = 0ull;
  return (u & 0x8000000000000000ull) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double value_of_key(uint32_t k) {
  const uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return static_cast<double>(__uint_as_float(u));
}
__device__ __forceinline__ double value_of_key(uint64_t k) {
  const uint64_t u = (k & 0x8000000000000000ull) ? (k & 0x7fffffffffffffffull) : ~k;
  return __longlong_as_double(static_cast<long long>(u));
}

// ceil(alpha * C) exactly: alpha = m 2^(e - 1075) from its bit pattern (alpha in (0, 1]).
__device__ __forceinline__ uint64_t exact_threshold(double alpha, uint64_t C) {
  const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(alpha));
  const int e = static_cast<int>((bits >> 52) & 0x7ff);
  uint64_t m = bits & ((1ull << 52) - 1);
  int shift;
  if (e == 0) {
    shift = 1074;                     // subnormal: m 2^-1074
  } else {
    m |= (1ull << 52);
    shift = 1075 - e;
  }
  const unsigned __int128 prod = static_cast<unsigned __int128>(m) * C;
  if (shift >= 128) return prod != 0 ? 1ull : 0ull;
  uint64_t t = static_cast<uint64_t>(prod >> shift);
  const unsigned __int128 rem = prod & ((static_cast<unsigned __int128>(1) << shift) - 1);
  if (rem != 0) ++t;
  return t;
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ uint64_t wave_scan_u64(uint64_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t u = __shfl_up(v, o, kWave);
    if (lane >= o) v += u;
  }
  return v;
}

// ---------------------------------------------------------------- one launch per set
// One workgroup of 1024 threads per coefficient; thread t keeps the keys and quantised
// weights of particles t, t + 1024, ... (EPT of them) in registers.  Up to kColInline of
// them every workgroup also quantises the weights itself, which saves a launch; above, the
// M correctly rounded divisions in every workgroup cost more (about 20 us at M = 32768)
// than the one launch that does them once.  Then the total, the concentrations' sums, and one radix
// pass per 11-bit digit: a histogram per level in LDS and, per level, one wave that scans its 2048
// buckets (rows of 32 buckets padded by one, so that a lane's 32 consecutive buckets are read
// without bank conflicts).  In the first pass every level still matches every value, so one
// histogram serves all of them.
// Bound: the latency of the passes (about 2.5 us per digit, LDS atomics and barriers) and,
// for long rows, the transposed copy.  Measured per call at M = 16384, p = 200 FP32, 3
// levels and 2 tolerances, quantisation + column kernel: 12.7 + 21.7 us, against 190 us of
// kernels for the multi-pass form (call 223 -> 53 us); M = 1024, p = 200: call 83 -> 35 us;
// M = 16384, p = 400 FP64: 397 -> 107 us.  Sets above the register limit gain nothing from
// a second value buffer in LDS, which the histograms fill, and stay with the multi-pass form.
constexpr int kColThreads = 1024;
constexpr int kColWaves = kColThreads / 64;
constexpr int kColDigit = 11;
constexpr int kColBuckets = 1 << kColDigit;
constexpr int kColStride = kColBuckets + kColBuckets / 32;   // padded histogram length
// Above this many values per thread the weights are quantised by a launch of their own.
constexpr int kColInline = 4;
__host__ __device__ constexpr int col_ept_max(bool f64) { return f64 ? 16 : 32; }   // 128 VGPRs at 16 waves


// The largest weight over M and whether the weights are valid, the same in every thread of
// a workgroup of kColThreads.
__device__ __forceinline__ bool col_weight_max(double &mx, int bad, bool logw, double *smax, int *sbad) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  mx = wave_max(mx);
  bad = wave_sum_int(bad);
  if (lane == 0) {
    smax[wave] = mx;
    sbad[wave] = bad;
  }
  __syncthreads();
  mx = logw ? -INFINITY : 0.0;
  bad = 0;
  for (int k = 0; k < kColWaves; ++k) {
    mx = fmax(mx, smax[k]);
    bad += sbad[k];
  }
  return bad == 0 && (logw ? mx != -INFINITY : mx > 0.0);
}
__device__ __forceinline__ bool col_bad_weight(double v, bool logw) {
  return logw ? (isnan(v) || v == INFINITY) : (!(v >= 0.0) || !isfinite(v));
}
__device__ __forceinline__ uint64_t col_quantise(double v, double mx, bool logw, int K) {
  const double r = logw ? exp(v - mx) : __ddiv_rn(v, mx);   // correctly rounded division
  return static_cast<uint64_t>(floor(ldexp(r, K)));
}

// Workgroups 0 .. nq-1: the quantised weights of kColThreads particles each; every one
// finds the largest weight itself (M doubles from the L2).  Invalid weights: flag
// (nullable) and all q = 0, which the column kernel takes as the sign to leave.
// The others (when keys are wanted): 64 x 64 tiles of the values into key columns.
template <typename VT, typename KT>
__global__ __launch_bounds__(kColThreads) void sq_prep_kernel(const VT *__restrict__ vals, int M, int p,
                                                              const double *__restrict__ w, bool logw, int K, int nq,
                                                              uint64_t *__restrict__ q, KT *__restrict__ keys,
                                                              int *__restrict__ flag) {
  __shared__ KT tile[64][65];
  __shared__ double smax[kColWaves];
  __shared__ int sbad[kColWaves];
  if (static_cast<int>(blockIdx.x) < nq) {
    const int i = blockIdx.x * kColThreads + threadIdx.x;
    double mx = logw ? -INFINITY : 0.0;
    int bad = 0;
#pragma unroll 8
    for (int k = threadIdx.x; k < M; k += kColThreads) {
      const double v = w[k];
      if (col_bad_weight(v, logw)) bad = 1;
      else mx = fmax(mx, v);
    }
    const bool ok = col_weight_max(mx, bad, logw, smax, sbad);
    if (i == 0 && flag) *flag = ok ? 0 : 1;
    if (i < M) q[i] = ok ? col_quantise(w[i], mx, logw, K) : 0ull;
    return;
  }
  const int tc = (p + 63) / 64, t = static_cast<int>(blockIdx.x) - nq;
  const int i0 = t / tc * 64, j0 = t % tc * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;   // 64 x 16 threads
#pragma unroll
  for (int r = 0; r < 64; r += 16) {                        // whole rows and columns by clamping, edges not stored
    const int i = min(i0 + r + ty, M - 1), j = min(j0 + tx, p - 1);
    tile[r + ty][tx] = key_of(vals[(size_t)i * p + j]);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 64; r += 16) {
    const int i = i0 + tx, j = j0 + r + ty;
    if (i < M && j < p) keys[(size_t)j * M + i] = tile[tx][r + ty];
  }
}

template <typename VT, typename KT, int EPT, bool KEYS>
__global__ __launch_bounds__(kColThreads) void sq_column_kernel(const VT *__restrict__ vals,
                                                                const KT *__restrict__ keys, int M, int p,
                                                                const double *__restrict__ w, bool logw, int K,
                                                                const uint64_t *__restrict__ qin, SqLevels lv,
                                                                int *__restrict__ flag, double *__restrict__ quant,
                                                                double *__restrict__ conc) {
  extern __shared__ __align__(16) unsigned long long hist[];   // L x kColStride
  __shared__ double smax[kColWaves];
  __shared__ int sbad[kColWaves];
  __shared__ unsigned long long stot[1 + kSqMaxLevels];        // total weight, weight inside each tolerance
  __shared__ uint64_t sthr[kSqMaxLevels], sbelow[kSqMaxLevels], spre[kSqMaxLevels];
  constexpr int BITS = 8 * (int)sizeof(KT);
  // consecutive columns on one XCD (workgroups go round-robin to the 8 XCDs)
  const int per = (p + 7) / 8;
  const int j = static_cast<int>(blockIdx.x & 7) * per + static_cast<int>(blockIdx.x >> 3);
  if (j >= p) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  KT key[EPT];
  uint64_t q[EPT], acc = 0;
  // unconditional loads of clamped indices, so that all are in flight together
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int i = min(tid + kColThreads * e, M - 1);
    if constexpr (KEYS) key[e] = keys[(size_t)j * M + i];
    else key[e] = key_of(vals[(size_t)i * p + j]);
    if constexpr (EPT > kColInline) q[e] = qin[i];
  }
  // entries beyond M: no weight, and a key (of a NaN) that no level's prefix matches, or their
  // additions of nothing to the last value's bucket would be most of a call of few values
#pragma unroll
  for (int e = 0; e < EPT; ++e)
    if (tid + kColThreads * e >= M) {
      key[e] = static_cast<KT>(~KT(0));
      q[e] = 0;
    }
  if (tid <= kSqMaxLevels) stot[tid] = 0ull;
  if constexpr (EPT <= kColInline) {
    double wv[EPT], mx = logw ? -INFINITY : 0.0;
    int bad = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      wv[e] = w[min(tid + kColThreads * e, M - 1)];
      if (col_bad_weight(wv[e], logw)) bad = 1;
      else mx = fmax(mx, wv[e]);
    }
    const bool ok = col_weight_max(mx, bad, logw, smax, sbad);
    if (j == 0 && tid == 0 && flag) *flag = ok ? 0 : 1;
    if (!ok) return;                         // the same in every thread of every workgroup
#pragma unroll
    for (int e = 0; e < EPT; ++e) q[e] = tid + kColThreads * e < M ? col_quantise(wv[e], mx, logw, K) : 0ull;
  } else {
    __syncthreads();                         // stot is clear
  }
#pragma unroll
  for (int e = 0; e < EPT; ++e) acc += q[e];
  acc = wave_sum_u64(acc);
  if (lane == 0) atomicAdd(&stot[0], static_cast<unsigned long long>(acc));
  for (int d = 0; d < lv.D; ++d) {
    uint64_t s = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (fabs(value_of_key(key[e])) < lv.delta[d]) s += q[e];
    s = wave_sum_u64(s);
    if (lane == 0 && s != 0) atomicAdd(&stot[1 + d], static_cast<unsigned long long>(s));
  }
  __syncthreads();
  const uint64_t C = stot[0];
  if (C == 0) return;                        // invalid weights (the largest weight quantises to 2^K)
  if (tid < lv.L) {
    sthr[tid] = exact_threshold(lv.alpha[tid], C);
    sbelow[tid] = 0;
    spre[tid] = 0;
  }
  if (tid < lv.D)
    conc[(size_t)tid * p + j] = 1.0 - static_cast<double>(stot[1 + tid]) / static_cast<double>(C);
  if (lv.L == 0) return;
#pragma unroll 1
  for (int hi = BITS; hi > 0;) {
    const bool first = hi == BITS;
    const int width = min(kColDigit, hi), lo = hi - width;
    for (int k = tid; k < (first ? 1 : lv.L) * kColStride; k += kColThreads) hist[k] = 0ull;
    __syncthreads();
    if (first) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int b = static_cast<int>(key[e] >> lo) & ((1 << width) - 1);
        if (q[e] != 0) atomicAdd(&hist[b + (b >> 5)], static_cast<unsigned long long>(q[e]));
      }
    } else {
      // few values still match a level: one comparison per value and level, and the digit
      // only for a wave that holds a match
      for (int l = 0; l < lv.L; ++l) {
        const KT pre = static_cast<KT>(spre[l]);
#pragma unroll
        for (int e = 0; e < EPT; ++e)
          if ((key[e] >> hi) == pre) {
            const int b = static_cast<int>(key[e] >> lo) & ((1 << width) - 1);
            atomicAdd(&hist[l * kColStride + b + (b >> 5)], static_cast<unsigned long long>(q[e]));
          }
      }
    }
    __syncthreads();
    if (wave < lv.L) {                       // level `wave`: the bucket that crosses its threshold
      const unsigned long long *h = hist + (first ? 0 : wave) * kColStride;
      uint64_t loc = 0;
#pragma unroll
      for (int k = 0; k < 32; ++k) loc += h[33 * lane + k];
      const uint64_t need = sthr[wave] - sbelow[wave];   // > 0 and <= the weight still in range
      // the row of 32 buckets that crosses, then its bucket: two wave scans (always found
      // for valid weights)
      const uint64_t incl = wave_scan_u64(loc);
      const unsigned long long brow = __ballot(incl >= need);
      const int row = brow ? __builtin_ctzll(brow) : 63;
      const uint64_t before = __shfl(incl - loc, row, kWave);
      const uint64_t cb = lane < 32 ? h[33 * row + lane] : 0ull;
      const uint64_t in2 = before + wave_scan_u64(cb);
      const unsigned long long bb = __ballot(in2 >= need);
      const int src = bb ? min(__builtin_ctzll(bb), 31) : 31;
      if (lane == src) {
        const uint64_t pre = (spre[wave] << width) | static_cast<uint64_t>(32 * row + src);
        spre[wave] = pre;
        sbelow[wave] += in2 - cb;
        if (lo == 0) quant[(size_t)wave * p + j] = value_of_key(static_cast<KT>(pre));
      }
    }
    __syncthreads();
    hi = lo;
  }
}

// ---------------------------------------------------------------- multi-pass form
// One workgroup: max weight, validation, quantised weights, their total and the exact
// thresholds of every level.  st->flags bit 0: invalid weights.
__global__ __launch_bounds__(kPrepThreads) void sq_prepare_kernel(const double *__restrict__ w, int M,
                                                                   bool logw, int K, SqLevels lv,
                                                                   uint64_t *__restrict__ q,
                                                                   SqState *__restrict__ st) {
  __shared__ double smax[kPrepThreads / 64];
  __shared__ uint64_t ssum[kPrepThreads / 64];
  __shared__ int sbad[kPrepThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double mx = logw ? -INFINITY : 0.0;
  int bad = 0;
  for (int i = tid; i < M; i += kPrepThreads) {
    const double v = w[i];
    if (logw ? (isnan(v) || v == INFINITY) : (!(v >= 0.0) || !isfinite(v))) bad = 1;
    else mx = fmax(mx, v);
  }
  mx = wave_max(mx);
  bad = wave_sum_int(bad);
  if (lane == 0) {
    smax[wave] = mx;
    sbad[wave] = bad;
  }
  __syncthreads();
  mx = logw ? -INFINITY : 0.0;
  bad = 0;
  for (int k = 0; k < kPrepThreads / 64; ++k) {
    mx = fmax(mx, smax[k]);
    bad += sbad[k];
  }
  if (bad > 0 || (logw ? mx == -INFINITY : !(mx > 0.0))) {
    if (tid == 0) st->flags = 1;
    return;
  }
  uint64_t acc = 0;
  for (int i = tid; i < M; i += kPrepThreads) {
    const double r = logw ? exp(w[i] - mx) : __ddiv_rn(w[i], mx);   // correctly rounded division
    const uint64_t qi = static_cast<uint64_t>(floor(ldexp(r, K)));
    q[i] = qi;
    acc += qi;
  }
  acc = wave_sum_u64(acc);
  if (lane == 0) ssum[wave] = acc;
  __syncthreads();
  if (tid == 0) {
    uint64_t C = 0;
    for (int k = 0; k < kPrepThreads / 64; ++k) C += ssum[k];
    st->flags = 0;
    st->total = C;
    for (int l = 0; l < lv.L; ++l) st->thr[l] = exact_threshold(lv.alpha[l], C);
  }
}

// Transpose values (M x p row-major) into key columns (p x M), and count the quantised
// weight of |v| < Delta_d per coefficient (exact integer sums, any order).  A workgroup takes
// `per` tiles of 32 rows and adds its sums to the totals once, so that a total is added to by 64
// workgroups or so (one addition per 32 rows spent 96 us on the contended atomics at M = 16384, p =
// 200, most of the pass); one tile where no tolerance is given and nothing is added (M = 33000,
// p = 40, one level: the call 125 us with 16 tiles, 103 with one).
constexpr int kKeyAdds = 64, kKeyTilesMax = 16;
inline int key_tiles(int M, int D) {
  return D > 0 ? std::min(kKeyTilesMax, std::max(1, (M + 31) / 32 / kKeyAdds)) : 1;
}

template <typename VT, typename KT, bool CONC>   // CONC: any tolerances
__global__ void sq_keys_kernel(const VT *__restrict__ vals, int M, int p, const uint64_t *__restrict__ q,
                               SqLevels lv, int per, KT *__restrict__ keys,
                               unsigned long long *__restrict__ inside) {
  __shared__ VT tile[32][33];
  const int j0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8 threads
  constexpr int ND = CONC ? kSqMaxLevels : 0;
  uint64_t in[4][CONC ? kSqMaxLevels : 1];                  // this thread's columns ty, ty + 8, ...
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int d = 0; d < ND; ++d) in[c][d] = 0;
  for (int it = 0; it < per; ++it) {
    const int i0 = (blockIdx.x * per + it) * 32;
    if (i0 >= M) break;
    __syncthreads();                                        // the previous tile has been read
    for (int r = ty; r < 32; r += 8) {
      const int i = i0 + r, j = j0 + tx;
      tile[r][tx] = (i < M && j < p) ? vals[(size_t)i * p + j] : VT(0);
    }
    __syncthreads();
    const int i = i0 + tx;
    const uint64_t qi = CONC && i < M ? q[i] : 0ull;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = j0 + ty + 8 * c;
      const VT v = tile[tx][ty + 8 * c];
      if (i < M && j < p) keys[(size_t)j * M + i] = key_of(v);
#pragma unroll
      for (int d = 0; d < ND; ++d)
        if (d < lv.D && fabs(static_cast<double>(v)) < lv.delta[d]) in[c][d] += qi;
    }
  }
  // lanes tx of one column share its sums
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int j = j0 + ty + 8 * c;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      if (d >= lv.D) continue;
      uint64_t s = in[c][d];
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o, 32);
      if (tx == 0 && s != 0 && j < p)
        atomicAdd(&inside[(size_t)d * p + j], static_cast<unsigned long long>(s));
    }
  }
}

// Weighted digit histograms of one pass.  grid = (chunks of kChunk values, p).
template <typename KT>
__global__ __launch_bounds__(kHistThreads) void sq_hist_kernel(const KT *__restrict__ keys, int M, int p,
                                                               const uint64_t *__restrict__ q, int L,
                                                               int shift, const SqSel *__restrict__ sel,
                                                               unsigned long long *__restrict__ hist) {
  __shared__ unsigned long long h[kSqMaxLevels][kBuckets];
  const int j = blockIdx.y;
  const int tid = threadIdx.x;
  for (int k = tid; k < L * kBuckets; k += kHistThreads) h[k / kBuckets][k % kBuckets] = 0ull;
  __syncthreads();
  KT pre[kSqMaxLevels];
  for (int l = 0; l < L; ++l) pre[l] = static_cast<KT>(sel[(size_t)j * kSqMaxLevels + l].prefix);
  const int hi_shift = shift + 8;   // bits above the current digit
  const KT *kc = keys + (size_t)j * M;
  const int b0 = blockIdx.x * kChunk, b1 = min(M, b0 + kChunk);
  for (int i = b0 + tid; i < b1; i += kHistThreads) {
    const KT k = kc[i];
    const uint64_t w = q[i];
    if (w == 0) continue;
    const int dig = static_cast<int>((k >> shift) & 0xff);
    const KT hi = (hi_shift >= static_cast<int>(8 * sizeof(KT))) ? KT(0) : (k >> hi_shift);
    for (int l = 0; l < L; ++l)
      if (hi == pre[l]) atomicAdd(&h[l][dig], static_cast<unsigned long long>(w));
  }
  __syncthreads();
  for (int k = tid; k < L * kBuckets; k += kHistThreads) {
    const unsigned long long v = h[k / kBuckets][k % kBuckets];
    if (v) atomicAdd(&hist[((size_t)j * kSqMaxLevels + k / kBuckets) * kBuckets + k % kBuckets], v);
  }
}

// Pick each (coefficient, level)'s digit: the bucket where below + cumulative weight
// reaches the threshold; clears the histogram for the next pass.  One wave per pair.
template <typename KT>
__global__ void sq_select_kernel(int p, int L, int last, const SqState *__restrict__ st,
                                 SqSel *__restrict__ sel, unsigned long long *__restrict__ hist,
                                 double *__restrict__ quant) {
  const int lane = threadIdx.x & 63;
  const int pair = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (pair >= p * L) return;
  const int j = pair / L, l = pair % L;
  SqSel &s = sel[(size_t)j * kSqMaxLevels + l];
  unsigned long long *hb = hist + ((size_t)j * kSqMaxLevels + l) * kBuckets;
  // 4 buckets per lane, in bucket order
  uint64_t c[4], loc = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    c[k] = hb[lane * 4 + k];
    loc += c[k];
  }
  // exclusive scan of the lanes' sums
  uint64_t incl = loc;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t v = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += v;
  }
  const uint64_t excl = incl - loc;
  const uint64_t need = st->thr[l] - s.below;   // > 0 and <= the weight still in range
  int found = -1;
  uint64_t below_b = 0;
  uint64_t run = excl;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (found < 0 && run + c[k] >= need) {
      found = lane * 4 + k;
      below_b = run;
    }
    run += c[k];
  }
  // the first lane holding the crossing bucket decides
  const unsigned long long ball = __ballot(found >= 0);
  const int src = ball ? __ffsll(static_cast<long long>(ball)) - 1 : 63;
  int b = __shfl(found, src, kWave);
  const uint64_t bb = __shfl(below_b, src, kWave);
  if (b < 0) b = kBuckets - 1;   // unreachable for valid weights (the range holds the target)
#pragma unroll
  for (int k = 0; k < 4; ++k) hb[lane * 4 + k] = 0ull;
  if (lane == 0) {
    s.prefix = (s.prefix << 8) | static_cast<uint64_t>(b);
    s.below += bb;
    if (last) quant[(size_t)l * p + j] = value_of_key(static_cast<KT>(s.prefix));
  }
}

__global__ void sq_conc_kernel(int p, int D, const SqState *__restrict__ st,
                               const unsigned long long *__restrict__ inside, double *__restrict__ conc) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= p * D) return;
  conc[k] = 1.0 - static_cast<double>(inside[k]) / static_cast<double>(st->total);
}

__global__ void sq_init_kernel(int p, SqSel *__restrict__ sel, unsigned long long *__restrict__ inside, int D) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < p * kSqMaxLevels) {
    sel[k].prefix = 0;
    sel[k].below = 0;
  }
  if (k < p * D) inside[k] = 0ull;
}

// Pooled weights of the c-marginal mixture: w_ti = exp(log_z_t - max_s log_z_s + logW_ti),
// and the posterior over the scale p_t = exp(log_z_t - logsumexp(log_z)).
__global__ void sq_mixture_weights_kernel(const double *__restrict__ log_z, int T, int N,
                                          const double *__restrict__ logW, double *__restrict__ w,
                                          double *__restrict__ scale_post) {
  __shared__ double s_m, s_l;
  if (threadIdx.x == 0) {
    double m = -INFINITY;
    for (int t = 0; t < T; ++t) m = fmax(m, log_z[t]);
    double e = 0.0;
    for (int t = 0; t < T; ++t) e += exp(log_z[t] - m);
    s_m = m;
    s_l = m + log(e);
  }
  __syncthreads();
  const size_t tot = (size_t)T * N;
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < tot; k += (size_t)gridDim.x * blockDim.x) {
    const int t = static_cast<int>(k / N);
    w[k] = exp((log_z[t] - s_m) + logW[k]);
  }
  if (blockIdx.x == 0 && scale_post)
    for (int t = threadIdx.x; t < T; t += blockDim.x) scale_post[t] = exp(log_z[t] - s_l);
}

}  // namespace

int sq_key_bytes(bool f64) { return f64 ? 8 : 4; }

template <typename VT, typename KT, int EPT, bool KEYS>
static hipError_t launch_column(const SqArgs &a, int K, hipStream_t s) {
  auto kern = sq_column_kernel<VT, KT, EPT, KEYS>;
  const size_t lds = sizeof(unsigned long long) * kColStride * (size_t)a.lv.L;
  static OncePerDevice once;
  const hipError_t e = raise_lds_limit(once, kern, sizeof(unsigned long long) * kColStride * kSqMaxLevels);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(8 * ((a.p + 7) / 8)), dim3(kColThreads), lds, s,
                     reinterpret_cast<const VT *>(a.values), reinterpret_cast<const KT *>(a.keys), a.M, a.p, a.w, a.log_weights, K, a.q, a.lv, a.flag, a.quant,
                     a.conc);
  return hipGetLastError();
}

template <typename VT, typename KT>
static hipError_t launch_columns(const SqArgs &a, int K, hipStream_t s) {
  const int ept = (a.M + kColThreads - 1) / kColThreads;
  if (ept <= 1) return launch_column<VT, KT, 1, false>(a, K, s);
  if (ept <= 2) return launch_column<VT, KT, 2, false>(a, K, s);
  if (ept <= 4) return launch_column<VT, KT, 4, false>(a, K, s);
  const bool keys = sq_key_columns(a.f64, a.M, a.p);
  const int tiles = keys ? ((a.M + 63) / 64) * ((a.p + 63) / 64) : 0;
  hipLaunchKernelGGL((sq_prep_kernel<VT, KT>), dim3(ept + tiles), dim3(kColThreads), 0, s,
                     reinterpret_cast<const VT *>(a.values), a.M, a.p, a.w, a.log_weights, K, ept, a.q,
                     reinterpret_cast<KT *>(a.keys), a.flag);
  if (ept <= 8) return keys ? launch_column<VT, KT, 8, true>(a, K, s) : launch_column<VT, KT, 8, false>(a, K, s);
  if (ept <= 16) return keys ? launch_column<VT, KT, 16, true>(a, K, s) : launch_column<VT, KT, 16, false>(a, K, s);
  if constexpr (sizeof(VT) == 4)
    return keys ? launch_column<VT, KT, 32, true>(a, K, s) : launch_column<VT, KT, 32, false>(a, K, s);
  return hipErrorInvalidValue;
}

// Whether the column form reads transposed key columns: rows longer than a cache line, of
// which every workgroup would fetch a line per row for 4 or 8 bytes (measured at M = 16384,
// p = 200 FP32: 19 us for the strided read in the column kernel).
bool sq_key_columns(bool f64, long long M, int p) {
  return M > kColInline * kColThreads && (long long)p * sq_key_bytes(f64) > 128;
}

// Whether one workgroup per coefficient summarises the set: it has to fit the registers, and
// not to be of few values and many coefficients, where a workgroup costs the same for each
// coefficient and the passes over all of them next to nothing.  The line is fitted to 592 calls
// measured in both forms (M = 1 .. 16000, p = 5 .. 20000, 1 to 8 levels; 0.1 % slower than the
// better form on average): M = 100 FP32, 8 levels and tolerances, p = 1000 85 us against 110 of
// the passes, p = 8000 495 against 321; M = 1000, p = 20000, 3 levels 512 against 613.
bool sq_one_launch(bool f64, long long M, int p, int L) {
  if (M > (long long)kColThreads * col_ept_max(f64)) return false;
  return p * (1.0 + 0.37 * L - (0.34 + 0.68 * L) * 1e-3 * static_cast<double>(M)) <= 6500.0 || p > 65535;
}

hipError_t launch_weighted_summaries(const SqArgs &a, hipStream_t s) {
  const int M = a.M, p = a.p, L = a.lv.L, D = a.lv.D;
  const int K = 63 - ceil_log2_ll(M);
  if (sq_one_launch(a.f64, M, p, L))
    return a.f64 ? launch_columns<double, uint64_t>(a, K, s) : launch_columns<float, uint32_t>(a, K, s);
  hipLaunchKernelGGL(sq_init_kernel, dim3((p * kSqMaxLevels + 255) / 256), dim3(256), 0, s, p, a.sel,
                     a.inside, D);
  hipLaunchKernelGGL(sq_prepare_kernel, dim3(1), dim3(kPrepThreads), 0, s, a.w, M, a.log_weights, K, a.lv, a.q,
                     a.st);
  const int per = key_tiles(M, D);
  const dim3 tg((M + 32 * per - 1) / (32 * per), (p + 31) / 32);
  auto keys = [&](auto kern, auto *values, auto *out) {
    hipLaunchKernelGGL(kern, tg, dim3(256), 0, s, values, M, p, a.q, a.lv, per, out, a.inside);
  };
  if (a.f64) {
    const auto *v = static_cast<const double *>(a.values);
    auto *out = static_cast<uint64_t *>(a.keys);
    if (D > 0) keys(sq_keys_kernel<double, uint64_t, true>, v, out);
    else keys(sq_keys_kernel<double, uint64_t, false>, v, out);
  } else {
    const auto *v = static_cast<const float *>(a.values);
    auto *out = static_cast<uint32_t *>(a.keys);
    if (D > 0) keys(sq_keys_kernel<float, uint32_t, true>, v, out);
    else keys(sq_keys_kernel<float, uint32_t, false>, v, out);
  }
  if (L > 0) {
    const int bits = a.f64 ? 64 : 32;
    const dim3 hg((M + kChunk - 1) / kChunk, p);
    const int sgrid = (p * L + 3) / 4;
    for (int shift = bits - 8; shift >= 0; shift -= 8) {
      const int last = shift == 0;
      if (a.f64) {
        hipLaunchKernelGGL((sq_hist_kernel<uint64_t>), hg, dim3(kHistThreads), 0, s,
                           reinterpret_cast<const uint64_t *>(a.keys), M, p, a.q, L, shift, a.sel, a.hist);
        hipLaunchKernelGGL((sq_select_kernel<uint64_t>), dim3(sgrid), dim3(256), 0, s, p, L, last, a.st, a.sel,
                           a.hist, a.quant);
      } else {
        hipLaunchKernelGGL((sq_hist_kernel<uint32_t>), hg, dim3(kHistThreads), 0, s,
                           reinterpret_cast<const uint32_t *>(a.keys), M, p, a.q, L, shift, a.sel, a.hist);
        hipLaunchKernelGGL((sq_select_kernel<uint32_t>), dim3(sgrid), dim3(256), 0, s, p, L, last, a.st, a.sel,
                           a.hist, a.quant);
      }
    }
  }
  if (D > 0)
    hipLaunchKernelGGL(sq_conc_kernel, dim3((p * D + 255) / 256), dim3(256), 0, s, p, D, a.st, a.inside, a.conc);
  return hipGetLastError();
}

hipError_t launch_mixture_weights(const double *log_z, int T, int N, const double *logW, double *w,
                                  double *scale_post, hipStream_t s) {
  const size_t tot = (size_t)T * N;
  const int grid = static_cast<int>(std::min<size_t>((tot + 255) / 256, 4096));
  hipLaunchKernelGGL(sq_mixture_weights_kernel, dim3(grid), dim3(256), 0, s, log_z, T, N, logW, w, scale_post);
  return hipGetLastError();
}

}  // namespace spa
