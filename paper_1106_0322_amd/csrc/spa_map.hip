// MAP estimates under the Gt(a, c) prior by EM (Section 2.1) and the MAP path of
// Section 4.1, on the GPU, in FP64.
//
// EM: E step w_j = (a+1)/(a c + |beta_j|) (1/c for the double exponential); M step: the
// weighted-L1 logistic problem by cyclic coordinate ascent with the curvature bound n/4,
// beta_j <- S(beta_j + 4 g_j / n, 4 w_j / n), g_j = sum_k (y_k - sigma(eta_k)) X_std,kj.
//
// One workgroup of one to eight wave64s per start point.  Thread t of T holds individuals t,
// t+T, ...: E_k = exp(-eta_k) and the residual u_k = y_k - sigma(eta_k) = y_k - 1 / (1 + E_k) in
// registers (E = +inf and y = 0 in padded ones: u = -2^-1000; an E that is not a number counts as
// sigma = 0).  A column of standardised genotypes is x = (c - mu_j)/s_j, c = 0, 1, 2, so
//   g_j = (sum_k (c_kj - mu_j) u_k) / s_j,
// with c - mu formed per individual by one FMA: the genotype's two bits shifted to the exponent's
// lowest bits are the double c 2^-1022, so that a column costs two integer instructions and two
// FMAs per individual, no table (the standardised values read from LDS, 8 bytes per individual
// and column, were the longest part of a sweep over zero coefficients).  Subtracting mu from the
// sums instead, sum c u - mu sum u, would save one FMA but cancels where sum u is large (unbalanced
// labels), and 1 / s_j enlarges what is left (rare markers): errors of the mode 1e-14 against
// 1e-16 at 90 % cases and an allele frequency of 0.0005.  A move
// beta_j += delta multiplies every E_k by one of three constants exp(-delta x_c): lanes 0..3 of
// each wave put them in a table in LDS (1 for padded individuals), then per individual one table
// read, one multiply and a reciprocal (hardware estimate refined by one Newton step).  A thread's
// genotypes of a column are two-bit fields of one word (two above 16 individuals): one load per
// thread and column.  As in the oracle, eta is recomputed from the coefficients at the start of every
// coordinate sweep, which also bounds the rounding of the products to one sweep; zero
// coefficients add nothing and are passed over.
//
// Columns that need no look.  A move of delta in any coefficient changes u_k by at most
// |delta x_k| / 4, so the vector u by at most |delta| sqrt(n) / 4 in norm, and 4 g_j / n of any
// other column (of norm sqrt(n)) by at most |delta|.  So a zero coefficient whose |4 g_j / n|,
// when it was last formed, plus the path length sum |delta| of the moves since stays below its
// threshold 4 w_j / n is certain to stay zero: its update is decided without forming g_j.  What
// the fresh predictor of a sweep changes in u (rounding, or products that had left the range of
// a double) is measured and counts as path.  The path is rounded up at every addition and starts
// again from zero at each E step (what has been walked is added to the columns' |4 g_j / n|), so
// that moves far below it still count; kMargin covers the rounding of g_j and of u; a NaN or an
// infinity fails the comparison, so its columns are looked at.  Close to a mode the moves are
// small and nearly all zero coefficients are decided so.
//
// Runs of columns.  An update that leaves beta_j as it was does not change u, so the gradients
// of the columns after it are those of the same u.  Of the columns that need a look, one, two,
// four or eight (by how many zero coefficients come first: a coefficient that is zero usually
// stays so) are reduced together: one barrier and one reduction latency for the run.
// The reduction of 2, 4 or 8 values over a wave halves the number of values at each of its
// first steps; after the barrier the lane that holds a column's coefficient decides it, and a
// ballot finds the first that moves.  The columns before it are done, the gradients after it
// are dropped.  So every update is that of the sequential sweep.  Non-zero columns that come
// first are taken one after the other by a shorter path (uniform constants, one sum, no
// ballots; with more than 12 individuals per thread its registers would spill and the general
// path is the faster one).
//
// Lanes hold columns: a block of 64 columns (32 where a thread has two words per column) has
// its coefficients, thresholds and constants in the lanes of every wave, the same in all, and
// goes back to LDS at the block's end.  The words of a column stay in LDS: all columns where
// they fit, else one slot per column of a block, filled on demand (the support's columns are
// the ones that are asked for, sweep after sweep).
//
// What bounds it: a chain of coordinate updates, each a reduction and a barrier; the start
// points' workgroups are all the parallelism there is.  Two starts, 10 x 5 sweeps, against one
// update per barrier in 512 threads with the standardised values in a table (ms):
//   n = 5000, p = 200: 13 of 400 coefficients non-zero 10.66 -> 3.07, 368 15.3 -> 14.1, all
//   15.4 -> 14.3; n = 10000, p = 100: 18 of 200 12.8 -> 3.0, all 16.5 -> 12.4; n = 1000, p = 100:
//   1 of 200 2.94 -> 0.47, all 3.91 -> 3.66; n = 500, p = 50: none 1.22 -> 0.14, 66 of 100 1.58 ->
//   1.25, all 1.72 -> 1.58; n = 120, p = 50: none 1.21 -> 0.085, all 1.72 -> 1.24.
// With every coefficient non-zero nothing is passed over: what counts is the latency of an
// update, that is the table reads and the chains of E and u side by side (see move) and the
// predictor's loads ahead of their use.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "spa_common.hpp"
#include "spa_internal.hpp"
#include "spa_lanes.hpp"
#include "spa_map.hpp"

namespace spa {

namespace {

constexpr int kMapMaxThreads = 512;
// Words of two-bit genotypes per thread and column for R individuals per thread.
constexpr int map_words(int R) { return R <= 16 ? 1 : 2; }
// Threads of a start point's workgroup and individuals per thread.  Fewer waves make the
// reduction and the barrier of an update cheaper, fewer individuals per thread its vector
// work: one wave up to four per thread, then one per SIMD, then two (n = 500, p = 50, 50
// sweeps from two starts: every coefficient non-zero 1.75 ms in 128 threads of 4, 1.57 ms in 256
// of 2; none 0.118 and 0.102 ms).
inline int map_threads(int n_pad) { return n_pad <= 256 ? 64 : n_pad <= 1024 ? 256 : 512; }
inline int map_rows(int n_pad) {
  const int t = map_threads(n_pad), R = (n_pad + t - 1) / t;
  return R <= 1 ? 1 : R <= 2 ? 2 : R <= 4 ? 4 : R <= 6 ? 6 : R <= 8 ? 8 : R <= 10 ? 10 : R <= 12 ? 12 : R <= 16 ? 16 : 20;
}

// 1 / (1 + e) for e >= 0 (2^-1000 for +inf and for NaN): hardware reciprocal of inv1p_arg (relative
// error near 2^-23) and one Newton step (error near 2^-46, squared by the step).
__device__ __forceinline__ double inv1p_arg(double e) { return fmin(1.0 + e, 0x1p1000); }
__device__ __forceinline__ double inv1p(double e) {
  const double d = inv1p_arg(e);
  double r = __builtin_amdgcn_rcp(d);
  const double q = fma(-d, r, 1.0);
  return fma(r, q, r);
}

// c - mu for the genotype c of a thread's r-th individual (2 bits each), rounded once; and c.
template <int R>
__device__ __forceinline__ double centred_at(const uint32_t (&w)[map_words(R)], int r, double mu) {
  const int at = 2 * (r % 16);
  const uint32_t f = at <= 20 ? w[r / 16] << (20 - at) : w[r / 16] >> (at - 20);
  return fma(__hiloint2double(static_cast<int>(f & 0x300000u), 0), 0x1p1022, -mu);   // c 2^-1022
}
template <int R>
__device__ __forceinline__ int code_at(const uint32_t (&w)[map_words(R)], int r) {
  return static_cast<int>((w[r / 16] >> (2 * (r % 16))) & 3u);
}

// Label of the value a lane ends with in wave_sums: lane bits x0..x3 give
// (x0 ^ x2) + 2 (x1 ^ x2) + 4 (x2 ^ x3), which changes in its first, second and third bit
// across the partners of the first three steps and not across those of the steps after it.
// Lanes 0..7 hold the eight labels once each.
__device__ __forceinline__ int lane_label() {
  const int x = threadIdx.x;
  return ((x ^ (x >> 2)) & 1) | (((x >> 1) ^ (x >> 2)) & 1) << 1 | (((x >> 2) ^ (x >> 3)) & 1) << 2;
}

// Sums of V values over the wave: the lane gets that of value (label mod V).  At a halving
// step a lane keeps one of two values and adds its partner's copy of it.
template <int V>
__device__ __forceinline__ double wave_sums(const double (&v)[V], int label) {
  static_assert(V == 2 || V == 4 || V == 8, "one to three halving steps");
  double a[V / 2];
#pragma unroll
  for (int i = 0; i < V / 2; ++i) {                                   // partner i ^ 1
    const double keep = (label & 1) ? v[2 * i + 1] : v[2 * i], send = (label & 1) ? v[2 * i] : v[2 * i + 1];
    a[i] = keep + dpp_move_f64<0xB1>(send);
  }
  double b[V >= 4 ? V / 4 : 1];
  if constexpr (V >= 4) {
#pragma unroll
    for (int i = 0; i < V / 4; ++i) {                                 // partner i ^ 2
      const double keep = (label & 2) ? a[2 * i + 1] : a[2 * i], send = (label & 2) ? a[2 * i] : a[2 * i + 1];
      b[i] = keep + dpp_move_f64<0x4E>(send);
    }
  } else {
    b[0] = a[0] + dpp_move_f64<0x4E>(a[0]);
  }
  double c;
  if constexpr (V == 8) {                                             // partner i ^ 7
    const double keep = (label & 4) ? b[1] : b[0], send = (label & 4) ? b[0] : b[1];
    c = keep + dpp_move_f64<0x141>(send);
  } else {
    c = b[0] + dpp_move_f64<0x141>(b[0]);
  }
  c += dpp_move_f64<0x140>(c);                                        // partner i ^ 15
  c += swizzle_xor16_f64(c);
  c += __shfl_xor(c, 32, kWave);
  return c;
}

// What |4 g_j / n| may be off by within a sweep.  Its own sum, at most 20 terms per thread and 9
// levels: 32 eps 4 mean |x u| <= 1.5e-14, eps = 2^-53, as mean |x u| <= 1 whatever the allele
// frequency (mean x^2 = 1).  E and u, each rounded by less than 3 eps per move: 12 eps a move,
// 7e-13 in the at most 512 of a sweep (the next predictor measures and counts what there was).
constexpr double kMargin = 1e-12;
// a + d for a, d >= 0, not below the sum.
__device__ __forceinline__ double add_up(double a, double d) {
  const double s = a + d;
  return fma(s, 0x1p-51, s);
}
// Columns per block (and slots, where the columns do not all fit), and LDS bytes of the slots.
constexpr int map_block(int R) { return map_words(R) == 1 ? 64 : 32; }
constexpr size_t kMapSlotBytes = size_t(128) << 10;
inline bool map_resident(int NT, int R, int p) { return (size_t)p * NT * map_words(R) * 4 <= kMapSlotBytes; }

template <typename IT, int NT, int R>
__global__ __launch_bounds__(NT) void map_em_kernel(MapArgs a, int resident) {
  constexpr int WN = map_words(R), NW = NT / 64, BS = map_block(R);
  extern __shared__ __align__(16) uint32_t slots[];   // [column or slot][WN][NT]
  __shared__ double bl[kMapMaxP], tl[kMapMaxP], gl[kMapMaxP], pl[kMapMaxP], mul[kMapMaxP], isl[kMapMaxP];
  __shared__ __align__(16) double part[2][NW][8];
  __shared__ double red[NW];
  __shared__ double cltab[NW][4];          // per wave: exp(-delta x_c), 1 for code 3
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = blockIdx.x;                      // start point
  const int n = a.n, p = a.p;
  const IT *b0 = reinterpret_cast<const IT *>(a.beta0) + (size_t)s * p;
  const Prior pr = a.prior;
  const double inv_n4 = 4.0 / static_cast<double>(n);
  const int label = lane_label();

  for (int j = tid; j < p; j += NT) {
    bl[j] = static_cast<double>(b0[j]);
    gl[j] = INFINITY;                            // |4 g_j / n| when last formed, ...
    pl[j] = 0.0;                                 // ... and the path length then
    mul[j] = a.mu[j];
    isl[j] = a.inv_s[j];
  }
  double yk[R];                                  // labels of individuals tid + NT r, 0 in padded ones
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = tid + NT * r;
    yk[r] = k < n && a.y[k] ? 1.0 : 0.0;
  }
  // one column's words of this wave's threads -> a slot
  auto fill = [&](const int c, const int slot) {
#pragma unroll
    for (int q = 0; q < WN; ++q)
      __builtin_amdgcn_global_load_lds(a.codes + ((size_t)c * WN + q) * NT + tid, slots + (slot * WN + q) * NT + wave * 64, 4,
                                       0, 0);
  };
  if (resident) {
    for (int c = 0; c < p; ++c) fill(c, c);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();
  double E[R], u[R] = {};
  // eta_k from the coefficients (the sweep's fresh linear predictor), non-zero columns only, in
  // groups of up to four of a block of 64, the next group's words in flight
  auto predictor = [&](double (&eta)[R]) {
    constexpr int B = 4;
    double bsl = 0.0, mul64 = 0.0;               // lanes: b / s and mu of 64 columns
#pragma unroll
    for (int r = 0; r < R; ++r) eta[r] = 0.0;
    int base = -64;
    unsigned long long left = 0;
    auto group = [&](double (&bs)[B], double (&m)[B], uint32_t (&w)[B][WN]) -> bool {
      while (left == 0) {
        base += 64;
        if (base >= p) return false;
        const int j = min(base + lane, p - 1);
        const double bj = base + lane < p ? bl[j] : 0.0;
        bsl = bj * isl[j];
        mul64 = mul[j];
        left = __ballot(bj != 0.0);
      }
      int l = 0;
#pragma unroll
      for (int q = 0; q < B; ++q) {              // absent columns repeat the last one, times zero
        const bool there = left != 0;
        l = there ? __builtin_ctzll(left) : l;
        left &= left - 1;
        bs[q] = there ? read_lane_f64(bsl, l) : 0.0;
        m[q] = read_lane_f64(mul64, l);
        const uint32_t *col = a.codes + (size_t)(base + l) * WN * NT + tid;
#pragma unroll
        for (int k = 0; k < WN; ++k) w[q][k] = col[k * NT];
      }
      return true;
    };
    double bs[B], bn[B], m[B], mn[B];
    uint32_t w[B][WN], wn[B][WN];
    bool more = group(bs, m, w);
    while (more) {
      more = group(bn, mn, wn);
#pragma unroll
      for (int q = 0; q < B; ++q)
#pragma unroll
        for (int r = 0; r < R; ++r) eta[r] = fma(bs[q], centred_at<R>(w[q], r, m[q]), eta[r]);
#pragma unroll
      for (int q = 0; q < B; ++q) {
        bs[q] = bn[q];
        m[q] = mn[q];
#pragma unroll
        for (int k = 0; k < WN; ++k) w[q][k] = wn[q][k];
      }
    }
  };

  // one wave per SIMD and few individuals per thread: a move's factors are selected from registers
  constexpr bool SELECT = R <= 4 && NW <= 4;
  // the standardised value of code 0, 1, 2 in lanes 0..2 (SELECT: of each four), zero in lane 3
  auto code_values = [&](const double cmu, const double cis) {
    const int code = SELECT ? lane & 3 : lane;
    return code < 3 ? (static_cast<double>(code) - cmu) * cis : 0.0;
  };
  // a coefficient moves by delta (the same in every lane); xc: its column's code_values
  auto move = [&](const double delta, const double xc, const uint32_t (&wd)[WN]) {
    // SELECT: the factors broadcast in each four lanes and selected (padded individuals: any of
    // them, E is infinite); n = 1000, p = 100, every coefficient non-zero, 0.82 -> 0.73 us per
    // update.  Else lanes 0..3 put them in the wave's
    // table (1 for code 3; n = 2000: 1.00 us, selected 1.08); a wave's LDS accesses are processed in
    // order, and the wave barrier keeps the compiler from moving the table reads above the write
    double f0 = 0.0, f1 = 0.0, f2 = 0.0;
    if constexpr (SELECT) {
      const double factor = exp(-delta * xc);
      f0 = dpp_move_f64<0x00>(factor);
      f1 = dpp_move_f64<0x55>(factor);
      f2 = dpp_move_f64<0xAA>(factor);
    } else {
      if (lane < 4) cltab[wave][lane] = exp(-delta * xc);
      __builtin_amdgcn_wave_barrier();
    }
    // in stages over U individuals: the table reads in flight together and the chains of E and u
    // side by side (left alone, the scheduler takes the individuals one after the other, a wait
    // for LDS each: n = 1000, p = 100, every coefficient non-zero, 0.91 us per update)
    constexpr int U = R <= 10 ? R : R / 2;
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += U) {
      double d[U], q[U];
#pragma unroll
      for (int r = 0; r < U; ++r) {
        if constexpr (SELECT) {
          const uint32_t at = wd[0] >> (2 * (r0 + r));
          d[r] = (at & 2u) ? f2 : (at & 1u) ? f1 : f0;
        } else {
          d[r] = cltab[wave][code_at<R>(wd, r0 + r)];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < U; ++r) {
        E[r0 + r] *= d[r];
        d[r] = inv1p_arg(E[r0 + r]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < U; ++r) q[r] = __builtin_amdgcn_rcp(d[r]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < U; ++r) d[r] = fma(-d[r], q[r], 1.0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < U; ++r) u[r0 + r] = yk[r0 + r] - fma(q[r], d[r], q[r]);
    }
  };
  int parity = 0, tag = -1;                      // tag: the block whose column this lane's slot holds
  double path = 0.0;                             // sum of |delta| since the E step (uniform)
  for (int it = 0; it < a.outer; ++it) {
    for (int sw = 0; sw < a.inner; ++sw) {
      __syncthreads();                           // the previous sweep's coefficients
      if (sw == 0) {                             // E step: |4 w_j / n| thresholds of this M step
        for (int j = tid; j < p; j += NT) {
          tl[j] = inv_n4 * (pr.inf ? 1.0 / pr.lam : (pr.a + 1.0) / (pr.a * pr.lam + fabs(bl[j])));
          gl[j] = add_up(gl[j], path - pl[j]);
          pl[j] = 0.0;
        }
        path = 0.0;
        __syncthreads();
      }
      {
        double eta[R], drift = 0.0;
        predictor(eta);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double old = u[r];
          E[r] = tid + NT * r < n ? exp(-eta[r]) : INFINITY;
          u[r] = yk[r] - inv1p(E[r]);
          drift += fabs(u[r] - old);
        }
        // by how much the products' residuals were off counts as path: |4 dg_j / n| <= 4 sum |du|
        drift = wave_sum(drift);
        if constexpr (NW > 1) {
          if (lane == 0) red[wave] = drift;
          __syncthreads();
          drift = red[0];
#pragma unroll
          for (int k = 1; k < NW; ++k) drift += red[k];
        }
        if (it + sw > 0) path = add_up(path, 4.0 * drift);   // (the first one starts from nothing)
      }
      for (int blk = 0; blk * BS < p; ++blk) {
        const int c0 = blk * BS, col = min(c0 + lane, p - 1);
        const bool in = lane < BS && c0 + lane < p;
        double b = bl[col], g4 = gl[col], at4 = pl[col];
        const double mu = mul[col], is = isl[col], thr = tl[col];
        int pos = 0;                             // columns of the block before this lane are done
        const int slot0 = resident ? c0 : 0;
        bool look = false;
        uint32_t w0[WN];
        // the block's remaining candidates, their words in LDS and the first one's words on their way
        auto scan = [&]() -> unsigned long long {
          look = in && lane >= pos && !(b == 0.0 && add_up(g4, path - at4) + kMargin <= thr);
          const unsigned long long c = __ballot(look);
          if (c == 0) return c;
          if (!resident) {                       // words that are not in their slot: one wait for all
            unsigned long long miss = __ballot(look && tag != blk);
            if (miss) {
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slots' last reads
              if ((miss >> lane) & 1) tag = blk;
              while (miss) {
                const int l = __builtin_ctzll(miss);
                miss &= miss - 1;
                fill(c0 + l, l);
              }
              asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
          }
#pragma unroll
          for (int k = 0; k < WN; ++k) w0[k] = slots[((slot0 + __builtin_ctzll(c)) * WN + k) * NT + tid];
          return c;
        };
        unsigned long long cand = scan();
        while (cand) {
          // zero coefficients that come first among the candidates
          const unsigned long long nzc = __ballot(look && b != 0.0);
          if (R <= 12 && (nzc & cand & (0ull - cand))) {   // non-zero columns first: one after the other
            int f = __builtin_ctzll(cand);
            double g4f = g4, at4f = at4, bf = b;
            for (;;) {
              uint32_t w[WN];
#pragma unroll
              for (int k = 0; k < WN; ++k) w[k] = w0[k];
              const bool more = f < 63 && ((nzc >> (f + 1)) & 1);
              if (more) {
#pragma unroll
                for (int k = 0; k < WN; ++k) w0[k] = slots[((slot0 + f + 1) * WN + k) * NT + tid];
              }
              const double fmu = read_lane_f64(mu, f), fis = read_lane_f64(is, f), fthr = read_lane_f64(thr, f);
              const double fb = read_lane_f64(b, f), scale = inv_n4 * fis;
              double fx = code_values(fmu, fis);
              if constexpr (SELECT) asm volatile("" : "+v"(fx));   // formed here, not after the decision
              double g = 0.0;
#pragma unroll
              for (int r = 0; r < R; ++r) g = fma(centred_at<R>(w, r, fmu), u[r], g);
              double t;
              if constexpr (NW == 1) {
                t = wave_total_f64(g);
              } else {
                g = wave_last_f64(g);
                if (lane == 63) part[parity][wave][0] = g;
                __syncthreads();
                t = part[parity][lane & (NW - 1)][0];
                t += dpp_move_f64<0xB1>(t);
                if constexpr (NW >= 4) t += dpp_move_f64<0x4E>(t);
                if constexpr (NW == 8) t += dpp_move_f64<0x141>(t);
                parity ^= 1;
              }
              const double z = fma(scale, t, fb);   // t, and so delta, is the same in every lane
              const double nb = z > fthr ? z - fthr : (z < -fthr ? z + fthr : 0.0);
              const double delta = nb - fb;
              if (lane == f) {
                g4f = fabs(scale * t);
                at4f = path;
                bf = nb;
              }
              if (__any(delta != 0.0)) {
                path = add_up(path, fabs(delta));
                move(delta, fx, w);
              }
              if (!more) break;
              ++f;
            }
            g4 = g4f;
            at4 = at4f;
            b = bf;
            pos = f + 1;
            cand = scan();
            continue;
          }
          const int zeros = __popcll(nzc ? cand & ((nzc & (0ull - nzc)) - 1) : cand);
          const int rank = __popcll(cand & ((1ull << lane) - 1));   // a candidate's place
          double t = 0.0;
          auto sums = [&](auto v_c) {
            constexpr int V = decltype(v_c)::value;
            uint32_t w[V][WN];
            double m[V], g[V];
            unsigned long long c = cand;
#pragma unroll
            for (int q = 0; q < V; ++q) {        // absent candidates repeat the last one, unused
              const int l = __builtin_ctzll(c);
              if (c & (c - 1)) c &= c - 1;
              m[q] = read_lane_f64(mu, l);
              g[q] = 0.0;
#pragma unroll
              for (int k = 0; k < WN; ++k) w[q][k] = q == 0 ? w0[k] : slots[((slot0 + l) * WN + k) * NT + tid];
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
              for (int q = 0; q < V; ++q) g[q] = fma(centred_at<R>(w[q], r, m[q]), u[r], g[q]);
            const int want = min(rank, V - 1);   // the value this lane's column takes
            double x;
            if constexpr (V == 1) x = wave_total_f64(g[0]);
            else x = wave_sums<V>(g, label);
            if constexpr (NW > 1) {
              if (lane < 8 && label < V) part[parity][wave][label] = x;
              __syncthreads();
              // lane 8 q + k: value q of wave k mod NW; the same sums in the same order in every wave
              double z = part[parity][lane & (NW - 1)][lane >> 3];
              z += dpp_move_f64<0xB1>(z);                             // partner k ^ 1
              if constexpr (NW >= 4) z += dpp_move_f64<0x4E>(z);      // k ^ 2
              if constexpr (NW == 8) z += dpp_move_f64<0x141>(z);     // 7 - k
              t = V == 1 ? read_lane_f64(z, 0) : __shfl(z, 8 * want, kWave);
              parity ^= 1;
            } else {
              // from the lane of lanes 0..7 that holds the value
              const int x2 = (want >> 2) & 1;
              t = V == 1 ? x : __shfl(x, ((want ^ (x2 ? 3 : 0)) & 3) | x2 << 2, kWave);
            }
          };
          const int V = zeros == 0 ? 1 : zeros == 1 ? 2 : zeros <= 3 ? 4 : 8;
          if (V == 8)
            sums(std::integral_constant<int, 8>{});
          else if (V == 4)
            sums(std::integral_constant<int, 4>{});
          else if (V == 2 || R <= 12)            // (up to 12: a zero coefficient comes first)
            sums(std::integral_constant<int, 2>{});
          else
            sums(std::integral_constant<int, 1>{});
          const bool mine = look && rank < V;
          const double gs = inv_n4 * (t * is), z = b + gs;
          const double nb = z > thr ? z - thr : (z < -thr ? z + thr : 0.0);
          const double d = nb - b;
          const unsigned long long moved = __ballot(mine && d != 0.0), decided = __ballot(mine);
          // the last column that is done: the first that moves, or the run's last
          const int last = moved ? __builtin_ctzll(moved) : 63 - __builtin_clzll(decided);
          pos = last + 1;
          if (mine && lane <= last) {
            g4 = fabs(gs);
            at4 = path;
            b = nb;
          }
          const double delta = moved ? read_lane_f64(d, last) : 0.0;
          if (moved) path = add_up(path, fabs(delta));
          cand = scan();                         // its LDS reads run beside the move
          if (moved) {                           // uniform: column c0 + last moves by delta
            const double dmu = read_lane_f64(mu, last), dis = read_lane_f64(is, last);
            uint32_t wd[WN];
#pragma unroll
            for (int k = 0; k < WN; ++k) wd[k] = slots[((slot0 + last) * WN + k) * NT + tid];
            move(delta, code_values(dmu, dis), wd);
          }
        }
        if (wave == 0 && in) {                   // every wave holds the same values
          bl[col] = b;
          gl[col] = g4;
          pl[col] = at4;
        }
      }
    }
  }
  __syncthreads();
  // log posterior at the mode: sum_k [y eta - softplus(eta)] + sum_j log Gt(beta_j)
  double eta[R];
  predictor(eta);
  double acc = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = tid + NT * r;
    if (k < n) acc += yk[r] * eta[r] - (fmax(eta[r], 0.0) + log1p(exp(-fabs(eta[r]))));
  }
  for (int j = tid; j < p; j += NT) acc += gt_logpdf(bl[j], pr);
  acc = wave_sum(acc);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  if (tid == 0) {
    double lp = red[0];
    for (int w = 1; w < NW; ++w) lp += red[w];
    a.logpost[s] = lp;
  }
  for (int j = tid; j < p; j += NT) a.mode[(size_t)s * p + j] = bl[j];
}

// A thread's genotypes per column, two bits each (3 in padded individuals), for the EM kernel.
__global__ void map_cols_kernel(const uint8_t *__restrict__ X, int n, int p, int WN, int NT,
                                uint32_t *__restrict__ codes) {
  const size_t total = (size_t)p * WN * NT;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < total;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int t = static_cast<int>(idx % NT), q = static_cast<int>(idx / NT % WN);
    const int j = static_cast<int>(idx / NT / WN);
    uint32_t w = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int k = t + NT * (16 * q + r);
      w |= (k < n ? static_cast<uint32_t>(X[(size_t)k * p + j]) : 3u) << (2 * r);
    }
    codes[idx] = w;
  }
}

// Log posterior of every particle at scale lam and the first index of its maximum.
// One workgroup of 1024 threads; a wave per particle, particles strided.
template <typename IT>
__global__ __launch_bounds__(1024) void best_particle_kernel(const IT *__restrict__ beta, const double *__restrict__ ll,
                                                             int M, int p, Prior pr, int *__restrict__ best) {
  __shared__ double sv[16];
  __shared__ int si[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double bv = -INFINITY;
  int bi = 0x7fffffff;
  for (int i = wave; i < M; i += 16) {
    double lp = 0.0;
    for (int j = lane; j < p; j += 64) lp += gt_logpdf(static_cast<double>(beta[(size_t)i * p + j]), pr);
    lp = wave_sum(lp) + ll[i];
    if (lp > bv) {                               // strictly: keeps the first index of a tie
      bv = lp;
      bi = i;
    }
  }
  if (lane == 0) {
    sv[wave] = bv;
    si[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
    double v = sv[0];
    int idx = si[0];
    for (int w = 1; w < 16; ++w)
      if (sv[w] > v || (sv[w] == v && si[w] < idx)) {
        v = sv[w];
        idx = si[w];
      }
    best[0] = idx == 0x7fffffff ? 0 : idx;     // no finite density: the first particle
  }
}

// Gather the EM starts of one scale: the best particle, then (if any) the previous MAP.
template <typename IT>
__global__ void map_starts_kernel(const IT *__restrict__ beta, const int *__restrict__ best, int p,
                                  const double *__restrict__ prev, double *__restrict__ starts) {
  for (int j = threadIdx.x; j < p; j += blockDim.x) {
    starts[j] = static_cast<double>(beta[(size_t)best[0] * p + j]);
    if (prev) starts[p + j] = prev[j];
  }
}

// Keep the start whose mode has the higher posterior density (the first on ties).
__global__ void map_pick_kernel(const double *__restrict__ modes, const double *__restrict__ lp, int ns, int p,
                                double *__restrict__ out, double *__restrict__ out_lp) {
  int k = 0;
  for (int s = 1; s < ns; ++s)
    if (lp[s] > lp[k]) k = s;
  for (int j = threadIdx.x; j < p; j += blockDim.x) out[j] = modes[(size_t)k * p + j];
  if (threadIdx.x == 0) out_lp[0] = lp[k];
}

template <typename IT, int NT, int R>
hipError_t launch_em_r(const MapArgs &a, hipStream_t st) {
  auto kern = map_em_kernel<IT, NT, R>;
  const bool resident = map_resident(NT, R, a.p);
  const size_t column = (size_t)NT * map_words(R) * 4;
  const size_t lds = column * (resident ? a.p : map_block(R));
  static OncePerDevice once;
  const hipError_t e = raise_lds_limit(once, kern, kMapSlotBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.M), dim3(NT), lds, st, a, resident ? 1 : 0);
  return hipGetLastError();
}

template <typename IT>
hipError_t launch_em_t(const MapArgs &a, hipStream_t st) {
  const int R = map_rows(a.n_pad);
  switch (map_threads(a.n_pad)) {
    case 64:
      return R == 1 ? launch_em_r<IT, 64, 1>(a, st)
                    : R == 2 ? launch_em_r<IT, 64, 2>(a, st) : launch_em_r<IT, 64, 4>(a, st);
    case 256: return R == 2 ? launch_em_r<IT, 256, 2>(a, st) : launch_em_r<IT, 256, 4>(a, st);
  }
  switch (R) {
    case 4: return launch_em_r<IT, 512, 4>(a, st);
    case 6: return launch_em_r<IT, 512, 6>(a, st);
    case 8: return launch_em_r<IT, 512, 8>(a, st);
    case 10: return launch_em_r<IT, 512, 10>(a, st);
    case 12: return launch_em_r<IT, 512, 12>(a, st);
    case 16: return launch_em_r<IT, 512, 16>(a, st);
    case 20: return launch_em_r<IT, 512, 20>(a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int map_max_n() { return kMapMaxThreads * 20; }

size_t map_code_words(int n_pad, int p) {
  return (size_t)p * map_words(map_rows(n_pad)) * map_threads(n_pad);
}

hipError_t launch_map_cols(const uint8_t *X, int n, int p, int n_pad, uint32_t *codes, hipStream_t st) {
  const int WN = map_words(map_rows(n_pad));
  const size_t total = map_code_words(n_pad, p);
  const int grid = static_cast<int>(std::min<size_t>((total + 255) / 256, 4096));
  hipLaunchKernelGGL(map_cols_kernel, dim3(grid), dim3(256), 0, st, X, n, p, WN, map_threads(n_pad), codes);
  return hipGetLastError();
}

hipError_t launch_map_em(bool in_f64, const MapArgs &a, hipStream_t st) {
  if (a.p > kMapMaxP || a.M < 1 || a.n_pad > map_max_n()) return hipErrorInvalidValue;
  return in_f64 ? launch_em_t<double>(a, st) : launch_em_t<float>(a, st);
}

hipError_t launch_best_particle(bool f64, const void *beta, const double *ll, int M, int p, const Prior &pr,
                                int *best, hipStream_t st) {
  if (f64)
    hipLaunchKernelGGL(best_particle_kernel<double>, dim3(1), dim3(1024), 0, st,
                       reinterpret_cast<const double *>(beta), ll, M, p, pr, best);
  else
    hipLaunchKernelGGL(best_particle_kernel<float>, dim3(1), dim3(1024), 0, st,
                       reinterpret_cast<const float *>(beta), ll, M, p, pr, best);
  return hipGetLastError();
}

hipError_t launch_map_starts(bool f64, const void *beta, const int *best, int p, const double *prev,
                             double *starts, hipStream_t st) {
  if (f64)
    hipLaunchKernelGGL(map_starts_kernel<double>, dim3(1), dim3(256), 0, st,
                       reinterpret_cast<const double *>(beta), best, p, prev, starts);
  else
    hipLaunchKernelGGL(map_starts_kernel<float>, dim3(1), dim3(256), 0, st,
                       reinterpret_cast<const float *>(beta), best, p, prev, starts);
  return hipGetLastError();
}

hipError_t launch_map_pick(const double *modes, const double *lp, int ns, int p, double *out, double *out_lp,
                           hipStream_t st) {
  hipLaunchKernelGGL(map_pick_kernel, dim3(1), dim3(256), 0, st, modes, lp, ns, p, out, out_lp);
  return hipGetLastError();
}

}  // namespace spa
