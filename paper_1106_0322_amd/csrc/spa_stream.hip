// Log-likelihood contraction in FP32 and FP64 (and the FP64 adjoint), streamed: no tile staging
// and no barriers in the loop over individuals.
//
//   eta_ik = sum_j X_kj b_ij - m_i,  b_ij = beta_ij / s_j,  m_i = sum_j mu_j b_ij,
//   ll_i   = (X_std^T y) . beta_i - sum_k softplus(eta_ik),
//   g_ij   = (X_std^T y)_j - (sum_k sigma_ik X_kj - mu_j sum_k sigma_ik) / s_j
// (Section 2 likelihood, Section 3 standardisation folded into the coefficients).
//
// Work split.  A workgroup owns 16 particles, one column block of the 16x16x4 MFMA; each of
// its waves holds the same coefficient fragments in registers and takes every NW-th block of
// 16 individuals.  The genotypes are one-byte codes laid out per lane (spa_stream.hpp): a
// lane reads the codes of up to 16 k-steps as one 16-byte load, coalesced over the wave, and
// turns a byte into an operand with one conversion per MFMA (4 of the MFMA's 32 or 64 clocks).
// So a block of individuals costs its n p bytes from the L2 and nothing through LDS, and few
// particles still fill the chip: M = 1000 particles are 63 workgroups of 8 waves times S
// ranges, where a tile shared by 8 waves of different particles gave 8 times S.
// What bounds it: the FP32/FP64 matrix rate at large M (K padded to the next multiple of 4
// only), the elementwise FP64 exp and log for short FP64 rows, launch latency at small M.
// Measured per call, tiled kernel with its packing launch before -> streamed (us): FP32
// loglik n = 1859, p = 184, M = 1000: 51 -> 15; n = 5000, p = 200, M = 16384: 351 -> 295;
// n = 10000, p = 500, M = 16: 245 -> 18; FP64 loglik n = 500, p = 10, M = 64: 15.3 -> 7.4;
// n = 10000, p = 30, M = 30: 123 -> 10; n = 5000, p = 200, M = 16384: 1060 -> 777; FP64
// gradient n = 10000, p = 250, M = 300: 517 -> 132; n = 5000, p = 200, M = 16384: 1980 -> 1672.
//
// Sums: FP32 takes log2(prod (1 + e)) and half of sum |z| per lane and block (as the BF16
// contraction does: the genotypes are centred); FP64 takes sum max(eta, 0) and one log1p
// of the product of the lane's four factors 1 + e^-|eta|, less one, per block; both add per block in
// FP64, then lane groups, waves and ranges in order.
#include <algorithm>
#include <cmath>

#include "spa_lanes.hpp"
#include "spa_moves.hpp"
#include "spa_stream.hpp"

namespace spa {

namespace {

template <Prec P>
struct ST;
template <>
struct ST<Prec::F32> {
  using EL = float;
  using AC = f32x4;
  static __device__ __forceinline__ constexpr int crow(int g, int v) { return 4 * g + v; }
  static __device__ __forceinline__ AC mfma(float a, float b, AC c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct ST<Prec::F64> {
  using EL = double;
  using AC = f64x4;
  static __device__ __forceinline__ constexpr int crow(int g, int v) { return g + 4 * v; }
  static __device__ __forceinline__ AC mfma(double a, double b, AC c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// Instantiated widths in groups of 16 markers and the smallest width each one serves.
constexpr int width_min(int ND) {
  return ND == 1 ? 1 : ND == 2 ? 2 : ND == 4 ? 3 : ND == 8 ? 5 : ND == 13 ? 9 : ND == 16 ? 14 : ND == 24 ? 17 : 25;
}
constexpr int code_regs(int ND) { return ND <= 2 ? ND : (ND + 3) / 4 * 4; }
// LDS row of 16 ND coefficients, padded so that 16 rows' consecutive entries hit distinct banks.
constexpr int row_stride(int ND) { return 16 * ND + 4; }

template <bool ADJOINT>
__global__ void stream_pack_kernel(const uint8_t *__restrict__ X, int n, int p, int nblk, int stride,
                                   uint32_t *__restrict__ out) {
  const size_t total = (size_t)nblk * 64 * stride;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < total;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int d = static_cast<int>(idx % stride), lane = static_cast<int>(idx / stride % 64);
    const int ib = static_cast<int>(idx / stride / 64), lr = lane & 15, lg = lane >> 4;
    uint32_t f = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = ib * 16 + (ADJOINT ? ST<Prec::F64>::crow(lg, q) : lr);
      const int j = 16 * d + (ADJOINT ? lr : 4 * q + lg);
      if (k < n && j < p) f |= static_cast<uint32_t>(X[(size_t)k * p + j]) << (8 * q);
    }
    out[idx] = f;
  }
}

// A lane's code words of one block.
template <int ND>
__device__ __forceinline__ void load_words(const uint32_t *__restrict__ X, int ib, int lane, int stride,
                                           uint32_t (&c)[code_regs(ND)]) {
  const uint32_t *src = X + ((size_t)ib * 64 + lane) * stride;
  if constexpr (ND == 1) {
    c[0] = src[0];
  } else if constexpr (ND == 2) {
    const uint2 v = *reinterpret_cast<const uint2 *>(src);
    c[0] = v.x;
    c[1] = v.y;
  } else {
#pragma unroll
    for (int q = 0; q < code_regs(ND) / 4; ++q)
      if (4 * q < width_min(ND) || 4 * q < stride) {   // uniform
        const uint4 v = *reinterpret_cast<const uint4 *>(src + 4 * q);
        c[4 * q] = v.x;
        c[4 * q + 1] = v.y;
        c[4 * q + 2] = v.z;
        c[4 * q + 3] = v.w;
      }
  }
}

template <typename EL>
__device__ __forceinline__ EL code_value(uint32_t w, int q) {
  return static_cast<EL>((w >> (8 * q)) & 0xffu);
}

// Softplus sum of a lane's four individuals of a block (those before n), and the logistics.
template <Prec P, bool SIG, bool MASKED>
__device__ __forceinline__ double block_softplus(const typename ST<P>::AC &acc, typename ST<P>::EL moff, int k0, int lg,
                                                 int n, typename ST<P>::EL (&sig)[4]) {
  using T = ST<P>;
  if constexpr (P == Prec::F64) {
    double sp = 0.0, f = 0.0;                                    // f = prod (1 + e) - 1
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double eta = acc[v] - moff;
      const double e = exp(-fabs(eta));
      const double d = 1.0 + e;
      const bool valid = !MASKED || k0 + T::crow(lg, v) < n;
      sp += valid ? fmax(eta, 0.0) : 0.0;
      if (valid) f = fma(f, e, f) + e;
      if constexpr (SIG) sig[v] = valid ? (eta >= 0.0 ? 1.0 / d : e / d) : 0.0;
    }
    return sp + log1p(f);
  } else {
    float prod = 1.0f, mx = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float z = acc[v] - moff;
      const float e = __builtin_amdgcn_exp2f(-fabsf(z));
      const bool valid = !MASKED || k0 + T::crow(lg, v) < n;
      if (valid) {
        prod = fmaf(prod, e, prod);
        mx += fabsf(z);
      }
      if constexpr (SIG) {
        const float rc = __builtin_amdgcn_rcpf(1.0f + e);
        sig[v] = valid ? (z >= 0.0f ? rc : e * rc) : 0.0f;
      }
    }
    return static_cast<double>(0.6931471805599453f * (0.5f * mx + __builtin_amdgcn_logf(prod)));
  }
}

// Blocks in flight per wave: two independent MFMA chains where the registers allow.
template <Prec P, int ND, bool GRAD>
constexpr int chains() {
  return !GRAD && ND <= (P == Prec::F32 ? 16 : 8) ? 2 : 1;
}

// The blocks b0 + wave U, ... of [b0, b1) against the wave's 16 particles.  bh: fragments
// of the coefficient rows (lane: particle lane % 16, marker 4 ks + lane / 16).
template <Prec P, int ND, bool GRAD>
__device__ __forceinline__ void stream_blocks(const uint32_t *__restrict__ Xb, const uint32_t *__restrict__ Xtb,
                                              int stride, int n, int p, int b0, int b1, int wave, int nw, int lane,
                                              const typename ST<P>::EL (&bh)[4 * ND], typename ST<P>::EL moff,
                                              double &spl, double &rho, typename ST<P>::AC (&G)[GRAD ? ND : 1]) {
  using T = ST<P>;
  using EL = typename T::EL;
  using AC = typename T::AC;
  constexpr int U = chains<P, ND, GRAD>();
  constexpr int NC = code_regs(ND);
  const int lg = lane >> 4;
  const int nks = (p + 3) / 4, nd = (p + 15) / 16;
  uint32_t c[U][NC];
  const int first = b0 + wave * U;
  if (first < b1) {
#pragma unroll
    for (int u = 0; u < U; ++u) load_words<ND>(Xb, min(first + u, b1 - 1), lane, stride, c[u]);
  }
#pragma unroll 1
  for (int ib = first; ib < b1; ib += nw * U) {
    uint32_t ct[U][GRAD ? NC : 1];
    if constexpr (GRAD) {
#pragma unroll
      for (int u = 0; u < U; ++u) load_words<ND>(Xtb, min(ib + u, b1 - 1), lane, stride, ct[u]);
    }
    AC acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = AC{0, 0, 0, 0};
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      if (d >= width_min(ND) && d >= nd) continue;                      // uniform
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (d >= width_min(ND) - 1 && q > 0 && 4 * d + q >= nks) continue;   // uniform
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = T::mfma(code_value<EL>(c[u][d], q), bh[4 * d + q], acc[u]);
      }
    }
    // the next blocks' codes, in flight during the elementwise step
    const int nx = ib + nw * U;
    if (nx < b1) {
#pragma unroll
      for (int u = 0; u < U; ++u) load_words<ND>(Xb, min(nx + u, b1 - 1), lane, stride, c[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && ib + u >= b1) continue;                              // uniform
      EL sig[4];
      const int k0 = (ib + u) * 16;
      if (k0 + 16 > n) spl += block_softplus<P, GRAD, true>(acc[u], moff, k0, lg, n, sig);
      else spl += block_softplus<P, GRAD, false>(acc[u], moff, k0, lg, n, sig);
      if constexpr (GRAD) {
        rho += (static_cast<double>(sig[0]) + static_cast<double>(sig[1])) +
               (static_cast<double>(sig[2]) + static_cast<double>(sig[3]));
#pragma unroll
        for (int v = 0; v < 4; ++v)                                     // consecutive MFMAs are independent
#pragma unroll
          for (int mb = 0; mb < ND; ++mb) {
            if (mb >= width_min(ND) && mb >= nd) continue;              // uniform
            G[mb] = T::mfma(code_value<EL>(ct[u][mb], v), sig[v], G[mb]);
          }
      }
    }
  }
}

// Particle blocks from which each wave of a gradient workgroup takes its own: then every
// SIMD has one (n = 200, p = 200, M = 30000 FP64: 223 us per call, 361 with shared blocks; tiled
// kernel before 251).
constexpr int kOwnTiles = 1024;

// Waves per workgroup of the contraction: the gradient's accumulators leave one wave per
// SIMD; the forward form has two.
template <bool GRAD>
constexpr int stream_waves() { return GRAD ? 4 : 8; }

// Rows of which a workgroup of 8 waves fills a CU's registers.  With more blocks of particles than
// CUs they run in workgroups of 4, two to a CU, one of which packs its rows while the other
// contracts: log-likelihoods M = 32768, FP64 n = 130, p = 250 109 us in 8 waves, 82 in 4 (tiled kernel
// before 103), FP32 n = 300, p = 500 165 and 127; with one block per CU 8 waves are up to 28 % faster.
constexpr bool wide(Prec prec, int nd) { return nd > (prec == Prec::F64 ? 8 : 16); }
constexpr int kCUs = 256;

// TILES = 1: the workgroup's waves share one block of 16 particles; TILES = NW: each wave has
// its own (many particles with a gradient: no sum over waves, no idle wave when the blocks
// of individuals do not divide by NW).  The gradient of short rows leaves room for two waves
// per SIMD, longer ones take a SIMD's registers.
template <Prec P, int ND, bool GRAD, int NW, int TILES>
__global__ __launch_bounds__(64 * NW, GRAD && ND <= 8 ? 2 : 1) void stream_kernel(StreamArgs a) {
  using T = ST<P>;
  using EL = typename T::EL;
  using AC = typename T::AC;
  static_assert(TILES == 1 || TILES == NW, "one block of particles, or one per wave");
  constexpr int RS = row_stride(ND), W16 = 16 * ND;
  constexpr int RB = TILES == 1 ? 16 / NW : 4;                   // rows packed together by a wave
  extern __shared__ __align__(16) unsigned char sraw[];
  __shared__ EL smoff[TILES][16];
  __shared__ double syb[TILES][16], ssum[2][NW][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int split = static_cast<int>(blockIdx.x) % a.S, tile = static_cast<int>(blockIdx.x) / a.S;
  const int tw = TILES == 1 ? 0 : wave;                          // this wave's tile in the workgroup
  const int r0 = (tile * TILES + tw) * kStreamRows;
  EL *rows = reinterpret_cast<EL *>(sraw) + (size_t)tw * 16 * RS;   // 16 x RS per tile, then the reduction of G
  const int n = a.n, p = a.p, nblk = (n + 15) / 16;
  const int per = (nblk + a.S - 1) / a.S;
  const int b0 = min(nblk, split * per), b1 = min(nblk, b0 + per);

  // ---- coefficient rows in LDS: a row group's loads are all issued before the first is used (one
  // by one, their latencies were most of a call of few individuals: n = 100, p = 500, M = 32768 FP32
  // 130 us, of which the contraction is 40)
  constexpr int NJ = (W16 + 63) / 64;
  double is[NJ], mu[NJ], ys[NJ];
  if (a.beta) {
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
      const int j = lane + 64 * q, jc = min(j, p - 1);
      is[q] = a.inv_s[jc];
      mu[q] = a.mu[jc];
      ys[q] = a.ytil[jc] * a.s[jc];
    }
  }
#pragma unroll 1
  for (int rb = TILES == 1 ? wave * RB : 0; rb < (TILES == 1 ? wave * RB + RB : 16); rb += RB) {
    if (a.beta) {
      double v[RB][NJ];
      auto load = [&](auto *beta) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const auto *row = beta + (size_t)min(r0 + rb + r, a.M - 1) * p;   // padded rows repeat the last one, unused
#pragma unroll
          for (int q = 0; q < NJ; ++q) v[r][q] = static_cast<double>(row[min(lane + 64 * q, p - 1)]);
        }
      };
      if (a.beta_f64) load(static_cast<const double *>(a.beta));
      else load(static_cast<const float *>(a.beta));
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        double m = 0.0, ybv = 0.0;
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
          const int j = lane + 64 * q;
          const bool in = j < p;
          EL h[1];
          double used;
          BPack<P>::put(in ? v[r][q] * is[q] : 0.0, h, h, 0, used);
          if (j < W16) rows[(rb + r) * RS + j] = h[0];
          if (in) {
            m += mu[q] * used;
            ybv += ys[q] * used;
          }
        }
        m = wave_total_f64(m);
        ybv = wave_total_f64(ybv);
        const int i = r0 + rb + r;
        if (lane == 0) {
          smoff[tw][rb + r] = static_cast<EL>(m);
          syb[tw][rb + r] = ybv / BPack<P>::scale;
          if (split == 0 && i < a.M) a.yb[i] = ybv / BPack<P>::scale;
        }
      }
    } else {
      EL v[RB][NJ];
      const int il = min(r0 + rb + min(lane, RB - 1), a.M - 1);      // lane r: row r of the group
      const EL mr = static_cast<EL>(a.moff[il]);
      const double yr = a.yb[il];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const EL *row = static_cast<const EL *>(a.B) + (size_t)min(r0 + rb + r, a.M - 1) * a.PP;
#pragma unroll
        for (int q = 0; q < NJ; ++q) v[r][q] = row[min(lane + 64 * q, p - 1)];
      }
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
          const int j = lane + 64 * q;
          if (j < W16) rows[(rb + r) * RS + j] = j < p ? v[r][q] : EL(0);
        }
      if (lane < RB) {
        smoff[tw][rb + lane] = mr;
        syb[tw][rb + lane] = yr;
      }
    }
  }
  __syncthreads();
  EL bh[4 * ND];
#pragma unroll
  for (int ks = 0; ks < 4 * ND; ++ks) bh[ks] = rows[lr * RS + 4 * ks + lg];
  const EL moff = smoff[tw][lr];

  AC G[GRAD ? ND : 1];
#pragma unroll
  for (int mb = 0; mb < (GRAD ? ND : 1); ++mb) G[mb] = AC{0, 0, 0, 0};
  double spl = 0.0, rho = 0.0;
  stream_blocks<P, ND, GRAD>(a.Xb, a.Xtb, stream_stride(p), n, p, b0, b1, TILES == 1 ? wave : 0,
                             TILES == 1 ? NW : 1, lane, bh, moff, spl, rho, G);

  // ---- lane groups, then (one tile) waves in order
  spl += __shfl_xor(spl, 16, 64);
  spl += __shfl_xor(spl, 32, 64);
  if constexpr (GRAD) {
    rho += __shfl_xor(rho, 16, 64);
    rho += __shfl_xor(rho, 32, 64);
  }
  if (lg == 0) {
    ssum[0][wave][lr] = spl;
    if constexpr (GRAD) ssum[1][wave][lr] = rho;
  }
  __syncthreads();                                               // (also: every wave has read its rows)
  const int rt = TILES == 1 ? tid : lane;                        // the row this thread finishes
  const int i = r0 + rt;
  if (rt < 16 && i < a.M) {
    double sp = 0.0, rh = 0.0;
    for (int w = TILES == 1 ? 0 : wave; w < (TILES == 1 ? NW : wave + 1); ++w) {
      sp += ssum[0][w][rt];
      if constexpr (GRAD) rh += ssum[1][w][rt];
    }
    if (a.spl_part) a.spl_part[split * a.Mp + i] = sp;
    else a.ll[i] = syb[tw][rt] - sp;
    if constexpr (GRAD) static_cast<EL *>(a.g_part)[(split * a.Mp + i) * a.PP + a.PP - 1] = static_cast<EL>(rh);
  }
  if constexpr (GRAD && TILES == 1) {
    // adjoints of the four waves: (0 + 2) + (1 + 3), in wave 0
    static_assert(NW == 4, "tree of four waves");
    AC *gl = reinterpret_cast<AC *>(sraw);                       // 2 x ND x 64
    if (wave >= 2) {
#pragma unroll
      for (int mb = 0; mb < ND; ++mb) gl[((wave - 2) * ND + mb) * 64 + lane] = G[mb];
    }
    __syncthreads();
    if (wave < 2) {
#pragma unroll
      for (int mb = 0; mb < ND; ++mb) G[mb] += gl[(wave * ND + mb) * 64 + lane];
    }
    __syncthreads();
    if (wave == 1) {
#pragma unroll
      for (int mb = 0; mb < ND; ++mb) gl[mb * 64 + lane] = G[mb];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int mb = 0; mb < ND; ++mb) G[mb] += gl[mb * 64 + lane];
    }
  }
  if constexpr (GRAD) {
    const int ig = r0 + lr;
    if ((TILES > 1 || wave == 0) && ig < a.M) {
      EL *gp = static_cast<EL *>(a.g_part) + (split * a.Mp + ig) * a.PP;
#pragma unroll
      for (int mb = 0; mb < ND; ++mb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int j = mb * 16 + T::crow(lg, v);
          if (j < p) gp[j] = G[mb][v];
        }
    }
  }
}

// ------------------------------------------------------------------ combination of ranges
// Forward: one thread per particle.
__global__ void stream_final_ll_kernel(const double *__restrict__ part, const double *__restrict__ yb, int S, size_t Mp,
                                       int M, double *__restrict__ ll) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  double sp = 0.0;
#pragma unroll 8
  for (int s = 0; s < S; ++s) sp += part[s * Mp + i];            // eight loads in flight, added in order
  ll[i] = yb[i] - sp;
}

// Gradient rows, LP lanes per particle and U coefficients per lane at a time: the ranges' adjoints
// summed in order, the standardisation, the prior's gradient and log density (the log of a product
// of U factors where that product is finite), each in FP64 and rounded once to the output type.
// Bound by memory: S float or double adjoints, the particle and the gradient of a coefficient.
// For the tiled contractions it replaces a finalize, a prior and (FP64 callers) a conversion
// launch, 45 us at 16384 x 200, BF16, by one of 35 us.
template <typename GP, typename BT, typename GO, int LP, int U>
__global__ __launch_bounds__(256) void stream_final_grad_kernel(const double *__restrict__ spl, const GP *__restrict__ gp,
                                                                const double *__restrict__ yb, int S, size_t Mp, int PP,
                                                                int M, int p, const double *__restrict__ mu,
                                                                const double *__restrict__ inv_s,
                                                                const double *__restrict__ ytil,
                                                                const BT *__restrict__ beta, Prior pr, int with_prior,
                                                                GO *__restrict__ g, double *__restrict__ ll,
                                                                double *__restrict__ logpost) {
  const int lane = threadIdx.x & (LP - 1);
  const int i = static_cast<int>((blockIdx.x * blockDim.x + threadIdx.x) / LP);
  if (i >= M) return;                                            // whole groups leave together
  double rho = 0.0, sp = 0.0, lsum = 0.0;
#pragma unroll 8
  for (int s = 0; s < S; ++s) {
    rho += static_cast<double>(gp[(s * Mp + i) * PP + PP - 1]);
    sp += spl[s * Mp + i];
  }
  const double lli = yb[i] - sp;
  for (int j0 = lane; j0 < p; j0 += U * LP) {
    double acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.0;
#pragma unroll 8
    for (int s = 0; s < S; ++s) {                                // eight ranges' loads in flight, added in order
      const GP *row = gp + (s * Mp + i) * PP;
#pragma unroll
      for (int u = 0; u < U; ++u) acc[u] += static_cast<double>(row[min(j0 + u * LP, p - 1)]);
    }
    double fac = 1.0, fx[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * LP;
      fx[u] = 0.0;
      if (j >= p) continue;
      double gj = ytil[j] - (acc[u] - mu[j] * rho) * inv_s[j];
      if (with_prior) {
        const double b = static_cast<double>(beta[(size_t)i * p + j]);
        gj += gt_grad(b, pr);
        if (pr.inf) lsum -= fabs(b) / pr.lam;
        else fx[u] = fabs(b) / (pr.a * pr.lam);
        fac *= 1.0 + fx[u];
      }
      g[(size_t)i * p + j] = static_cast<GO>(gj);
    }
    if (with_prior && !pr.inf) {
      if (fac < INFINITY) lsum -= (pr.a + 1.0) * log(fac);
      else                                                       // overflow, infinite or NaN coefficients
        for (int u = 0; u < U; ++u) lsum -= (pr.a + 1.0) * log1p(fx[u]);
    }
  }
  if (with_prior) lsum = lane_group_sum<LP>(lsum);
  if (lane == 0) {
    if (ll) ll[i] = lli;
    if (logpost) logpost[i] = lli + (lsum - static_cast<double>(p) * pr.log2lam);
  }
}

// ------------------------------------------------------------------ random-walk sweeps
// All sweeps of a random-walk scale in one launch: particles do not interact between the
// resampling steps and the step size is fixed within a scale, so a workgroup keeps its 16
// particles (rows in registers, the proposals' operand in LDS) through propose ->
// contraction -> decision of every sweep, with two barriers per sweep.  Against separate
// proposal/decision and contraction launches this saves the launches, the particle rows'
// round trips through memory (about 40 bytes per coefficient and sweep) and the copies of
// the split partials.  The row arithmetic is the move kernels' (same Philox counters, same
// order of operations), 32 lanes per row, lane l holding markers 4l + 128 kb + 0..3.
// (Drawing the next sweep's normals into LDS after a wave's share of the contraction, one
// Philox block or Box-Muller pair per thread, shortened the FP32 sweep by 2 % and lengthened
// the FP64 one by 6 %: the row work is a latency chain, not a throughput one.)
// FP32 rows leave room for two workgroups of 8 waves per CU (128 VGPRs), whose row work and
// contractions overlap (rows of 200 markers, which have since left this form: n = 5000, N = 16384
// 3.71 -> 3.56 ms per scale of 10 sweeps, one workgroup against two); FP64 rows would spill
// (663 -> 792 us at n = 1000, p = 100).
template <Prec P, int ND, int NW>
__global__ __launch_bounds__(64 * NW, P == Prec::F32 ? 4 : 2) void rwm_sweeps_kernel(RwmArgs a) {
  using T = ST<P>;
  using EL = typename T::EL;                                     // particle and contraction type
  using AC = typename T::AC;
  constexpr int RS = row_stride(ND), W16 = 16 * ND, KB = ND <= 8 ? 1 : 2;
  static_assert(W16 <= 128 * KB, "32 lanes of 4 KB markers cover a row");
  static_assert(64 * NW >= 512, "a thread per row lane");
  extern __shared__ __align__(16) unsigned char sraw[];
  EL *rows = reinterpret_cast<EL *>(sraw);                       // 16 x RS
  __shared__ EL smoff[16];
  __shared__ double ssum[NW][16];
  __shared__ int scnt[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int n = a.n, p = a.p, nblk = (n + 15) / 16;
  const Prior pr = a.prior;
  if (tid < 2) scnt[tid] = 0;

  // ---- the step size (burn-in: from the previous sweep's)
  double step = a.step;
  unsigned long long *count = a.count;
  if (a.ring_step) {
    const int now = a.sweep0 % 3, prev = (a.sweep0 + 2) % 3;
    if (!a.first) {
      step = a.ring_step[prev];
      if (a.adapt) {
        const double l2 = 0.69314718055994530942;
        double d = static_cast<double>(a.ring_cnt[prev]) / static_cast<double>(a.M) - a.target;
        d = fmin(fmax(d, -l2), l2);
        step *= exp(d);
      }
    }
    count = nullptr;
    if (blockIdx.x == 0 && tid == 0) {
      a.ring_step[now] = step;
      a.ring_cnt[(a.sweep0 + 1) % 3] = 0ull;
    }
  }

  // ---- this thread's part of a particle row
  const bool rowt = tid < 512;
  const int row = (tid >> 5) & 15, l = tid & 31;
  const int i = blockIdx.x * kStreamRows + row;
  const bool live = rowt && i < a.M;
  const EL inv_ac = pr.inf ? EL(0) : static_cast<EL>(1.0 / (pr.a * pr.lam));
  const double base = -static_cast<double>(p) * pr.log2lam;
  const double pscale = pr.inf ? 1.0 / pr.lam : pr.a + 1.0;
  const EL st = static_cast<EL>(step);
  EL *beta = static_cast<EL *>(a.beta) + (size_t)(live ? i : 0) * p;
  EL cur[KB][4], nv[KB][4], ss[KB][4];
  double ll = 0.0, lpc = 0.0;
  int cnt = 0;
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    EL fc = EL(1), lc = EL(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = 4 * l + 128 * kb + k;
      const bool in = live && j < p;
      cur[kb][k] = in ? beta[j] : EL(0);
      ss[kb][k] = in ? st * static_cast<EL>(a.sigma[j]) : EL(0);
      if (in) {
        if (pr.inf) lc += fabs(cur[kb][k]);
        else fc *= gt_factor<EL>(cur[kb][k], inv_ac);
      }
    }
    if (pr.inf) lpc += static_cast<double>(lc);
    else lpc += static_cast<double>(fast_log(fc));
  }
  if (rowt) lpc = lane_group_sum<32>(lpc);
  lpc = base - pscale * lpc;
  if (live) ll = a.ll[i];

  for (int sw = 0; sw < a.sweeps; ++sw) {
    const uint32_t sweep = static_cast<uint32_t>(a.sweep0 + sw);
    double lpp = 0.0, ybv = 0.0;
    if (rowt) {
      double m = 0.0;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const int b0 = 4 * l + 128 * kb;
        if (b0 >= W16) continue;
        EL z[4] = {0, 0, 0, 0};
        const bool act = live && b0 < p;
        if (act)
          block_normals(philox4x32_10(make_uint4(static_cast<uint32_t>(i), static_cast<uint32_t>(b0 >> 2), sweep,
                                                 word3(a.t, kTagNormal)),
                                      a.k0, a.k1),
                        z);
        EL fp = EL(1), lpn = EL(0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int j = b0 + k;
          const bool in = act && j < p;
          nv[kb][k] = in ? cur[kb][k] + ss[kb][k] * z[k] : EL(0);
          double bj = 0.0, muj = 0.0, ytj = 0.0;
          if (in) {
            if (pr.inf) lpn += fabs(nv[kb][k]);
            else fp *= gt_factor<EL>(nv[kb][k], inv_ac);
            bj = static_cast<double>(nv[kb][k]) * a.inv_s[j];
            muj = a.mu[j];
            ytj = a.ytil[j] * a.s[j];
          }
          EL h[1];
          double used;
          BPack<P>::put(bj, h, h, 0, used);
          rows[row * RS + j] = h[0];
          m += muj * used;
          ybv += ytj * used;
        }
        if (pr.inf) lpp += static_cast<double>(lpn);
        else lpp += static_cast<double>(fast_log(fp));
      }
      m = lane_group_sum<32>(m);
      ybv = lane_group_sum<32>(ybv);
      lpp = lane_group_sum<32>(lpp);
      if (l == 0) smoff[row] = static_cast<EL>(m);
    }
    __syncthreads();
    EL bh[4 * ND];
#pragma unroll
    for (int ks = 0; ks < 4 * ND; ++ks) bh[ks] = rows[lr * RS + 4 * ks + lg];
    double spl = 0.0, rho = 0.0;
    AC G[1];
    stream_blocks<P, ND, false>(a.Xb, nullptr, stream_stride(p), n, p, 0, nblk, wave, NW, lane, bh, smoff[lr], spl, rho,
                                G);
    spl += __shfl_xor(spl, 16, 64);
    spl += __shfl_xor(spl, 32, 64);
    if (lg == 0) ssum[wave][lr] = spl;
    __syncthreads();
    if (rowt) {
      double sp = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) sp += ssum[w][row];
      const double llp = ybv / BPack<P>::scale - sp, lppv = base - pscale * lpp;
      const double log_alpha = llp - ll + lppv - lpc;
      const uint4 w = philox4x32_10(make_uint4(static_cast<uint32_t>(i), 0u, sweep, word3(a.t, kTagUniform)), a.k0,
                                    a.k1);
      const double u = (static_cast<double>(w.x) + 0.5) * 0x1p-32;
      if (log(u) < log_alpha) {                                  // false for NaN; the same in every lane of the row
        ll = llp;
        lpc = lppv;
        ++cnt;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int k = 0; k < 4; ++k) cur[kb][k] = nv[kb][k];
      }
    }
  }
  if (live) {
    if (cnt > 0) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int j = 4 * l + 128 * kb + k;
          if (j < p) beta[j] = cur[kb][k];
        }
    }
    if (l == 0) {
      if (cnt > 0) {
        a.ll[i] = ll;
        atomicAdd(&scnt[0], cnt);
      }
      if (!isfinite(ll)) atomicAdd(&scnt[1], 1);
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (a.ring_step) {
      if (scnt[0]) atomicAdd(&a.ring_cnt[a.sweep0 % 3], static_cast<unsigned long long>(scnt[0]));
    } else {
      if (scnt[0]) atomicAdd(&count[0], static_cast<unsigned long long>(scnt[0]));
      if (scnt[1]) atomicAdd(&count[1], static_cast<unsigned long long>(scnt[1]));
    }
  }
}

template <Prec P, int ND, bool GRAD, int NW, int TILES>
hipError_t launch_waves(const StreamArgs &a, hipStream_t s) {
  using EL = typename ST<P>::EL;
  constexpr size_t rows = (size_t)TILES * 16 * row_stride(ND) * sizeof(EL);
  constexpr size_t red = GRAD && TILES == 1 ? 2 * (size_t)ND * 64 * 4 * sizeof(EL) : 0;
  constexpr size_t lds = rows > red ? rows : red;
  static_assert(lds <= 140 * 1024, "LDS budget");
  auto kern = stream_kernel<P, ND, GRAD, NW, TILES>;
  static OncePerDevice once;
  const hipError_t e = raise_lds_limit(once, kern, lds);
  if (e != hipSuccess) return e;
  const int tiles = (a.M + kStreamRows * TILES - 1) / (kStreamRows * TILES);
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles * a.S), dim3(64 * NW), lds, s, a);
  return hipGetLastError();
}

template <Prec P, int ND, bool GRAD>
hipError_t launch_one(const StreamArgs &a, hipStream_t s) {
  const int tiles = (a.M + kStreamRows - 1) / kStreamRows;
  if constexpr (GRAD) {
    if (tiles >= kOwnTiles) return launch_waves<P, ND, GRAD, 4, 4>(a, s);
    return launch_waves<P, ND, GRAD, 4, 1>(a, s);
  } else {
    if constexpr (ND <= 4)   // one range of few particles: twice the waves, half the latency
      if (a.S == 1 && tiles <= 256) return launch_waves<P, ND, GRAD, 16, 1>(a, s);
    if constexpr (wide(P, ND))
      if (tiles > kCUs) return launch_waves<P, ND, GRAD, 4, 1>(a, s);
    return launch_waves<P, ND, GRAD, stream_waves<GRAD>(), 1>(a, s);
  }
}

template <Prec P, bool GRAD>   // the gradient in FP64 only
hipError_t launch_width(const StreamArgs &a, hipStream_t s) {
  const int nd = stream_dwords(a.p);
  if (nd <= 1) return launch_one<P, 1, GRAD>(a, s);
  if (nd <= 2) return launch_one<P, 2, GRAD>(a, s);
  if (nd <= 4) return launch_one<P, 4, GRAD>(a, s);
  if (nd <= 8) return launch_one<P, 8, GRAD>(a, s);
  if (nd <= 13) return launch_one<P, 13, GRAD>(a, s);
  if (nd <= 16) return launch_one<P, 16, GRAD>(a, s);
  if constexpr (P == Prec::F32) {
    if (nd <= 24) return launch_one<P, 24, GRAD>(a, s);
    if (nd <= 32) return launch_one<P, 32, GRAD>(a, s);
  }
  return hipErrorInvalidValue;
}

// (rwm_sweeps measured: run of 100 scales x 10 sweeps and 200 burn-in sweeps at n = 2000,
// p = 50, N = 8192 FP32: 56.4 -> 33.3 ms, 23 us a sweep of which 11.6 are the FP32 matrix
// rate; FP32 MFMAs and vector instructions of a SIMD do not overlap here: without the
// MFMAs a sweep takes 10.3 us.  20 scales x 5 sweeps and 200 burn-in sweeps at n = 500, p = 10,
// N = 1024 FP64: 10.7 -> 6.0 ms.)
template <Prec P, int ND, int NW>
hipError_t launch_rwm_one(const RwmArgs &a, hipStream_t s) {
  constexpr size_t lds = 16 * (size_t)row_stride(ND) * sizeof(typename ST<P>::EL);
  auto kern = rwm_sweeps_kernel<P, ND, NW>;
  static OncePerDevice once;
  const hipError_t e = raise_lds_limit(once, kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((a.M + kStreamRows - 1) / kStreamRows), dim3(64 * NW), lds, s, a);
  return hipGetLastError();
}

constexpr int kRwmMarkersF32 = 128;   // longest FP32 rows of the one-launch sweeps
template <Prec P>
hipError_t launch_rwm_width(const RwmArgs &a, hipStream_t s) {
  const int nd = stream_dwords(a.p);
  // few workgroups: 16 waves each; else 8, two or more workgroups per CU in different phases
  const bool few = (a.M + kStreamRows - 1) / kStreamRows <= 256;
  if (nd <= 1) return few ? launch_rwm_one<P, 1, 16>(a, s) : launch_rwm_one<P, 1, 8>(a, s);
  if (nd <= 2) return few ? launch_rwm_one<P, 2, 16>(a, s) : launch_rwm_one<P, 2, 8>(a, s);
  if (nd <= 4) return few && P == Prec::F32 ? launch_rwm_one<P, 4, 16>(a, s) : launch_rwm_one<P, 4, 8>(a, s);
  if (nd <= 8) return launch_rwm_one<P, 8, 8>(a, s);
  if constexpr (P == Prec::F64) {
    if (nd <= 13) return launch_rwm_one<P, 13, 8>(a, s);
    if (nd <= 16) return launch_rwm_one<P, 16, 8>(a, s);
  }
  return hipErrorInvalidValue;
}

// Clocks of one block of 16 individuals against 16 particles on one SIMD: matrix
// instructions and the elementwise step (a wave's, as issued).
double block_clocks(Prec prec, int p) {
  const int nks = (p + 3) / 4;
  return prec == Prec::F64 ? nks * 64.0 + 1500.0 : nks * 32.0 + 200.0;
}

}  // namespace

template <bool ADJOINT>
static hipError_t launch_pack(const uint8_t *X, int n, int p, uint32_t *out, hipStream_t s) {
  const int nblk = stream_blocks(n), stride = stream_stride(p);
  const size_t total = (size_t)nblk * 64 * stride;
  const int grid = static_cast<int>(std::min<size_t>((total + 255) / 256, 8192));
  hipLaunchKernelGGL(stream_pack_kernel<ADJOINT>, dim3(grid), dim3(256), 0, s, X, n, p, nblk, stride, out);
  return hipGetLastError();
}
hipError_t launch_stream_pack(const uint8_t *X, int n, int p, uint32_t *Xb, hipStream_t s) {
  return launch_pack<false>(X, n, p, Xb, s);
}
hipError_t launch_stream_pack_adjoint(const uint8_t *X, int n, int p, uint32_t *Xtb, hipStream_t s) {
  return launch_pack<true>(X, n, p, Xtb, s);
}

// The power of two of least estimated time, in clocks: rounds of workgroups over the CUs, each a
// range's blocks of one SIMD's waves and the workgroup's rows; the latency that a workgroup's end
// leaves uncovered (where a CU holds several); what the ranges' partials cost to combine.
// The numbers are fitted to 1046 calls measured with 1 to 64 ranges (n = 100 .. 10000, p = 12 .. 500,
// M = 16 .. 32768): the chosen count is 0.2 % (FP64 gradient) and 2 % (log-likelihoods) slower than
// the best one on average.  Doubling until a number of workgroups is reached was 5 to 9 % slower and
// left a last round nearly empty (FP64 gradient n = 10000, p = 200, M = 4100: 1 range 1717 us, 4 1103,
// tiled kernel before 1369; n = 5000, p = 200, M = 9000: 1 range 1300, 4 1064; log-likelihoods n = 1600,
// p = 250, M = 2000: 8 ranges 77, 2 46).
int stream_splits(Prec prec, bool grad, int n, int p, int M, int smax) {
  const bool f64 = prec == Prec::F64;
  const int nblk = stream_blocks(n), nd = stream_dwords(p), nks = (p + 3) / 4;
  if (!grad && nblk * block_clocks(prec, p) <= 4 * 16000.0) return 1;   // the combination's launch costs more
  const long long tiles = (M + kStreamRows - 1) / kStreamRows;
  const bool own = grad && tiles >= kOwnTiles;
  const long long wgs = own ? (tiles + 3) / 4 : tiles;
  const int group = grad ? 4 : !wide(prec, nd) ? 16 : tiles > kCUs ? 4 : 8;   // blocks of a pass of the workgroup's waves
  // whether a CU holds several workgroups, so that one's rows run beside another's blocks
  const bool several = grad ? nd <= 8 : nd <= (f64 ? 4 : 16) || (wide(prec, nd) && tiles > kCUs);
  const double mfma = (nks + (grad ? 4 * nd : 0)) * (f64 ? 64.0 : 32.0), rp = static_cast<double>(p) * (own ? 4 : 1);
  const double block = grad ? 1.235 * mfma + 830.0 : f64 ? 1.224 * mfma + 1015.0 : 0.902 * mfma + 94.0;
  const double rows = grad ? 670.0 + 96.0 * rp : f64 ? 1140.0 + 39.0 * rp : 1250.0 + 16.0 * rp;
  const double tail = !several ? 0.0 : grad ? 0.54 : f64 ? 0.09 : 0.16;
  const double again = !several ? 1.0 : grad ? 1.24 : f64 ? 0.70 : 0.78;   // a further round's rows
  const double launch = grad ? 2200.0 : f64 ? 8100.0 : 5300.0;
  const double partial = grad ? 375.0 + 0.0006 * M * gemm_pad_markers(p, prec) : f64 ? 240.0 + 0.018 * M : 80.0 + 0.0045 * M;
  int best = 1;
  double least = 0.0;
  for (int S = 1; S <= smax && S <= nblk; S *= 2) {
    if (!grad && S > 1 && 8ull * S * tiles * kStreamRows > kStreamPartialBytes) break;
    const int per = (nblk + S - 1) / S;
    const int blocks = own ? per : grad ? (per + 3) / 4 : (per + group - 1) / group * (group / 4);
    const double rounds = static_cast<double>((wgs * S + kCUs - 1) / kCUs);
    const double t = (rounds + tail) * blocks * block + (1.0 + again * (rounds - 1.0)) * rows +
                     (S > 1 ? launch : 0.0) + S * partial;
    if (S == 1 || t < least) {
      best = S;
      least = t;
    }
  }
  return best;
}

hipError_t launch_stream(const StreamArgs &a, hipStream_t s) {
  if (a.S < 1 || (a.S > 1 && !a.spl_part) || (a.grad && (!a.spl_part || !a.g_part || !a.Xtb))) return hipErrorInvalidValue;
  if (a.prec == Prec::F64)
    return a.grad ? launch_width<Prec::F64, true>(a, s) : launch_width<Prec::F64, false>(a, s);
  if (a.prec == Prec::F32)
    return a.grad ? hipErrorInvalidValue : launch_width<Prec::F32, false>(a, s);   // the FP32 adjoint is tiled
  return hipErrorInvalidValue;
}

hipError_t launch_stream_finalize(const StreamFinal &f, hipStream_t s) {
  const StreamArgs &a = *f.a;
  if (!f.g) {
    hipLaunchKernelGGL(stream_final_ll_kernel, dim3((a.M + 255) / 256), dim3(256), 0, s, a.spl_part, a.yb, a.S, a.Mp,
                       a.M, a.ll);
    return hipGetLastError();
  }
  const Prior pr = f.prior ? *f.prior : Prior{};
  // few particles: a wave each, one coefficient per lane (latency); else four per lane, or two for
  // rows that do not end near a multiple of 256
  const int LP = a.M <= 2048 ? 64 : a.p <= 64 ? 16 : a.p <= 128 ? 32 : 64;
  const dim3 grid((unsigned)(((size_t)a.M * LP + 255) / 256));
#define SPA_FG(GP, BT, GO, LPV, UV)                                                                                 \
  hipLaunchKernelGGL((stream_final_grad_kernel<GP, BT, GO, LPV, UV>), grid, dim3(256), 0, s, a.spl_part,                 \
                     static_cast<const GP *>(a.g_part), a.yb, a.S, a.Mp, a.PP, a.M, a.p, a.mu, a.inv_s, a.ytil,      \
                     static_cast<const BT *>(a.beta), pr, f.prior ? 1 : 0, static_cast<GO *>(f.g), a.ll, f.logpost)
#define SPA_FG_LP(GP, BT, GO)                          \
  do {                                                 \
    if (a.M <= 2048) SPA_FG(GP, BT, GO, 64, 1);        \
    else if (a.p > 256) SPA_FG(GP, BT, GO, 64, 2);     \
    else if (LP == 16) SPA_FG(GP, BT, GO, 16, 4);      \
    else if (LP == 32) SPA_FG(GP, BT, GO, 32, 4);      \
    else SPA_FG(GP, BT, GO, 64, 4);                    \
  } while (0)
  // the caller's particles and gradient share their type
  if (f.part_f32) {
    if (f.g_f64) SPA_FG_LP(float, double, double);
    else SPA_FG_LP(float, float, float);
  } else {
    if (f.g_f64) SPA_FG_LP(double, double, double);
    else SPA_FG_LP(double, float, float);
  }
#undef SPA_FG_LP
#undef SPA_FG
  return hipGetLastError();
}

// Estimated clocks of a sweep in both forms: rounds of workgroups over the CUs, each its blocks of
// individuals and its rows, against the split contraction at its best count of ranges plus the
// proposal and decision launches and their passes over the rows.  Fitted to 982 workloads measured
// in both forms (n = 60 .. 10000, p = 5 .. 250, N = 64 .. 32768): the chosen form is 0.02 % (FP32) and
// 0.2 % (FP64) slower than the better one on average.  Per sweep (us), one launch and apart, near the
// line: FP32 n = 6400, p = 60, N = 3000 42.5 and 41.8, n = 1600, p = 60, N = 9000 37.6 and 42.4; FP64 n =
// 60, p = 120, N = 32768 82 and 90, n = 200, p = 250, N = 16384 107 and 93 (the first is taken); beyond it
// FP32 n = 6400, p = 120, N = 1000 71 and 33, FP64 n = 6400, p = 250, N = 9000 907 and 670.  FP32 rows
// of more than 128 markers spilled in one launch: apart was the better one, or within 1 %, in all of 133.
bool rwm_one_launch(Prec prec, int n, int p, int M) {
  const bool f64 = prec == Prec::F64;
  if ((!f64 && prec != Prec::F32) || p > (f64 ? 256 : kRwmMarkersF32)) return false;
  const int nblk = stream_blocks(n), nd = stream_dwords(p), nks = (p + 3) / 4;
  const int tiles = (M + kStreamRows - 1) / kStreamRows;
  const double block = f64 ? 0.88 * 64.0 * nks + 820.0 : 1.07 * 32.0 * nks + 100.0;
  const int group = wide(prec, nd) ? 8 : 16, agroup = wide(prec, nd) && tiles > kCUs ? 4 : group;
  const double mine = (nblk + group - 1) / group * (group / 4) * block, rounds = (tiles + kCUs - 1) / kCUs;
  double split = 0.0;
  for (int S = 1; S <= 16 && S <= nblk; S *= 2) {
    const int per = (nblk + S - 1) / S;
    const double t = static_cast<double>((static_cast<long long>(tiles) * S + kCUs - 1) / kCUs) *
                     ((per + agroup - 1) / agroup * (agroup / 4) * block + 1500.0);
    if (S == 1 || t < split) split = t;
  }
  const double one = f64 ? rounds * (1.065 * mine + 11500.0 + 5.5 * p + (p > 128 ? 9100.0 : 0.0)) + 2500.0
                         : rounds * (1.39 * mine + 4570.0 + 6.3 * p) + 13300.0;
  const double rows = static_cast<double>(tiles) * p / kCUs;
  const double apart = f64 ? 1.066 * split + 24100.0 + 68.0 * rows : 1.387 * split + 35500.0 + 12.2 * rows;
  return one <= apart;
}

hipError_t launch_rwm_sweeps(const RwmArgs &a, hipStream_t s) {
  return a.prec == Prec::F64 ? launch_rwm_width<Prec::F64>(a, s) : launch_rwm_width<Prec::F32>(a, s);
}

}  // namespace spa
