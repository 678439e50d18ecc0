// Log-likelihood contraction of all particles against the genotype matrix, on MFMA: BF16
// hi+lo, and every FP32 gradient, the FP32 MALA sweeps' included (FP32 log-likelihoods and all
// FP64 evaluations are streamed, spa_stream.hip).
//
// For particles i and individuals k (Section 2 likelihood on standardised genotypes,
// Section 3):
//   eta_ik = sum_j X_kj b_ij - m_i,    b_ij = beta_ij / s_j,   m_i = sum_j mu_j b_ij
//            (the standardisation folded into the coefficients: X stays exact 0/1/2)
//   ll_i   = (X_std^T y) . beta_i - sum_k softplus(eta_ik)
//   g_ij   = (X_std^T y)_j - (sum_k sigma_ik X_kj - mu_j sum_k sigma_ik) / s_j,
//            sigma_ik = logistic(eta_ik)   (the likelihood gradient X_std^T (y - sigma))
//
// Work decomposition.  A workgroup of 8 wave64s (4 for rows of more than 256 markers) owns 16
// particles per wave; each wave keeps the BF16 hi/lo (or FP32) fragments of its particles in
// registers for the whole pass.  Individuals are split into S contiguous ranges, one per workgroup of a
// "split"; the workgroup -> (split, particle tile) map follows the round-robin dispatch of
// workgroups to the 8 XCDs so that the XCDs of one split share its genotype slice in their
// L2.  A workgroup streams its slice in tiles of NT individuals through double-buffered LDS (the
// next tile is copied there while the current one is used; FP8 codes are widened to BF16 on the
// way, through registers): the individual-major tile feeds the forward MFMA (eta^T blocks,
// individuals x particles) and, for the gradient, the marker-major tile feeds the adjoint MFMA
// G^T += X^T sigma^T, whose B operand is the logistic of the forward output taken straight from
// the accumulator registers (a lane of an eta^T block holds four individuals of one particle,
// i.e. the K slots of an MFMA B fragment).  Softplus sums: per lane and tile, sum max(eta, 0) plus
// one log of prod (1 + exp(-|eta|)) (the product of at most 16 factors in (1, 2] cannot
// overflow), accumulated across tiles in FP64 in a fixed order; in reduced precision
// sum max(eta, 0) is taken as half of sum |eta| (the standardised genotypes are centred,
// so sum_k eta_ik = 0 over the real individuals).  With S > 1 each split
// writes partial sums that a finalize kernel adds in split order.
#include "spa_common.hpp"
#include "spa_internal.hpp"
#include "spa_lanes.hpp"

namespace spa {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <Prec P>
struct GT;

template <>
struct GT<Prec::BF16X2> {
  using LX = __bf16;   // genotype element in LDS
  using BT = __bf16;   // coefficient element in HBM
  using FR = bf16x8;   // MFMA A/B fragment (8 consecutive K values per lane)
  using AC = f32x4;
  using EL = float;
  static constexpr int KS = 32, KV = 8;
  // rows of a 16x16 output block held by lane group g: 4g + v
  static __device__ __forceinline__ constexpr int crow(int g, int v) { return 4 * g + v; }
  static __device__ __forceinline__ AC mfma(FR a, FR b, AC c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct GT<Prec::F32> {
  using LX = float;
  using BT = float;
  using FR = float;
  using AC = f32x4;
  using EL = float;
  static constexpr int KS = 4, KV = 1;
  static __device__ __forceinline__ constexpr int crow(int g, int v) { return 4 * g + v; }
  static __device__ __forceinline__ AC mfma(FR a, FR b, AC c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// LDS fragment reads kept in flight ahead of the MFMAs that consume them (BF16 path).
constexpr int kPrefetch = 4;

// Tile shape per precision and padded marker count.  Each wave owns 16 particles (one
// MFMA column block); a workgroup has NW waves.  With PP <= 256 the BF16 and FP32 variants
// fit two waves per SIMD (8 per workgroup), so one wave's elementwise VALU work overlaps
// the other's MFMAs; wider rows keep one wave per SIMD.
template <Prec P, int PP>
struct Shape {
  static constexpr int NT = (P == Prec::BF16X2) ? (PP <= 256 ? 64 : 32) : 16;   // individuals
  static constexpr int PB = 1;                                                   // 16-particle blocks per wave
  static constexpr int NW = PP <= 256 ? 8 : 4;               // waves per workgroup
  static constexpr int NTHR = 64 * NW;
  static constexpr int WGP = NW * 16 * PB;                                       // particles per workgroup
};

// LDS stage layout in 16-byte chunks ("slots").  The individual-major tile has NT rows of
// CPR = PP*es/16 chunks and the marker-major tile PP rows of CPT = NT*es/16 chunks; each region
// is rounded up to a multiple of the thread count so that every thread moves exactly one chunk
// per copy instruction.  Two stages (double buffering).
template <Prec P, int PP, bool GRAD>
struct Lds {
  using LX = typename GT<P>::LX;
  static constexpr int NT = Shape<P, PP>::NT;
  static constexpr int CPR = PP * (int)sizeof(LX) / 16;
  static constexpr int CPT = NT * (int)sizeof(LX) / 16;
  // slots from row to row: the chunks of a row are permuted (row_swizzle), or, in FP32 rows of up to
  // 128 and of 384 markers, the stride is padded to an odd one.  An FP32 fragment reads single
  // words, whose address is then an immediate offset, where a permuted one costs two
  // instructions beside each MFMA; the permuted tiles are smaller and their adjoint reads free of
  // conflicts (gradients, padded and permuted: n = 5000, p = 40, M = 40000 807 and 896 us, p = 300
  // 4060 and 4160; p = 200 1725 and 1609; p = 511, M = 9000 1290 and 1129)
  static constexpr bool PAD = P == Prec::F32 && (PP <= 128 || PP == 384);
  static constexpr int CX = CPR + PAD, CT = CPT + PAD;
  static constexpr int NTHR = Shape<P, PP>::NTHR;
  static constexpr int XSL = (NT * CX + NTHR - 1) / NTHR * NTHR;
  static constexpr int TSL = GRAD ? (PP * CT + NTHR - 1) / NTHR * NTHR : 0;
  static constexpr int STG = XSL + TSL;
  static constexpr size_t bytes = 2 * (size_t)STG * 16;
};

// One 16-byte global -> LDS copy per lane; lane i writes lds[i] (wave-uniform base).
__device__ __forceinline__ void lds_dma16(const void *g, uint4 *lds) {
  __builtin_amdgcn_global_load_lds(g, lds, 16, 0, 0);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// 16 FP8 (e4m3) codes -> two chunks of 8 BF16 values in LDS (exact for finite codes).
__device__ __forceinline__ void store_fp8_as_bf16(uint4 *dst0, uint4 *dst1, uint4 v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(w[q]), false);
    const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(w[q]), true);
    bf16x4 o;
    o[0] = static_cast<__bf16>(lo[0]);
    o[1] = static_cast<__bf16>(lo[1]);
    o[2] = static_cast<__bf16>(hi[0]);
    o[3] = static_cast<__bf16>(hi[1]);
    reinterpret_cast<bf16x4 *>(q < 2 ? dst0 : dst1)[q & 1] = o;
  }
}

// One workgroup per CU (the double-buffered tiles take most of the LDS): NW/4 waves per SIMD.
template <Prec P, int PP, bool GRAD, bool FP8>
__global__ __attribute__((amdgpu_flat_work_group_size(64, (Shape<P, PP>::NTHR))))
__attribute__((amdgpu_waves_per_eu((Shape<P, PP>::NW / 4), (Shape<P, PP>::NW / 4)))) void loglik_kernel(GemmArgs args) {
  using T = GT<P>;
  using LX = typename T::LX;
  using BT = typename T::BT;
  using FR = typename T::FR;
  using AC = typename T::AC;
  using EL = typename T::EL;
  using SH = Shape<P, PP>;
  using L = Lds<P, PP, GRAD>;
  using XG = typename std::conditional<FP8, uint8_t, LX>::type;   // genotype element in HBM
  constexpr int KS = T::KS, KV = T::KV, NT = SH::NT, PB = SH::PB, WGP = SH::WGP;
  constexpr int IB = NT / 16;    // 16-individual blocks per tile
  constexpr int QB = (P == Prec::BF16X2) ? 2 : 1;   // blocks per adjoint k-step
  constexpr int NKS = PP / KS;   // k-steps of the forward contraction
  constexpr int NMB = PP / 16;   // 16-marker blocks of the adjoint
  constexpr int CPR = L::CPR, CPT = L::CPT, CX = L::CX, CT = L::CT;
  constexpr int XSL = L::XSL, TSL = L::TSL, STG = L::STG;
  constexpr int NTHR = SH::NTHR;
  // what must stay on its side between two k-steps: everything, or all but vector and scalar
  // arithmetic and the copies
  constexpr int kKeepApart = SH::NW == 4 ? 0 : 0x416;
  // With two waves per SIMD the one in its MFMAs goes first: the other's vector work then falls
  // beside them (p = 200: 1646 -> 1631 us per scale, p = 250: 1920 -> 1878; rows of up to 128
  // markers and FP8 storage: nothing or slower)
  constexpr bool PRIO = P == Prec::BF16X2 && GRAD && !FP8 && PP > 128 && SH::NW == 8;
  constexpr int NQX = XSL / NTHR, NQT = GRAD ? TSL / NTHR : 1;   // copy instructions per thread
  static_assert(P != Prec::BF16X2 || IB % 2 == 0, "BF16 adjoint k-step spans two blocks");
  static_assert(P == Prec::BF16X2 || IB == 1, "FP32 adjoint uses one block per tile");
  static_assert(!FP8 || P == Prec::BF16X2, "FP8 storage feeds the BF16 path");

  extern __shared__ __align__(16) uint4 smem[];   // STG 16-byte slots per stage

  // ---- workgroup -> (split, particle tile); XCD-aware (workgroups go round-robin to 8 XCDs)
  const int S = args.S;
  const int g8 = 8 / S;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int split = xcd / g8;
  const int ptile = slot * g8 + (xcd % g8);
  const int ntiles_p = (args.M + WGP - 1) / WGP;
  if (ptile >= ntiles_p) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int wbase = ptile * WGP + wave * 16 * PB;
  const int n = args.n, n_pad = args.n_pad;
  const int chunk = ((n_pad + S - 1) / S + NT - 1) / NT * NT;
  const int i0 = min(n_pad, split * chunk);
  // tiles holding at least one real individual (n_pad may exceed n by more than a tile)
  const int i1 = min(min(n_pad, i0 + chunk), (n + NT - 1) / NT * NT);
  const int ntiles = max(0, (i1 - i0) / NT);

  // ---- coefficient fragments: register resident for the whole pass
  FR bh[PB][NKS];
  FR bl[PB][(P == Prec::BF16X2) ? NKS : 1];
  EL moff[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const size_t row = static_cast<size_t>(wbase + pb * 16 + lr);
    const BT *sh = reinterpret_cast<const BT *>(args.Bhi) + row * PP + lg * KV;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) bh[pb][ks] = *reinterpret_cast<const FR *>(sh + ks * KS);
    if constexpr (P == Prec::BF16X2) {
      const BT *sl = reinterpret_cast<const BT *>(args.Blo) + row * PP + lg * KV;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) bl[pb][ks] = *reinterpret_cast<const FR *>(sl + ks * KS);
    }
    moff[pb] = static_cast<EL>(args.moff[row]);
  }

  AC G[PB][GRAD ? NMB : 1];
  if constexpr (GRAD) {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) G[pb][mb] = AC{0, 0, 0, 0};
  }
  double spl[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) spl[pb] = 0.0;

  // ---- tile staging.  Slot q*NTHR + tid of a region is filled by this thread's q-th copy;
  // its source offset inside a tile does not depend on the tile and is computed once.
  // Padding slots copy the tile's first chunk (never read).
  int xoff[NQX], toff[NQT];
#pragma unroll
  for (int q = 0; q < NQX; ++q) {
    const int sl = q * NTHR + tid, r = sl / CX, at = sl % CX;
    const int c = CX == CPR ? at ^ row_swizzle<CPR>(r) : at;
    xoff[q] = (r < NT && c < CPR) ? r * PP * (int)sizeof(XG) + c * 16 * (int)sizeof(XG) / (int)sizeof(LX) : 0;
  }
#pragma unroll
  for (int q = 0; q < NQT; ++q) {
    const int sl = q * NTHR + tid, r = sl / CT, at = sl % CT;
    const int c = CT == CPT ? at ^ row_swizzle<CPT>(r) : at;
    toff[q] = (GRAD && r < PP && c < CPT) ? r * n_pad * (int)sizeof(XG) + c * 16 * (int)sizeof(XG) / (int)sizeof(LX) : 0;
  }
  const uint8_t *gxk = reinterpret_cast<const uint8_t *>(args.Xk);
  const uint8_t *gxt = reinterpret_cast<const uint8_t *>(args.Xt);

  // Asynchronous copy of one tile into a stage (global -> LDS DMA, 16 bytes per lane).
#define SPA_ISSUE(tile0_, stage_)                                                                        \
  do {                                                                                                   \
    const uint8_t *bx_ = gxk + (size_t)(tile0_) * PP * sizeof(XG);                                       \
    _Pragma("unroll") for (int q = 0; q < NQX; ++q)                                                      \
      lds_dma16(bx_ + xoff[q], smem + (stage_) * STG + q * NTHR + wave * 64);                           \
    if constexpr (GRAD) {                                                                                \
      const uint8_t *bt_ = gxt + (size_t)(tile0_) * sizeof(XG);                                          \
      _Pragma("unroll") for (int q = 0; q < NQT; ++q)                                                    \
        lds_dma16(bt_ + toff[q], smem + (stage_) * STG + XSL + q * NTHR + wave * 64);                   \
    }                                                                                                    \
  } while (0)
  // One of the NQX + NQT copy instructions of a tile (part < NQX: individual-major copy).
  auto issue_part = [&](const int tile0_, const int stage_, const int part) {
    if (part < NQX) {
      lds_dma16(gxk + (size_t)(tile0_) * PP * sizeof(XG) + xoff[part], smem + (stage_) * STG + part * NTHR + wave * 64);
    } else if constexpr (GRAD) {
      const int q = part - NQX;
      lds_dma16(gxt + (size_t)(tile0_) * sizeof(XG) + toff[q], smem + (stage_) * STG + XSL + q * NTHR + wave * 64);
    }
  };
  // FP8 storage: each 16-byte chunk of codes becomes two BF16 chunks, through registers.
#define SPA_COPY_FP8(tile0_, stage_)                                                                     \
  do {                                                                                                   \
    uint4 *sx_ = smem + (stage_) * STG;                                                                  \
    for (int c = tid; c < NT * PP / 16; c += NTHR) {                                                     \
      const int r = c / (PP / 16), cc = c % (PP / 16);                                                   \
      const uint4 v = *reinterpret_cast<const uint4 *>(gxk + (size_t)((tile0_) + r) * PP + cc * 16);     \
      const int s_ = row_swizzle<CPR>(r);                                                                \
      store_fp8_as_bf16(sx_ + r * CPR + ((2 * cc) ^ s_), sx_ + r * CPR + ((2 * cc + 1) ^ s_), v);        \
    }                                                                                                    \
    if constexpr (GRAD) {                                                                                \
      uint4 *st_ = smem + (stage_) * STG + XSL;                                                          \
      for (int c = tid; c < PP * NT / 16; c += NTHR) {                                                   \
        const int r = c / (NT / 16), cc = c % (NT / 16);                                                 \
        const uint4 v = *reinterpret_cast<const uint4 *>(gxt + (size_t)r * n_pad + (tile0_) + cc * 16); \
        const int s_ = row_swizzle<CPT>(r);                                                              \
        store_fp8_as_bf16(st_ + r * CPT + ((2 * cc) ^ s_), st_ + r * CPT + ((2 * cc + 1) ^ s_), v);      \
      }                                                                                                  \
    }                                                                                                    \
  } while (0)
  // FP8 storage, in two halves: the next tile's codes are loaded into registers at the
  // start of a tile (their latency hidden by the tile's MFMA work) and widened into the
  // idle stage at its end.
  constexpr int NFX = FP8 ? (NT * PP / 16 + NTHR - 1) / NTHR : 1;        // chunks per thread
  constexpr int NFT = (FP8 && GRAD) ? (PP * NT / 16 + NTHR - 1) / NTHR : 1;
  uint4 fx[NFX], ft[NFT];
  auto fp8_load = [&](const int tile0_) {
    if constexpr (FP8) {
#pragma unroll
      for (int u = 0; u < NFX; ++u) {
        const int c = tid + u * NTHR;
        if (c < NT * PP / 16) {
          const int r = c / (PP / 16), cc = c % (PP / 16);
          fx[u] = *reinterpret_cast<const uint4 *>(gxk + (size_t)(tile0_ + r) * PP + cc * 16);
        }
      }
      if constexpr (GRAD) {
#pragma unroll
        for (int u = 0; u < NFT; ++u) {
          const int c = tid + u * NTHR;
          if (c < PP * NT / 16) {
            const int r = c / (NT / 16), cc = c % (NT / 16);
            ft[u] = *reinterpret_cast<const uint4 *>(gxt + (size_t)r * n_pad + tile0_ + cc * 16);
          }
        }
      }
    }
  };
  auto fp8_store = [&](const int stage_) {
    if constexpr (FP8) {
      uint4 *sx_ = smem + stage_ * STG;
#pragma unroll
      for (int u = 0; u < NFX; ++u) {
        const int c = tid + u * NTHR;
        if (c < NT * PP / 16) {
          const int r = c / (PP / 16), cc = c % (PP / 16);
          const int s_ = row_swizzle<CPR>(r);
          store_fp8_as_bf16(sx_ + r * CPR + ((2 * cc) ^ s_), sx_ + r * CPR + ((2 * cc + 1) ^ s_), fx[u]);
        }
      }
      if constexpr (GRAD) {
        uint4 *st_ = smem + stage_ * STG + XSL;
#pragma unroll
        for (int u = 0; u < NFT; ++u) {
          const int c = tid + u * NTHR;
          if (c < PP * NT / 16) {
            const int r = c / (NT / 16), cc = c % (NT / 16);
            const int s_ = row_swizzle<CPT>(r);
            store_fp8_as_bf16(st_ + r * CPT + ((2 * cc) ^ s_), st_ + r * CPT + ((2 * cc + 1) ^ s_), ft[u]);
          }
        }
      }
    }
  };
  // Wait for this thread's copies, then make every wave's copies visible.
#define SPA_LAND()                                  \
  do {                                              \
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); \
    __syncthreads();                                \
  } while (0)

  if (ntiles > 0) {
    if constexpr (FP8) SPA_COPY_FP8(i0, 0);
    else SPA_ISSUE(i0, 0);
  }
  SPA_LAND();

  // One tile: forward -> elementwise -> adjoint per group of QB 16-individual blocks, while the
  // next tile's copy lands in the other stage.  MASKED: the tile holds padded individuals,
  // which happens only for the last tile holding real ones (peeled off the main loop, so the
  // main loop body is one straight block).
  auto tile_step = [&](const int it, auto masked_c) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int tile0 = i0 + it * NT;
    const int stage = it & 1;
    // the next tile's copy; unconditional: the last tile re-copies itself into the idle
    // stage (never read).  BF16: its instructions are spread over the first group's MFMA
    // loops (one per forward k-step, one per other adjoint block) rather than issued in
    // one burst, which stalls the wave's issue (measured: ~4 % of the kernel time).
    const int ntile0 = i0 + min(it + 1, ntiles - 1) * NT;
    if constexpr (FP8) {
      if (it + 1 < ntiles) fp8_load(ntile0);
    }
    constexpr bool SPREAD = (P == Prec::BF16X2) && !FP8 && (NKS >= NQX) && (NMB >= 2 * NQT);
    if constexpr (!FP8 && !SPREAD) SPA_ISSUE(ntile0, stage ^ 1);
    const uint4 *sX = smem + stage * STG;          // individual-major tile, CX slots per row
    const uint4 *sXt = sX + XSL;                   // marker-major tile, CT slots per row
    // rows ib * 16 + lr and mb * 16 + lr: the swizzle is that of row lr, its low two bits
    // and the rest (which the k-step's chunk number does not reach and meets, respectively)
    const int fx_lo = row_swizzle<CPR>(lr) & 3, fx_hi = row_swizzle<CPR>(lr) & ~3;
    const int ft_lo = row_swizzle<CPT>(lr) & 3, ft_hi = row_swizzle<CPT>(lr) & ~3;
    // ---- per group of QB 16-individual blocks: forward -> elementwise -> adjoint
#pragma unroll
    for (int q = 0; q < IB / QB; ++q) {
      // forward: eta^T blocks (individuals x particles)
      AC acc[QB][PB];
#pragma unroll
      for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[b][pb] = AC{0, 0, 0, 0};
      // BF16: fragments are read kPrefetch k-steps ahead of their MFMAs, and the k-steps are kept
      // apart (the scheduler, left alone, waits on every read right before its use): reads and
      // MFMAs with two waves per SIMD, whose vector work may move, all with one (forward, p =
      // 500: 366 us with the looser rule, 315 us with this one, 361 us without either).  The MFMAs
      // of a block's hi and lo parts alternate with those of the other block.
      auto xfrag = [&](const int ks, const int b) -> FR {
        const uint4 *row = sX + ((q * QB + b) * 16 + lr) * CX;
        // chunk 4 ks + lg (BF16); word lg of chunk ks (FP32)
        if constexpr (P == Prec::BF16X2) return *reinterpret_cast<const FR *>(row + ((4 * ks) ^ fx_hi) + (lg ^ fx_lo));
        else if constexpr (L::PAD) return reinterpret_cast<const FR *>(row)[4 * ks + lg];
        else return reinterpret_cast<const FR *>(row + (ks ^ (fx_hi | fx_lo)))[lg];
      };
      if constexpr (P == Prec::BF16X2) {
        static_assert(PB == 1, "one particle block per wave");
        constexpr int D = NKS < kPrefetch ? NKS : kPrefetch;
        FR a[D][QB];
#pragma unroll
        for (int ks = 0; ks < D; ++ks)
#pragma unroll
          for (int b = 0; b < QB; ++b) a[ks][b] = xfrag(ks, b);
        __builtin_amdgcn_sched_barrier(kKeepApart);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          if constexpr (SPREAD) {
            if (q == 0 && ks < NQX) issue_part(ntile0, stage ^ 1, ks);
          }
#pragma unroll
          for (int b = 0; b < QB; ++b) acc[b][0] = T::mfma(a[ks % D][b], bh[0][ks], acc[b][0]);
#pragma unroll
          for (int b = 0; b < QB; ++b) acc[b][0] = T::mfma(a[ks % D][b], bl[0][ks], acc[b][0]);
          if (ks + D < NKS) {
#pragma unroll
            for (int b = 0; b < QB; ++b) a[ks % D][b] = xfrag(ks + D, b);
          }
          __builtin_amdgcn_sched_barrier(kKeepApart);
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
          for (int b = 0; b < QB; ++b) {
            const FR a = xfrag(ks, b);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) acc[b][pb] = T::mfma(a, bh[pb][ks], acc[b][pb]);
          }
      }
      // the first fragments of the adjoint arrive during the elementwise step
      constexpr int DA = NMB < kPrefetch ? NMB : kPrefetch;
      auto tfrag = [&](const int mb) -> bf16x8 {   // this lane group's 8 K slots, contiguous
        return *reinterpret_cast<const bf16x8 *>(sXt + (mb * 16 + lr) * CPT + ((q * 4) ^ ft_hi) + (lg ^ ft_lo));
      };
      bf16x8 ta[DA];
      if constexpr (GRAD && P == Prec::BF16X2) {
#pragma unroll
        for (int mb = 0; mb < DA; ++mb) ta[mb] = tfrag(mb);
        __builtin_amdgcn_sched_barrier(kKeepApart);
      }

      if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
      // elementwise (lane: particle lr of each block, individuals crow(lg, v) of each block).
      // Padded genotype rows, ones column included, are zero: only the softplus sum masks them.
      EL sig[GRAD ? QB : 1][PB][4];
#define SPA_ELEMENTWISE(MASKED)                                                                   \
  _Pragma("unroll") for (int pb = 0; pb < PB; ++pb) {                                             \
      /* reduced precision: the operand carries log2(e), so z = eta log2(e); the genotypes  */    \
      /* are centred, so sum_k eta_ik = 0 over the real individuals and sum_k max(z, 0) is  */    \
      /* half of sum_k |z| (one add with an abs modifier per element instead of two ops)   */     \
      float prod = 1.0f, mx = 0.0f;                                                               \
      _Pragma("unroll") for (int b = 0; b < QB; ++b) _Pragma("unroll") for (int v = 0; v < 4; ++v) { \
        const float z = acc[b][pb][v] - moff[pb];                                                 \
        const float e = fast_exp2(-fabsf(z));                                                     \
        if (!(MASKED) || (tile0 + (q * QB + b) * 16 + T::crow(lg, v)) < n) {                      \
          prod = fmaf(prod, e, prod);                                                             \
          mx += fabsf(z);                                                                         \
        }                                                                                         \
        if constexpr (GRAD) {                                                                     \
          const float rc = fast_rcp(1.0f + e);                                                    \
          sig[b][pb][v] = z >= 0.0f ? rc : e * rc;                                                \
        }                                                                                         \
      }                                                                                           \
      spl[pb] += static_cast<double>(0.6931471805599453f * (0.5f * mx + fast_log2(prod)));       \
  }
      SPA_ELEMENTWISE(MASKED)
#undef SPA_ELEMENTWISE

      // adjoint: G^T (markers x particles) += X_tile^T . sigma^T
      if constexpr (GRAD) {
        if constexpr (P == Prec::BF16X2) {
          // K slot j of lane group lg: individual 4lg + j of block 2q (j < 4), of block 2q+1 (j >= 4)
          bf16x8 rh[PB], rl[PB];
#pragma unroll
          for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
              const f32x2 v = {sig[j >> 2][pb][j & 3], sig[j >> 2][pb][(j & 3) + 1]};
              const bf16x2 h = __builtin_convertvector(v, bf16x2);
              const f32x2 r = v - __builtin_convertvector(h, f32x2);
              const bf16x2 l = __builtin_convertvector(r, bf16x2);
              rh[pb][j] = h[0];
              rh[pb][j + 1] = h[1];
              rl[pb][j] = l[0];
              rl[pb][j + 1] = l[1];
            }
          if constexpr (PRIO) __builtin_amdgcn_s_setprio(2);
          static_assert(NMB % 2 == 0 && DA % 2 == 0, "adjoint blocks in pairs");
#pragma unroll
          for (int mb = 0; mb < NMB; mb += 2) {
            if constexpr (SPREAD) {
              if (q == 0 && mb / 2 < NQT) issue_part(ntile0, stage ^ 1, NQX + mb / 2);
            }
            // FP8 storage (more registers in use): alternating; else one block after the other
            // (measured: 1-2 % of a launch each way)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int b = FP8 ? k & 1 : k >> 1, lo = FP8 ? k >> 1 : k & 1;
              G[0][mb + b] = T::mfma(ta[(mb + b) % DA], lo ? rl[0] : rh[0], G[0][mb + b]);
            }
            if (mb + DA < NMB) {
#pragma unroll
              for (int b = 0; b < 2; ++b) ta[(mb + b) % DA] = tfrag(mb + b + DA);
            }
            __builtin_amdgcn_sched_barrier(kKeepApart);
          }
        } else {
          // 16x16x4: k-step v feeds the lane's v-th row, individual crow(lg, v)
#pragma unroll
          for (int mb = 0; mb < NMB; ++mb) {
            // the marker-major copy holds individuals crow(lg, 0..3) at positions 4lg..4lg+3
            const LX *row = reinterpret_cast<const LX *>(sXt + (mb * 16 + lr) * CT + (L::PAD ? lg : lg ^ ft_lo));
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const LX a = row[v];
#pragma unroll
              for (int pb = 0; pb < PB; ++pb) G[pb][mb] = T::mfma(a, sig[0][pb][v], G[pb][mb]);
            }
          }
        }
      }
    }

    if constexpr (FP8) {
      if (it + 1 < ntiles) fp8_store(stage ^ 1);
    }
    SPA_LAND();
  };
  const bool has_tail = ntiles > 0 && i0 + ntiles * NT > n;
  const int nfull = ntiles - (has_tail ? 1 : 0);
  for (int it = 0; it < nfull; ++it) tile_step(it, std::false_type{});
  if (has_tail) tile_step(nfull, std::true_type{});
#undef SPA_ISSUE
#undef SPA_COPY_FP8
#undef SPA_LAND


  // ---- softplus sums over the 4 lane groups sharing a particle
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    spl[pb] += __shfl_xor(spl[pb], 16, 64);
    spl[pb] += __shfl_xor(spl[pb], 32, 64);
  }

  const int M = args.M, p = args.p;
  using GO = float;
  if (S == 1) {
    // ---- epilogue: log-likelihood and standardised gradient
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      const int i = wbase + pb * 16 + lr;
      if (lg == 0 && i < M) args.ll[i] = args.yb[i] - spl[pb];
      if constexpr (GRAD) {
        // rho_i = sum_k sigma_ik: the all-ones column PP-1 (block NMB-1, lane group 3, element 3)
        const double rho = static_cast<double>(__shfl(G[pb][NMB - 1][3], lr + 48, 64));
        if (i < M) {
          GO *g = reinterpret_cast<GO *>(args.g) + static_cast<size_t>(i) * p;
#pragma unroll
          for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int j = mb * 16 + T::crow(lg, v);
              if (j < p)
                g[j] = static_cast<GO>(args.ytil[j] -
                                       (static_cast<double>(G[pb][mb][v]) - args.mu[j] * rho) * args.inv_s[j]);
            }
        }
      }
    }
  } else {
    // ---- partial sums of this split (combined in split order by the finalize kernel)
    const size_t Mp = static_cast<size_t>(args.M_pad);
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      const int i = wbase + pb * 16 + lr;
      if (lg == 0) args.spl_part[split * Mp + i] = spl[pb];
      if constexpr (GRAD) {
        GO *gp = reinterpret_cast<GO *>(args.g_part) + (split * Mp + i) * PP;
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) {
          *reinterpret_cast<f32x4 *>(gp + mb * 16 + lg * 4) = G[pb][mb];
        }
      }
    }
  }
}

// Split-marker form of the BF16 hi+lo contraction with the adjoint, for rows of 384 or 512
// markers.  A workgroup of 4 wave64s (one per SIMD, so that a wave has all 512 registers)
// owns 64 particles: the two waves of a pair share two blocks of 16 particles and each holds
// one half of the markers: coefficient fragments (hi and lo) and adjoint accumulators of both
// blocks.  Every genotype fragment read from LDS feeds four MFMAs.  Each wave adds up the
// forward sums of its half, hands those of the other wave's block over through LDS (float
// addition commutes), evaluates the elementwise step of its own block and hands its logistic
// values, already split in hi and lo, over for the adjoint.
//
// The three stages are those of three tiles of 32 individuals, one barrier per step: in step
// t the forward sums of tile t + 2, the elementwise step of tile t + 1 and the adjoint of tile
// t, independent of each other, so that the vector work runs beside the MFMAs of the same
// wave.  The last adjoint group of a step is left to the start of the next: its fragments are in
// registers, so it runs while the first LDS reads after the barrier are on their way.  Tiles are
// copied from HBM to LDS directly, D = buffers - 1 steps ahead, as they are stored: FP8 codes are widened when a fragment is read (four conversions for four MFMAs), which
// halves the LDS traffic of a tile and leaves room for a third buffer.  16-byte chunks of a row
// are permuted by the row's number so that the fragment reads of 16 rows hit distinct banks.
// The same arithmetic per element as loglik_kernel; a forward sum is formed as the sum of two
// half sums.
//
// What bounds it: a single wave per SIMD issues its 128 MFMAs (2048 cycles) and some 320 vector
// instructions per step one after the other, about 4000 cycles.  It replaced a form of 8 waves
// with 16 particles each, three barriers per tile, genotypes widened on their way to LDS and the
// elementwise step done by both waves of a pair, whose fragment reads alone took all of the LDS
// bandwidth.  32768 particles, n = 10000, p = 500, FP8: 1529 -> 1070 us per launch (1.25 PFLOP/s of
// executed MFMA); BF16: 4240 -> 1110 us.
template <int PP, bool FP8>
struct Wide {
  static constexpr int NT = 32, NTHR = 256, WGP = 64;
  static constexpr int ES = FP8 ? 1 : 2;                    // bytes of a genotype
  static constexpr int XB = NT * PP * ES;                   // bytes of a tile (either order)
  static constexpr int NBUF = FP8 ? 3 : 2;
  static constexpr int EX = 4 * 64 * 32;                    // exchange: 32 bytes per lane, twice
  static constexpr size_t bytes = (size_t)2 * NBUF * XB + 4 * EX;
};

template <int PP, bool FP8>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256))) __attribute__((amdgpu_waves_per_eu(1, 1)))
void loglik_wide_kernel(GemmArgs args) {
  constexpr Prec P = Prec::BF16X2;
  using T = GT<P>;
  using FR = bf16x8;
  using AC = f32x4;
  using W = Wide<PP, FP8>;
  constexpr int KS = 32, KV = 8, NT = W::NT, NTHR = W::NTHR, WGP = W::WGP, ES = W::ES, XB = W::XB;
  constexpr int NBUF = W::NBUF, D = NBUF - 1;
  constexpr int H = PP / 2;                      // markers per half
  constexpr int NKH = H / KS, NMH = H / 16;      // forward k-steps, adjoint blocks per half
  constexpr int CPR = PP * ES / 16, CPT = NT * ES / 16;   // chunks of a row of either order
  constexpr int NQ = XB / 16 / NTHR;             // copies per thread, tile and order
  static_assert(PP == 384 || PP == 512, "rows of 384 or 512 markers");
  static_assert(XB % (16 * NTHR) == 0 && NMH % 2 == 0, "whole copies, pairs of adjoint blocks");

  extern __shared__ __align__(16) uint4 smem[];
  uint8_t *lx = reinterpret_cast<uint8_t *>(smem), *lt = lx + NBUF * XB;
  uint8_t *esum = lt + NBUF * XB, *esig = esum + 2 * W::EX;

  const int S = args.S;
  const int g8 = 8 / S;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int split = xcd / g8;
  const int ptile = slot * g8 + (xcd % g8);
  const int ntiles_p = (args.M + WGP - 1) / WGP;
  if (ptile >= ntiles_p) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int half = wave & 1;                     // markers half * H ...; particle block of its own
  const int pbase = ptile * WGP + (wave >> 1) * 32;
  const int n = args.n, n_pad = args.n_pad;
  const int chunk = ((n_pad + S - 1) / S + NT - 1) / NT * NT;
  const int i0 = min(n_pad, split * chunk);
  const int i1 = min(min(n_pad, i0 + chunk), (n + NT - 1) / NT * NT);
  const int ntiles = max(0, (i1 - i0) / NT);

  // [0]: the wave's own particle block, [1]: its partner's
  FR bh[2][NKH], bl[2][NKH];
  float moff;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const size_t row = static_cast<size_t>(pbase + (half ^ q) * 16 + lr);
    const __bf16 *sh = reinterpret_cast<const __bf16 *>(args.Bhi) + row * PP + half * H + lg * KV;
    const __bf16 *sl = reinterpret_cast<const __bf16 *>(args.Blo) + row * PP + half * H + lg * KV;
#pragma unroll
    for (int ks = 0; ks < NKH; ++ks) {
      bh[q][ks] = *reinterpret_cast<const FR *>(sh + ks * KS);
      bl[q][ks] = *reinterpret_cast<const FR *>(sl + ks * KS);
    }
    if (q == 0) moff = static_cast<float>(args.moff[row]);
  }
  AC G[2][NMH];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int mb = 0; mb < NMH; ++mb) G[q][mb] = AC{0, 0, 0, 0};
  double spl = 0.0;

  // ---- tile copies: this thread's chunk of copy q, at slot q * NTHR + tid of the buffer
  const uint8_t *gx = reinterpret_cast<const uint8_t *>(args.Xk) + (size_t)i0 * PP * ES;
  const uint8_t *gt = reinterpret_cast<const uint8_t *>(args.Xt) + (size_t)i0 * ES;
  int xoff[NQ], toff[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int sl = q * NTHR + tid;
    const int rx = sl / CPR, rt = sl / CPT;
    xoff[q] = rx * PP * ES + ((sl % CPR) ^ row_swizzle<CPR>(rx)) * 16;
    toff[q] = rt * n_pad * ES + ((sl % CPT) ^ row_swizzle<CPT>(rt)) * 16;
  }
  // copy c of a step: the individual-major tile t + 2 + D, then the marker-major tile t + D
  // (clamped: a copy past the ends is not read, and the number in flight stays the same)
  auto copy = [&](const int t, const int c) {
    const int tile = c < NQ ? t + 2 + D : t + D, q = c < NQ ? c : c - NQ;
    const size_t at = (size_t)min(max(tile, 0), ntiles - 1) * NT;
    const uint8_t *src = c < NQ ? gx + at * PP * ES + xoff[q] : gt + at * ES + toff[q];
    uint8_t *dst = (c < NQ ? lx : lt) + (tile + NBUF) % NBUF * XB;
    lds_dma16(src, reinterpret_cast<uint4 *>(dst) + q * NTHR + wave * 64);
  };
  // a fragment's 8 genotypes as stored, and as BF16
  using RAW = typename std::conditional<FP8, u32x2, FR>::type;
  auto widen = [](const RAW v) -> FR {
    if constexpr (FP8) {
      FR o;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t w = v[k / 2];
        const bf16x2 c = (k & 1) ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true)
                                 : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
        o[2 * k] = c[0];
        o[2 * k + 1] = c[1];
      }
      return o;
    } else {
      return v;
    }
  };
  int xa[NKH];                                   // byte of the wave's fragment ks in a row tile
#pragma unroll
  for (int ks = 0; ks < NKH; ++ks) {
    const int at = half * H + ks * KS + lg * KV;           // first marker
    xa[ks] = lr * PP * ES + ((at * ES / 16) ^ row_swizzle<CPR>(lr)) * 16 + at * ES % 16;
  }
  const int ta = (half * H + lr) * NT * ES + ((lg * KV * ES / 16) ^ row_swizzle<CPT>(lr)) * 16 + lg * KV * ES % 16;

  AC own[2];                                     // forward sums of this half, the own block's
  FR rh, rl;                                     // logistic values of the own block, hi and lo
  FR ca[2], ch[2], cl[2];                        // the last adjoint group of a step is done in the next
  // Step t: forward of tile t + 2, elementwise of tile t + 1, adjoint of tile t, in NG groups of
  // eight MFMAs (a forward k-step, or two adjoint blocks) that the scheduler keeps apart, each
  // with its part of the rest: the next group's fragments widened, the fragments of the one after
  // it read, copies issued, one of the lane's eight elements.  (Left alone, the scheduler gathers the
  // adjoint's reads and spills accumulators to and fro.)  MASKED: tile t + 1 may hold padded
  // individuals (whose genotypes, ones column included, are zero: only the softplus sum leaves
  // them out).
  constexpr int NG = NKH + NMH / 2;
  constexpr int CPG = D == 1 ? 2 : 1;            // copies per group: one buffer ahead, early
  static_assert(NG >= 12 && CPG * NG >= 2 * NQ, "eight elements, their values and every copy find a group");
  auto step = [&](const int t, auto fwd_c, auto el_c, auto adj_c, auto carry_c, auto masked_c) {
    constexpr bool FWD = decltype(fwd_c)::value, EL = decltype(el_c)::value, ADJ = decltype(adj_c)::value;
    constexpr bool CARRY = decltype(carry_c)::value, MASKED = decltype(masked_c)::value;
    constexpr int first = FWD ? 0 : NKH, last = ADJ ? NG : FWD ? NKH : 0;   // groups with MFMAs
    const int par = t & 1;
    const uint8_t *sx = lx + (t + 2) % NBUF * XB, *st = lt + (t + NBUF) % NBUF * XB + ta;
    // the partner's sums of the own block (tile t + 1) and logistic values of its block (tile t)
    const uint8_t *rs = esum + (par ^ 1) * W::EX + ((wave ^ 1) * 64 + lane) * 16;
    const uint8_t *rg = esig + par * W::EX + ((wave ^ 1) * 64 + lane) * 16;
    uint8_t *ws = esum + par * W::EX + (wave * 64 + lane) * 16;
    uint8_t *wg = esig + (par ^ 1) * W::EX + (wave * 64 + lane) * 16;
    auto read = [&](const int g, const int b) -> RAW {   // group g's fragments
      return *reinterpret_cast<const RAW *>(g < NKH ? sx + xa[g] + b * 16 * PP * ES
                                                    : st + (2 * (g - NKH) + b) * 16 * NT * ES);
    };
    RAW raw[2][2];
    FR a[2], na[2];
#pragma unroll
    for (int g = first; g < min(first + 2, last); ++g)
#pragma unroll
      for (int b = 0; b < 2; ++b) raw[(g - first) & 1][b] = read(g, b);
    AC z[2], acc[2][2];
    FR oh, ol;
    const FR ph = rh, pl = rl;                   // the own block's, tile t
    if constexpr (EL) {
#pragma unroll
      for (int b = 0; b < 2; ++b) z[b] = *reinterpret_cast<const AC *>(rs + b * (W::EX / 2));
    }
    if constexpr (ADJ) {
      oh = *reinterpret_cast<const FR *>(rg);
      ol = *reinterpret_cast<const FR *>(rg + W::EX / 2);
    }
    if constexpr (CARRY) {
      constexpr int mb = NMH - 2;
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int b = 0; b < 2; ++b) G[q][mb + b] = T::mfma(ca[b], x ? cl[q] : ch[q], G[q][mb + b]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (first < last) {
#pragma unroll
      for (int b = 0; b < 2; ++b) a[b] = widen(raw[0][b]);
    }
    float prod = 1.0f, mx = 0.0f, sig[8];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (g >= first && g < last) {
        if (g + 1 < last) {
#pragma unroll
          for (int b = 0; b < 2; ++b) na[b] = widen(raw[(g + 1 - first) & 1][b]);
        }
        if (g + 2 < last) {
#pragma unroll
          for (int b = 0; b < 2; ++b) raw[(g - first) & 1][b] = read(g + 2, b);
        }
        if (g < NKH) {
#pragma unroll
          for (int x = 0; x < 2; ++x)            // hi, lo
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
              for (int b = 0; b < 2; ++b)
                acc[q][b] = T::mfma(a[b], x ? bl[q][g] : bh[q][g], g == 0 && x == 0 ? AC{0, 0, 0, 0} : acc[q][b]);
        } else if (g < NG - 1) {
          const int mb = 2 * (g - NKH);
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
              for (int b = 0; b < 2; ++b)
                G[q][mb + b] = T::mfma(a[b], x ? (q ? ol : pl) : (q ? oh : ph), G[q][mb + b]);
        }
      }
#pragma unroll
      for (int c = CPG * g; c < CPG * (g + 1); ++c)
        if (c < 2 * NQ) copy(t, c);
      if constexpr (EL) {
        if (g == 0) {
#pragma unroll
          for (int b = 0; b < 2; ++b) z[b] += own[b];
        } else if (g <= 8) {
          const int e = g - 1;
          const float y = z[e >> 2][e & 3] - moff;
          const float x = fast_exp2(-fabsf(y));
          if (!MASKED || (i0 + (t + 1) * NT + (e >> 2) * 16 + T::crow(lg, e & 3)) < n) {
            prod = fmaf(prod, x, prod);
            mx += fabsf(y);
          }
          const float rc = fast_rcp(1.0f + x);
          sig[e] = y >= 0.0f ? rc : x * rc;
        }
        if (g == 9) spl += static_cast<double>(0.6931471805599453f * (0.5f * mx + fast_log2(prod)));
        if (g >= 8 && g < 12) {
          const int j = 2 * (g - 8);
          const f32x2 v = {sig[j], sig[j + 1]};
          const bf16x2 h = __builtin_convertvector(v, bf16x2);
          const f32x2 r = v - __builtin_convertvector(h, f32x2);
          const bf16x2 l = __builtin_convertvector(r, bf16x2);
          rh[j] = h[0];
          rh[j + 1] = h[1];
          rl[j] = l[0];
          rl[j + 1] = l[1];
        }
        if (g == 11) {
          *reinterpret_cast<FR *>(wg) = rh;
          *reinterpret_cast<FR *>(wg + W::EX / 2) = rl;
        }
      }
      if constexpr (FWD) {
        if (g == NKH + 1) {                      // the last MFMAs of the sums are over
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            own[b] = acc[0][b];
            *reinterpret_cast<AC *>(ws + b * (W::EX / 2)) = acc[1][b];
          }
        }
      }
      if (g >= first && g + 1 < last) {
#pragma unroll
        for (int b = 0; b < 2; ++b) a[b] = na[b];
      }
      if (ADJ && g == NG - 2) {
#pragma unroll
        for (int b = 0; b < 2; ++b) ca[b] = na[b];
        ch[0] = ph;
        cl[0] = pl;
        ch[1] = oh;
        cl[1] = ol;
      }
      if (FP8 && g >= first && g < last) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {            // three vector instructions fit behind an MFMA
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // this step's LDS writes, and the copies that the next step reads (issued D - 1 steps ago or
    // before); not __syncthreads, which would wait for every copy
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((D - 1) * 2 * NQ) : "memory");
  };
  const std::true_type yes{};
  const std::false_type no{};
  if (ntiles > 0) {
#pragma unroll
    for (int t = 0; t < D; ++t)
#pragma unroll
      for (int c = 0; c < NQ; ++c) copy(t - 2 - D, c);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    step(-2, yes, no, no, no, no);
    if (ntiles > 2) {
      step(-1, yes, yes, no, no, no);
      step(0, yes, yes, yes, no, no);
      for (int t = 1; t < ntiles - 2; ++t) step(t, yes, yes, yes, yes, no);
      step(ntiles - 2, no, yes, yes, yes, yes);
      step(ntiles - 1, no, no, yes, yes, no);
    } else if (ntiles > 1) {
      step(-1, yes, yes, no, no, yes);
      step(0, no, yes, yes, no, yes);
      step(1, no, no, yes, yes, no);
    } else {
      step(-1, no, yes, no, no, yes);
      step(0, no, no, yes, no, no);
    }
    {                                            // the carried group of the last tile
      constexpr int mb = NMH - 2;
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int b = 0; b < 2; ++b) G[q][mb + b] = T::mfma(ca[b], x ? cl[q] : ch[q], G[q][mb + b]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                             // no copy and no read of the tiles is left
  }

  spl += __shfl_xor(spl, 16, 64);
  spl += __shfl_xor(spl, 32, 64);
  const int M = args.M, p = args.p;
  if (S == 1) {
    // rho_i = sum_k sigma_ik sits in the all-ones column PP-1 of the upper half
    float *rhob = reinterpret_cast<float *>(smem) + (wave >> 1) * 32 + lr;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float v = __shfl(G[q][NMH - 1][3], lr + 48, 64);
      if (half == 1 && lg == 0) rhob[(half ^ q) * 16] = v;
    }
    __syncthreads();
    const int own_i = pbase + half * 16 + lr;
    if (lg == 0 && own_i < M) args.ll[own_i] = args.yb[own_i] - spl;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int i = pbase + (half ^ q) * 16 + lr;
      const double rho = static_cast<double>(rhob[(half ^ q) * 16]);
      if (i < M) {
        float *g = reinterpret_cast<float *>(args.g) + static_cast<size_t>(i) * p;
#pragma unroll
        for (int mb = 0; mb < NMH; ++mb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int j = (half * NMH + mb) * 16 + T::crow(lg, v);
            if (j < p)
              g[j] = static_cast<float>(args.ytil[j] - (static_cast<double>(G[q][mb][v]) - args.mu[j] * rho) * args.inv_s[j]);
          }
      }
    }
  } else {
    const size_t Mp = static_cast<size_t>(args.M_pad);
    if (lg == 0) args.spl_part[split * Mp + pbase + half * 16 + lr] = spl;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const size_t i = static_cast<size_t>(pbase + (half ^ q) * 16 + lr);
      float *gp = reinterpret_cast<float *>(args.g_part) + (split * Mp + i) * PP + half * H;
#pragma unroll
      for (int mb = 0; mb < NMH; ++mb) *reinterpret_cast<f32x4 *>(gp + mb * 16 + lg * 4) = G[q][mb];
    }
  }
}

// Sum the S partials of every particle in split order and apply the epilogue.
template <typename GO, bool GRAD>
__global__ void gemm_finalize_kernel(GemmArgs args, int PP) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (i >= args.M) return;
  const size_t Mp = static_cast<size_t>(args.M_pad);
  const int S = args.S, p = args.p;
  if (lane == 0) {
    double spl = 0.0;
    for (int s = 0; s < S; ++s) spl += args.spl_part[s * Mp + i];
    args.ll[i] = args.yb[i] - spl;
  }
  if constexpr (GRAD) {
    const GO *gp = reinterpret_cast<const GO *>(args.g_part);
    double rho = 0.0;
    for (int s = 0; s < S; ++s) rho += static_cast<double>(gp[(s * Mp + i) * PP + PP - 1]);
    GO *g = reinterpret_cast<GO *>(args.g) + static_cast<size_t>(i) * p;
    for (int j = lane; j < p; j += 64) {
      double acc = 0.0;
      for (int s = 0; s < S; ++s) acc += static_cast<double>(gp[(s * Mp + i) * PP + j]);
      g[j] = static_cast<GO>(args.ytil[j] - (acc - args.mu[j] * rho) * args.inv_s[j]);
    }
  }
}

// ------------------------------------------------------------------- dispatch

static const int kPadBF[] = {32, 64, 128, 224, 256, 384, 512};
static const int kPad64[] = {32, 64, 128, 224, 256};

int gemm_pad_markers(int p, Prec prec) {
  const int need = p + 1;   // + the all-ones column
  if (prec == Prec::F64) {
    for (int v : kPad64)
      if (v >= need) return v;
    return -1;
  }
  for (int v : kPadBF)
    if (v >= need) return v;
  return -1;
}

int gemm_tile_individuals(Prec prec, int PP) {
  return prec == Prec::BF16X2 ? (PP <= 256 ? 64 : 32) : 16;
}

int gemm_particles_per_wg(Prec prec, int PP) {
  return prec == Prec::F64 ? 64 : (PP <= 256 ? 128 : 64);
}

int gemm_splits(Prec prec, int PP, int n_pad, int M, size_t x_bytes_both) {
  const int NT = gemm_tile_individuals(prec, PP);
  const int tiles_p = (M + gemm_particles_per_wg(prec, PP) - 1) / gemm_particles_per_wg(prec, PP);
  int S = 1;
  // keep one split's genotype slice (both orientations) within an XCD's L2 ...
  while (S < 8 && x_bytes_both / S > (size_t)3 * 1024 * 1024 && n_pad / (2 * S) >= NT) S *= 2;
  // ... and give every CU a workgroup
  while (S < 8 && (size_t)tiles_p * S < 256 && n_pad / (2 * S) >= NT) S *= 2;
  return S;
}

template <Prec P, int PP, bool GRAD, bool FP8>
static hipError_t launch_one(const GemmArgs &a, hipStream_t s) {
  constexpr size_t lds = Lds<P, PP, GRAD>::bytes;
  static_assert(lds <= 160 * 1024, "LDS budget of one CU");
  auto kern = loglik_kernel<P, PP, GRAD, FP8>;
  static OncePerDevice once;
  const hipError_t e = raise_lds_limit(once, kern, lds);
  if (e != hipSuccess) return e;
  constexpr int per_wg = Shape<P, PP>::WGP;
  const int tiles_p = (a.M + per_wg - 1) / per_wg;
  const int g8 = 8 / a.S;
  const int grid = 8 * ((tiles_p + g8 - 1) / g8);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(Shape<P, PP>::NTHR), lds, s, a);
  return hipGetLastError();
}

template <int PP, bool FP8>
static hipError_t launch_wide(const GemmArgs &a, hipStream_t s) {
  constexpr size_t lds = Wide<PP, FP8>::bytes;
  static_assert(lds <= 160 * 1024, "LDS budget of one CU");
  auto kern = loglik_wide_kernel<PP, FP8>;
  static OncePerDevice once;
  const hipError_t e = raise_lds_limit(once, kern, lds);
  if (e != hipSuccess) return e;
  const int tiles_p = (a.M + 63) / 64;
  const int g8 = 8 / a.S;
  const int grid = 8 * ((tiles_p + g8 - 1) / g8);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(Wide<PP, FP8>::NTHR), lds, s, a);
  return hipGetLastError();
}

template <Prec P, int PP>
static hipError_t launch_pp(const GemmArgs &a, hipStream_t s) {
  if constexpr (P == Prec::BF16X2 && (PP == 384 || PP == 512)) {
    if (a.grad) return a.x_fp8 ? launch_wide<PP, true>(a, s) : launch_wide<PP, false>(a, s);
  }
  if constexpr (P == Prec::BF16X2) {
    if (a.x_fp8) {
      if (a.grad) return launch_one<P, PP, true, true>(a, s);
      return launch_one<P, PP, false, true>(a, s);
    }
  }
  if (a.grad) return launch_one<P, PP, true, false>(a, s);
  if constexpr (P == Prec::BF16X2) return launch_one<P, PP, false, false>(a, s);
  return hipErrorInvalidValue;   // forward FP32 is streamed
}

hipError_t launch_gemm_finalize(const GemmArgs &a, hipStream_t s) {
  if (a.S == 1) return hipSuccess;
  const int grid = (a.M + 3) / 4;
  if (a.grad) hipLaunchKernelGGL((gemm_finalize_kernel<float, true>), dim3(grid), dim3(256), 0, s, a, a.PP);
  else hipLaunchKernelGGL((gemm_finalize_kernel<float, false>), dim3(grid), dim3(256), 0, s, a, a.PP);
  return hipGetLastError();
}

hipError_t launch_loglik(const GemmArgs &a, hipStream_t s) {
  if (a.S != 1 && a.S != 2 && a.S != 4 && a.S != 8) return hipErrorInvalidValue;
  if (a.M_pad % gemm_particles_per_wg(a.prec, a.PP) != 0) return hipErrorInvalidValue;
  switch (a.prec) {
    case Prec::BF16X2:
      switch (a.PP) {
        case 32: return launch_pp<Prec::BF16X2, 32>(a, s);
        case 64: return launch_pp<Prec::BF16X2, 64>(a, s);
        case 128: return launch_pp<Prec::BF16X2, 128>(a, s);
        case 224: return launch_pp<Prec::BF16X2, 224>(a, s);
        case 256: return launch_pp<Prec::BF16X2, 256>(a, s);
        case 384: return launch_pp<Prec::BF16X2, 384>(a, s);
        case 512: return launch_pp<Prec::BF16X2, 512>(a, s);
      }
      break;
    case Prec::F32:
      switch (a.PP) {
        case 32: return launch_pp<Prec::F32, 32>(a, s);
        case 64: return launch_pp<Prec::F32, 64>(a, s);
        case 128: return launch_pp<Prec::F32, 128>(a, s);
        case 224: return launch_pp<Prec::F32, 224>(a, s);
        case 256: return launch_pp<Prec::F32, 256>(a, s);
        case 384: return launch_pp<Prec::F32, 384>(a, s);
        case 512: return launch_pp<Prec::F32, 512>(a, s);
      }
      break;
    case Prec::F64:   // streamed
      break;
  }
  return hipErrorInvalidValue;
}

}  // namespace spa
