// Launch interface of the streamed FP32/FP64 contraction (see spa_stream.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spa_common.hpp"
#include "spa_internal.hpp"

namespace spa {

// Genotype codes for the K = 4 MFMAs, one byte per entry, in blocks of 16 individuals:
//   Xb [(block * 64 + lane) * stride + d], byte q: code of individual lane % 16 of the
//     block and marker 16 d + 4 q + lane / 16 (the lane's A operand of k-step 4 d + q);
//   Xtb[(block * 64 + lane) * stride + d], byte v: code of the block's individual
//     lane / 16 + 4 v (the FP64 MFMA's output rows) and marker 16 d + lane % 16, the A operands of
//     the FP64 adjoint.
// Entries outside the n x p genotypes are 0.
__host__ __device__ inline int stream_dwords(int p) { return (p + 15) / 16; }
__host__ __device__ inline int stream_stride(int p) {   // dwords per lane and block: 4-, 8- or 16-byte loads
  const int nd = stream_dwords(p);
  return nd <= 2 ? nd : (nd + 3) / 4 * 4;
}
inline int stream_blocks(int n) { return (n + 15) / 16; }
inline size_t stream_bytes(int n, int p) { return (size_t)stream_blocks(n) * 64 * 4 * stream_stride(p); }
hipError_t launch_stream_pack(const uint8_t *X, int n, int p, uint32_t *Xb, hipStream_t s);
hipError_t launch_stream_pack_adjoint(const uint8_t *X, int n, int p, uint32_t *Xtb, hipStream_t s);

struct StreamArgs {
  Prec prec;               // F32 or F64
  bool grad;
  const uint32_t *Xb, *Xtb;   // Xtb: gradients only
  int n, p, M;
  // operand: the particles themselves (packed by the kernel), or, with beta null, the
  // rows written by the proposal step
  const void *beta;        // M x p
  int beta_f64;
  const void *B;           // M_pad x PP scaled coefficients (float or double)
  const double *moff;      // M_pad (with B)
  const double *mu, *s, *inv_s, *ytil;
  int PP;                  // row length of B and of g_part
  int S;                   // ranges of individuals
  size_t Mp;               // rows per range of the partials
  double *spl_part;        // S x Mp softplus sums, or null (S == 1, no gradient): ll is written
  void *g_part;            // S x Mp x PP adjoints, sum_k sigma_ik in column PP - 1 (grad)
  double *yb;              // M: written when beta is given, read otherwise
  double *ll;              // M: yb - sum softplus
};

// Particles per workgroup (rows of the partials are padded to it).
constexpr int kStreamRows = 16;
// Most bytes of a log-likelihood call's partials (half of the array that calls without
// allocation use, which take the same ranges).
constexpr size_t kStreamPartialBytes = size_t(16) << 20;
// Ranges of individuals for M particles, at most smax (a power of two).
int stream_splits(Prec prec, bool grad, int n, int p, int M, int smax);
hipError_t launch_stream(const StreamArgs &a, hipStream_t s);

// Sum of the partials in range order and the outputs: ll, and (with g) the gradient in
// FP64, plus the prior's when `prior` is given, rounded once to the output type; logpost
// (nullable): ll + log prior.
struct StreamFinal {
  const StreamArgs *a;
  const Prior *prior;      // null: likelihood only
  void *g;                 // M x p (null: no gradient)
  int g_f64;
  double *logpost;
  int part_f32;            // g_part is float (the tiled contractions), else double
};
hipError_t launch_stream_finalize(const StreamFinal &f, hipStream_t s);

// All the random-walk sweeps of a scale (or one burn-in sweep) in one launch.
struct RwmArgs {
  Prec prec;
  const uint32_t *Xb;
  int n, p, M;
  void *beta;              // M x p state, updated
  double *ll;              // M state log-likelihoods, updated
  const double *mu, *s, *inv_s, *ytil, *sigma;
  Prior prior;
  int sweeps, sweep0;      // Philox sweep index of the first one
  int t;
  uint32_t k0, k1;
  double step;             // used when adapt is null
  // burn-in: the step size is a function of the previous sweep's step and accept count
  // (ring of three slots, slot k = sweep % 3): step_k = step_(k-1) exp(clip(count_(k-1)/M -
  // target, +-log 2)); the launch counts into its own slot and clears the next one
  double *ring_step;       // 3, or null
  unsigned long long *ring_cnt;
  int first, adapt;
  double target;
  unsigned long long *count;   // 2: accepted proposals, non-finite log-likelihoods (added to)
};
// Whether the sweeps of a random-walk scale are better run by one launch.
bool rwm_one_launch(Prec prec, int n, int p, int M);
hipError_t launch_rwm_sweeps(const RwmArgs &a, hipStream_t s);

}  // namespace spa
