// Cross-lane reductions of a wave64 by DPP moves (and one swizzle), in fixed orders.
#pragma once

#include <hip/hip_runtime.h>

namespace spa {

// DPP moves of a double (two 32-bit moves) and of a float (lanes of rows outside ROWS read
// 0); ds_swizzle exchange of lanes i and i ^ 16 inside each group of 32 lanes; a double
// read from one lane.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_move_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, ROWS, 0xf, false);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp_move_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ double swizzle_xor16_f64(double v) {
  constexpr int kXor16 = 0x1f | (0x10 << 10);   // bit mode: and 0x1f, or 0, xor 0x10
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_ds_swizzle(static_cast<int>(b), kXor16);
  const int hi = __builtin_amdgcn_ds_swizzle(static_cast<int>(b >> 32), kXor16);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}
__device__ __forceinline__ double read_lane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(b), l);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), l);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// Sum over groups of LP lanes (a particle's row), the same value in every lane of a group: a
// butterfly of pairwise sums (each step adds a lane's value to its partner's, so both
// hold the same sum: addition commutes) by DPP quad permutations (lanes i ^ 1, i ^ 2), the
// half-row and row mirrors (i ^ 7, i ^ 15 inside 8 and 16 lanes), a swizzle (i ^ 16) and,
// for 64 lanes, the two halves read from lanes 0 and 32.
template <int LP>
__device__ __forceinline__ double lane_group_sum(double v) {
  static_assert(LP == 8 || LP == 16 || LP == 32 || LP == 64, "groups of 8 to 64 lanes");
  v += dpp_move_f64<0xB1>(v);                         // quad_perm [1,0,3,2]
  v += dpp_move_f64<0x4E>(v);                         // quad_perm [2,3,0,1]
  v += dpp_move_f64<0x141>(v);                        // row_half_mirror
  if constexpr (LP >= 16) v += dpp_move_f64<0x140>(v);  // row_mirror
  if constexpr (LP >= 32) v += swizzle_xor16_f64(v);
  if constexpr (LP == 64) v = read_lane_f64(v, 0) + read_lane_f64(v, 32);
  return v;
}

// Sum over the 64 lanes of a wave in a fixed order, returned in every lane: butterflies
// inside each row of 16 lanes (quad permutations, half-row and row mirrors), the row totals
// chained by the row-15 and row-31 broadcasts, the total read from lane 63.  Six dependent
// DPP steps instead of six dependent cross-lane permutes through the LDS unit.
__device__ __forceinline__ double wave_last_f64(double v) {   // the total, in lane 63 only
  v += dpp_move_f64<0xB1>(v);        // quad_perm [1,0,3,2]
  v += dpp_move_f64<0x4E>(v);        // quad_perm [2,3,0,1]
  v += dpp_move_f64<0x141>(v);       // row_half_mirror
  v += dpp_move_f64<0x140>(v);       // row_mirror
  v += dpp_move_f64<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_move_f64<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ double wave_total_f64(double v) { return read_lane_f64(wave_last_f64(v), 63); }
__device__ __forceinline__ float wave_total_f32(float v) {
  v += dpp_move_f32<0xB1>(v);
  v += dpp_move_f32<0x4E>(v);
  v += dpp_move_f32<0x141>(v);
  v += dpp_move_f32<0x140>(v);
  v += dpp_move_f32<0x142, 0xA>(v);
  v += dpp_move_f32<0x143, 0xC>(v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Chunk c of row r of a tile with C chunks (16 bytes each) per row lies at slot
// r C + (c ^ row_swizzle<C>(r)).  A 16-byte read of a wave is served in four parts of 16 lanes, of
// two neighbouring lane groups g and g ^ 1: rows 0..3 and 12..15 of one, 4..11 of the other.  The
// numbers here put chunk g of the former and g ^ 1 of the latter at the 16 positions of a line of
// the 64 banks, once each (checked by the bank-conflict counter).  Rows padded to an odd stride
// do so for 16 rows of one lane group only: every fragment read takes 8 cycles for 4.  (FP32
// fragments are read word by word; their tiles are padded at some widths, spa_gemm.hip.)
// (With it and with fragments read further ahead: a MALA scale of 16384 particles, n = 5000, BF16,
// p = 200 1660 -> 1615 us, p = 250 2142 -> 1848; log-likelihoods of 16384 particles, n = 10000,
// p = 500, 361 -> 315 us; four FP8 terms, n = 5000, p = 200, 86 -> 79 us.)
template <int C>
__device__ __forceinline__ constexpr int row_swizzle(int r) {
  if (C % 16 == 0) return r & 15;
  if (C % 8 == 0) return (r >> 1) & 7;
  if (C % 4 == 0) return -(r >> 2) & 3;          // 0, 3, 2, 1
  return C % 2 == 0 ? (r >> 3) & 1 : 0;
}

}  // namespace spa
