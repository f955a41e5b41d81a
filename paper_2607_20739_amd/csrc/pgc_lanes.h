// Reductions over aligned groups of lanes of a gfx950 wave64, within 16-lane rows
// built from DPP lane moves, which go register to register (no LDS permute round
// trip).  Every reduction has a fixed order, so results are bitwise reproducible.
#pragma once
#include <hip/hip_runtime.h>

namespace pgc {

// v from the lane that DPP control `ctrl` selects (all rows and banks on).
template <int ctrl>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, true));
}

// A value that is the same in every lane, in scalar registers (a division leaves its
// result in vector ones).
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<int>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32));
  return static_cast<int64_t>(static_cast<uint64_t>(hi) << 32 | lo);
}

// DPP controls of the 16-lane row reductions: swap neighbours, swap pairs,
// mirror each half row, mirror the row.  After the two quad steps each lane
// holds its quad's result; each mirror step combines a lane with one holding
// the other half's result, so every lane of the row ends with the same value.
constexpr int kDppSwap1 = 0xB1, kDppSwap2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_move<kDppSwap1>(v));
  v = fmaxf(v, dpp_move<kDppSwap2>(v));
  v = fmaxf(v, dpp_move<kDppHalfMirror>(v));
  return fmaxf(v, dpp_move<kDppMirror>(v));
}

__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_move<kDppSwap1>(v);
  v += dpp_move<kDppSwap2>(v);
  v += dpp_move<kDppHalfMirror>(v);
  return v + dpp_move<kDppMirror>(v);
}

// Sum over each aligned group of LANES lanes (a power of two up to 64); every
// lane of a group ends with the same total.
template <int LANES>
__device__ __forceinline__ float lane_group_sum(float v) {
  if constexpr (LANES >= 2) v += dpp_move<kDppSwap1>(v);
  if constexpr (LANES >= 4) v += dpp_move<kDppSwap2>(v);
  if constexpr (LANES >= 8) v += dpp_move<kDppHalfMirror>(v);
  if constexpr (LANES >= 16) v += dpp_move<kDppMirror>(v);
  if constexpr (LANES >= 32) v += __shfl_xor(v, 16, 64);
  if constexpr (LANES >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}

}  // namespace pgc
