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
// Rotations of a row by 4 and 8 lanes.
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;

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

// The same move of a double, half by half.
template <int ctrl>
__device__ __forceinline__ double dpp_move(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), ctrl, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), ctrl, 0xF, 0xF, true);
  return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}

// Of two registers' values, the lower lanes' sum with their partners DISTANCE (16 or 32)
// lanes away for `a`, the upper lanes' for `b`: one lane swap and one addition.  With
// DISTANCE = 16 lower and upper are the rows of 16 lanes in turn.
template <int DISTANCE>
__device__ __forceinline__ double swap_sum(double a, double b) {
  static_assert(DISTANCE == 16 || DISTANCE == 32, "swaps");
  const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
  auto swap = [](uint32_t x, uint32_t y) {
    return DISTANCE == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                          : __builtin_amdgcn_permlane16_swap(x, y, false, false);
  };
  const auto lo = swap(static_cast<uint32_t>(ua), static_cast<uint32_t>(ub));
  const auto hi = swap(static_cast<uint32_t>(ua >> 32), static_cast<uint32_t>(ub >> 32));
  return __builtin_bit_cast(double, static_cast<uint64_t>(hi[0]) << 32 | lo[0]) +
         __builtin_bit_cast(double, static_cast<uint64_t>(hi[1]) << 32 | lo[1]);
}

// Sums of four values each over the lanes of the wave that are a multiple of LANES (a
// power of two up to 16) apart: lanes 16 i .. 16 i + 15 end with value i's, by class.
template <int LANES, class V4>
__device__ __forceinline__ double lane_stride_sums(V4 v) {
  static_assert(LANES <= 16, "a row of lanes per value");
  double s = swap_sum<16>(swap_sum<32>(v[0], v[2]), swap_sum<32>(v[1], v[3]));
  if constexpr (LANES <= 8) s += dpp_move<kDppRor8>(s);
  if constexpr (LANES <= 4) s += dpp_move<kDppRor4>(s);   // after the step of 8 as good as a swap
  if constexpr (LANES <= 2) s += dpp_move<kDppSwap2>(s);
  if constexpr (LANES <= 1) s += dpp_move<kDppSwap1>(s);
  return s;
}

}  // namespace pgc
