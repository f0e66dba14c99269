// Exchanges between the lanes of a wavefront (shifts, selects, sums), and the
// order in which the work-groups of the kernels that walk strips take them.
#pragma once

#include "gg_device.h"

namespace gg {

// The value of the lane to the left, to the right; `edge` where there is none.
__device__ __forceinline__ uint32_t lane_shr(uint32_t v, uint32_t edge) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t lane_shl(uint32_t v, uint32_t edge) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x130, 0xf, 0xf, false);
}

__device__ __forceinline__ float lane_shr(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_shl(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_shr(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, 0x138, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)lo | (uint64_t)hi << 32);
}
__device__ __forceinline__ double lane_shl(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, 0x130, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)lo | (uint64_t)hi << 32);
}

// bit `pos` of word ? a : b, without a compare.
__device__ __forceinline__ float bit_select(uint32_t word, int pos, float a, float b) {
  const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)word, pos, 1);
  return __builtin_bit_cast(float, (m & __builtin_bit_cast(uint32_t, a)) |
                                       (~m & __builtin_bit_cast(uint32_t, b)));
}
__device__ __forceinline__ double bit_select(uint32_t word, int pos, double a, double b) {
  const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)word, pos, 1);
  const uint64_t u = __builtin_bit_cast(uint64_t, a), v = __builtin_bit_cast(uint64_t, b);
  const uint32_t lo = (m & (uint32_t)u) | (~m & (uint32_t)v);
  const uint32_t hi = (m & (uint32_t)(u >> 32)) | (~m & (uint32_t)(v >> 32));
  return __builtin_bit_cast(double, (uint64_t)lo | (uint64_t)hi << 32);
}

// Lane s's value (s uniform).
__device__ __forceinline__ float lane_value(float v, int s) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), s));
}
__device__ __forceinline__ double lane_value(double v, int s) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(
      double, (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)b, s) |
                  (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), s) << 32);
}

// Sum over the 64 lanes of a wavefront; every lane must be active. Rotations
// within the rows of 16 lanes, then the four rows' sums: no LDS, which would be
// six dependent exchanges (2048 x 1024 FP32 with pressure segments, 64 steps:
// 747 us with these sums and the lane shifts through LDS, 722 without).
template <int N> __device__ __forceinline__ double row_rotate(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, 0x120 + N, 0xF, 0xF, true);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + N, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)lo | (uint64_t)hi << 32);
}
__device__ __forceinline__ double wave_sum(double v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  v += row_rotate<1>(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// The strip of work-group b: the segment strips (the longest to run) first,
// dealt to the XCDs one by one; then each XCD a contiguous run of the others.
// False: none.
__device__ __forceinline__ bool strip_of(int b, const Tile *seg_tiles, int n_seg,
                                         const Tile *tiles, int n_tiles, int per_xcd,
                                         const Tile *&list, int &tile) {
  const int seg_blocks = (n_seg + 7) & ~7;
  list = seg_tiles;
  tile = b;
  if (b < seg_blocks) return tile < n_seg;
  list = tiles;
  tile = ((b - seg_blocks) & 7) * per_xcd + ((b - seg_blocks) >> 3);
  return tile < n_tiles;
}

}  // namespace gg
