// Wave-level reductions on DPP lane moves (no LDS round trips): quad
// permutations, row mirrors and the gfx9 row broadcasts combine the 64 lanes
// in six steps; lane 63 then holds the result, which readlane makes uniform.
#pragma once
#include "internal.h"

namespace hodlr {

namespace dpp {
constexpr int kQuad1032 = 0xB1;      // quad_perm [1, 0, 3, 2]
constexpr int kQuad2301 = 0x4E;      // quad_perm [2, 3, 0, 1]
constexpr int kRowHalfMirror = 0x141;
constexpr int kRowMirror = 0x140;
constexpr int kRowBcast15 = 0x142;   // lane 15 of each row into the next row (rows 1, 3 enabled)
constexpr int kRowBcast31 = 0x143;   // lane 31 into rows 2 and 3

template <int CTRL, int ROWS>
__device__ __forceinline__ int mov(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int uniform63(int v) { return __builtin_amdgcn_readlane(v, 63); }
}  // namespace dpp

// Minimum and maximum over the wave, uniform results; every lane must take part.
__device__ __forceinline__ int wave_min(int v) {
  v = min(v, dpp::mov<dpp::kQuad1032, 0xf>(v));
  v = min(v, dpp::mov<dpp::kQuad2301, 0xf>(v));
  v = min(v, dpp::mov<dpp::kRowHalfMirror, 0xf>(v));
  v = min(v, dpp::mov<dpp::kRowMirror, 0xf>(v));
  v = min(v, dpp::mov<dpp::kRowBcast15, 0xa>(v));
  v = min(v, dpp::mov<dpp::kRowBcast31, 0xc>(v));
  return dpp::uniform63(v);
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max(v, (uint32_t)dpp::mov<dpp::kQuad1032, 0xf>((int)v));
  v = max(v, (uint32_t)dpp::mov<dpp::kQuad2301, 0xf>((int)v));
  v = max(v, (uint32_t)dpp::mov<dpp::kRowHalfMirror, 0xf>((int)v));
  v = max(v, (uint32_t)dpp::mov<dpp::kRowMirror, 0xf>((int)v));
  v = max(v, (uint32_t)dpp::mov<dpp::kRowBcast15, 0xa>((int)v));
  v = max(v, (uint32_t)dpp::mov<dpp::kRowBcast31, 0xc>((int)v));
  return (uint32_t)dpp::uniform63((int)v);
}

// Order of moduli as unsigned integers: the bits of |x| (NaN as infinity), in
// the high and, for FP64, the low word; open rows are one higher than zero, so
// closed rows (0) never win.
__device__ __forceinline__ void modulus_words(double x, bool open, uint32_t& hi, uint32_t& lo) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x) & 0x7fffffffffffffffull;
  const bool nan = b > 0x7ff0000000000000ull;
  hi = open ? (nan ? 0x7ff00000u : (uint32_t)(b >> 32)) + 1u : 0u;
  lo = nan ? 0u : (uint32_t)b;
}
__device__ __forceinline__ void modulus_words(float x, bool open, uint32_t& hi, uint32_t& lo) {
  const uint32_t b = __builtin_bit_cast(uint32_t, x) & 0x7fffffffu;
  hi = open ? min(b, 0x7f800000u) + 1u : 0u;
  lo = 0u;
}

}  // namespace hodlr
