// Reductions over the 64 lanes of a wave in its registers (data-parallel primitives and lane swaps,
// a few cycles a step; a shuffle goes through LDS, about a hundred).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nc {

// Lane controls: row_shl / row_shr n (from the lane n up / down in the same sixteen), row_ror n
// (rotation of the sixteen), the last lane of the row(s) before, wave_shr 1.
constexpr int kShl = 0x100, kShr = 0x110, kRor = 0x120, kWaveShr1 = 0x138, kBcast15 = 0x142,
              kBcast31 = 0x143;

// The value of the controlled lane, or `none` where there is none (rows outside kRows keep none).
template <int kCtrl, int kRows = 0xF>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v, uint32_t none = 0) {
  return uint32_t(__builtin_amdgcn_update_dpp(int(none), int(v), kCtrl, kRows, 0xF, false));
}
template <int kCtrl, int kRows = 0xF>
__device__ __forceinline__ float dpp_f(float v, float none = 0.f) {
  return __uint_as_float(dpp_u32<kCtrl, kRows>(__float_as_uint(v), __float_as_uint(none)));
}

__device__ __forceinline__ float read_lane(float v, int lane) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane));
}

// Inclusive prefix sums over the lanes.
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
  v += dpp_u32<kShr + 1>(v);
  v += dpp_u32<kShr + 2>(v);
  v += dpp_u32<kShr + 4>(v);
  v += dpp_u32<kShr + 8>(v);
  v += dpp_u32<kBcast15, 0xA>(v);
  v += dpp_u32<kBcast31, 0xC>(v);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  return uint32_t(__builtin_amdgcn_readlane(int(wave_scan_u32(v)), 63));
}
// Sum of 32-bit values (two sums of 16-bit halves, neither of which overflows).
__device__ __forceinline__ uint64_t wave_sum_u64(uint32_t v) {
  return (uint64_t(wave_sum_u32(v >> 16)) << 16) + wave_sum_u32(v & 0xFFFFu);
}

template <int kCtrl, int kRows = 0xF>
__device__ __forceinline__ uint64_t dpp_max_u64(uint64_t v) {
  const uint64_t o = uint64_t(dpp_u32<kCtrl, kRows>(uint32_t(v))) |
                     (uint64_t(dpp_u32<kCtrl, kRows>(uint32_t(v >> 32))) << 32);
  return o > v ? o : v;
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  v = dpp_max_u64<kShr + 1>(v);
  v = dpp_max_u64<kShr + 2>(v);
  v = dpp_max_u64<kShr + 4>(v);
  v = dpp_max_u64<kShr + 8>(v);
  v = dpp_max_u64<kBcast15, 0xA>(v);
  v = dpp_max_u64<kBcast31, 0xC>(v);
  return uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), 63))) |
         (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v >> 32)), 63))) << 32);
}

// Inclusive prefix maxima over the lanes.
__device__ __forceinline__ float wave_scan_max(float v) {
  v = fmaxf(v, dpp_f<kShr + 1>(v, -INFINITY));
  v = fmaxf(v, dpp_f<kShr + 2>(v, -INFINITY));
  v = fmaxf(v, dpp_f<kShr + 4>(v, -INFINITY));
  v = fmaxf(v, dpp_f<kShr + 8>(v, -INFINITY));
  v = fmaxf(v, dpp_f<kBcast15, 0xA>(v, -INFINITY));
  v = fmaxf(v, dpp_f<kBcast31, 0xC>(v, -INFINITY));
  return v;
}

// The values of lanes l and l ^ 32 (l ^ 16) combined, in every lane.
template <class Op>
__device__ __forceinline__ float combine_x32(float v, Op op) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float combine_x16(float v, Op op) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// Partners l ^ 32, l ^ 16, l ^ 8, l ^ 4, l ^ 2, l ^ 1 in that order; every lane gets the result.  op
// is commutative, and after the step of partner l ^ d the values repeat every d lanes of a row, so
// a rotation by d / 2 fetches the next partner's.
template <class Op>
__device__ __forceinline__ float wave_butterfly(float v, Op op) {
  v = combine_x32(v, op);
  v = combine_x16(v, op);
  v = op(v, dpp_f<kRor + 8>(v));
  v = op(v, dpp_f<kRor + 4>(v));
  v = op(v, dpp_f<kRor + 2>(v));
  return op(v, dpp_f<kRor + 1>(v));
}
__device__ __forceinline__ float wave_sum_f(float v) {
  return wave_butterfly(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max_f(float v) {
  return wave_butterfly(v, [](float a, float b) { return fmaxf(a, b); });
}

}  // namespace nc
