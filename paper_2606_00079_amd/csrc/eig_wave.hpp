// fp64 cross-lane helpers of the eigensolver kernels.
#pragma once

#include "common.hpp"

namespace bitsmoe {

// v of the lane that the DPP control selects (every lane takes part).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = static_cast<uint32_t>(
      __builtin_amdgcn_mov_dpp(static_cast<int>(u & 0xffffffffu), CTRL, 0xF, 0xF, false));
  const uint32_t hi = static_cast<uint32_t>(
      __builtin_amdgcn_mov_dpp(static_cast<int>(u >> 32), CTRL, 0xF, 0xF, false));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}
constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]: lane ^ 1
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]: lane ^ 2
constexpr int kDppXor3 = 0x1B;         // quad_perm [3,2,1,0]: lane ^ 3
constexpr int kDppHalfMirror = 0x141;  // lane ^ 7
constexpr int kDppMirror = 0x140;      // lane ^ 15
constexpr int kDppRor8 = 0x128;        // rotate 16 lanes by 8: lane ^ 8

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = static_cast<uint32_t>(
      __builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffu), lane));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// Sum over the wave in a fixed order, the same bits in every lane: four DPP
// steps inside the rows of 16 lanes, then the four row sums by readlane (a
// ds_bpermute butterfly takes about three times as long).
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v += dpp_f64<kDppXor1>(v);
  v += dpp_f64<kDppXor2>(v);
  v += dpp_f64<kDppHalfMirror>(v);
  v += dpp_f64<kDppMirror>(v);
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// Halves a pair of values over the lanes whose index differs in bit 5 (or
// 4): lanes with that bit clear get a summed over both lanes, the others b.
__device__ __forceinline__ double fold_bit5(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto l = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(x), static_cast<uint32_t>(y), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(x >> 32), static_cast<uint32_t>(y >> 32), false, false);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(h[0]) << 32) | l[0]) +
         __builtin_bit_cast(double, (static_cast<uint64_t>(h[1]) << 32) | l[1]);
}
__device__ __forceinline__ double fold_bit4(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto l = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(x), static_cast<uint32_t>(y), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(x >> 32), static_cast<uint32_t>(y >> 32), false, false);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(h[0]) << 32) | l[0]) +
         __builtin_bit_cast(double, (static_cast<uint64_t>(h[1]) << 32) | l[1]);
}
// The same by a DPP control whose partner lane differs in `bit` of the lane
// index (and possibly in lower bits, which carry no value index yet).
template <int CTRL>
__device__ __forceinline__ double fold_dpp(double a, double b, bool bit) {
  const double keep = bit ? b : a, send = bit ? a : b;
  return keep + dpp_f64<CTRL>(send);
}

// Sums of N = 8, 16 or 32 per-lane values over the wave (fixed order): lane
// l returns the sum of value l / (64 / N).
template <int N>
__device__ __forceinline__ double wave_fold(double (&v)[N], int lane) {
  static_assert(N == 8 || N == 16 || N == 32, "values per lane");
#pragma unroll
  for (int j = 0; j < N / 2; ++j) v[j] = fold_bit5(v[j], v[j + N / 2]);
#pragma unroll
  for (int j = 0; j < N / 4; ++j) v[j] = fold_bit4(v[j], v[j + N / 4]);
#pragma unroll
  for (int j = 0; j < N / 8; ++j) v[j] = fold_dpp<kDppRor8>(v[j], v[j + N / 8], (lane & 8) != 0);
  if constexpr (N >= 16) {
#pragma unroll
    for (int j = 0; j < N / 16; ++j)
      v[j] = fold_dpp<kDppHalfMirror>(v[j], v[j + N / 16], (lane & 4) != 0);
  } else {
    v[0] += dpp_f64<kDppHalfMirror>(v[0]);
  }
  if constexpr (N >= 32)
    v[0] = fold_dpp<kDppXor3>(v[0], v[1], (lane & 2) != 0);
  else
    v[0] += dpp_f64<kDppXor3>(v[0]);
  v[0] += dpp_f64<kDppXor1>(v[0]);
  return v[0];
}

// Barrier of the workgroup that publishes LDS writes only: __syncthreads()
// would also wait for global loads and stores in flight (about a microsecond).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) alone
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace bitsmoe
