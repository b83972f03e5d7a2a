// Sums over the 64 lanes of a wavefront.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbm {

// v from the lane N positions on in the row of 16 lanes (rotation).
template <int N>
__device__ __forceinline__ double row_rotate(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x120 + N, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x120 + N, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// v plus v of the lane 32 (or 16) away.
template <bool HALF>
__device__ __forceinline__ double swap_add(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t l = (uint32_t)u, h = (uint32_t)(u >> 32);
  const auto a = HALF ? __builtin_amdgcn_permlane32_swap(l, l, false, false)
                      : __builtin_amdgcn_permlane16_swap(l, l, false, false);
  const auto b = HALF ? __builtin_amdgcn_permlane32_swap(h, h, false, false)
                      : __builtin_amdgcn_permlane16_swap(h, h, false, false);
  return __longlong_as_double((long long)(((uint64_t)b[0] << 32) | a[0])) +
         __longlong_as_double((long long)(((uint64_t)b[1] << 32) | a[1]));
}

// Sum over the wavefront by the butterfly of distances 32, 16, 8, 4, 2, 1, in the vector registers
// (through LDS permutes the six sums of a workgroup took 1.7 us). Once the values repeat every 2d
// lanes, a rotation by d reads the lane at distance d.
__device__ __forceinline__ double wave_sum(double v) {
  v = swap_add<true>(v);
  v = swap_add<false>(v);
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  v += row_rotate<1>(v);
  return v;
}

}  // namespace lbm
