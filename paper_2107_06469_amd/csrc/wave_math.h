// Sums and maxima over the 64 lanes of a wave, every lane receiving the result: a butterfly in the order 32, 16, 8, 4, 2, 1.
// The exchanges are register moves (permlane swaps between the halves and quarters of a wave, DPP rotations and quad
// permutations inside a row of 16) instead of ds_bpermute round trips through the LDS unit: a row of 16 is rotated by 8 and 4,
// which reads the same values as lane^8 and lane^4 once the steps before have made them equal.
#pragma once
#include <hip/hip_runtime.h>

namespace hydra {

template <int CTRL>
__device__ __forceinline__ float wave_dpp(float v) {
  const int i = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
}
// {v of the lower, v of the upper} half (quarter pair) in every lane
__device__ __forceinline__ float2 wave_swap32(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return make_float2(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float2 wave_swap16(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return make_float2(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float wave_sum(float v) {
  float2 p = wave_swap32(v);
  v = p.x + p.y;
  p = wave_swap16(v);
  v = p.x + p.y;
  v += wave_dpp<0x128>(v);  // row_ror:8
  v += wave_dpp<0x124>(v);  // row_ror:4
  v += wave_dpp<0x4e>(v);   // quad_perm [2,3,0,1]
  return v + wave_dpp<0xb1>(v);  // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float wave_max(float v) {
  float2 p = wave_swap32(v);
  v = fmaxf(p.x, p.y);
  p = wave_swap16(v);
  v = fmaxf(p.x, p.y);
  v = fmaxf(v, wave_dpp<0x128>(v));
  v = fmaxf(v, wave_dpp<0x124>(v));
  v = fmaxf(v, wave_dpp<0x4e>(v));
  return fmaxf(v, wave_dpp<0xb1>(v));
}

}  // namespace hydra
