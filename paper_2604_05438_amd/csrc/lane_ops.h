// Reductions and prefix sums over the lanes of a wavefront by data-parallel-primitive moves (inside rows of 16 lanes) and lane swaps
// (across rows).  __shfl_xor and its kin go through the LDS pipe, which all wavefronts of a CU share: the 16 of a
// select workgroup were bound by it (their value sums alone 1.3 us longer; the whole kernel 17 against 14.5 us for the 1B layer at 4K).
// Every lane of the wavefront must be active.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace tkphi {

#ifdef __HIPCC__
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_move(T x) {
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
template <typename T, typename Op>
__device__ __forceinline__ T across_16(T x, Op op) {       // with the lane 16 further
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  return op(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
}
template <typename T, typename Op>
__device__ __forceinline__ T across_32(T x, Op op) {       // with the lane 32 further
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  return op(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
}
// over the n (4, 8, 16, 32 or 64, uniform) consecutive lanes that hold a lane's group, in every lane: the butterfly of xor by 1, 2, 4, ..
// (lanes that mirror each other in a half row / a row hold equal partial results after the steps before)
template <typename T, typename Op>
__device__ __forceinline__ T lanes_reduce(T x, int n, Op op) {
  x = op(x, dpp_move<0xB1>(x));                            // quad_perm [1, 0, 3, 2]
  x = op(x, dpp_move<0x4E>(x));                            // quad_perm [2, 3, 0, 1]
  if (n >= 8) x = op(x, dpp_move<0x141>(x));               // row_half_mirror
  if (n >= 16) x = op(x, dpp_move<0x140>(x));              // row_mirror
  if (n >= 32) x = across_16(x, op);
  if (n >= 64) x = across_32(x, op);
  return x;
}
struct AddOp { template <typename T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; } };
struct MaxOp {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
  __device__ __forceinline__ int operator()(int a, int b) const { return a > b ? a : b; }
  __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; }
};
template <typename T> __device__ __forceinline__ T lanes_sum(T x, int n) { return lanes_reduce(x, n, AddOp()); }
template <typename T> __device__ __forceinline__ T wave_sum(T x) { return lanes_reduce(x, 64, AddOp()); }
template <typename T> __device__ __forceinline__ T wave_max(T x) { return lanes_reduce(x, 64, MaxOp()); }
// over the lanes that are equal modulo n (8, 16, 32 or 64, uniform), in every lane
template <typename T>
__device__ __forceinline__ T strided_sum(T x, int n) {
  if (n <= 8) x += dpp_move<0x128>(x);                     // row_ror:8
  if (n <= 16) x = across_16(x, AddOp());
  if (n <= 32) x = across_32(x, AddOp());
  return x;
}
// inclusive prefix sum
__device__ __forceinline__ int wave_scan_incl(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
  return x;
}
#endif

}  // namespace tkphi
