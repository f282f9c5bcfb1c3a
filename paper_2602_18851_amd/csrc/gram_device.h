// Device helpers shared by the Gram-form kernels (gram.hip, gram_heads.hip):
// the block layout of a Gram matrix and the d_h-space matrix-vector product.
#pragma once

#include "sweep_device.h"

namespace sn {

// Upper-triangle block (bi, bj >= bi) of an RB x RB block matrix.
template <int RB>
__host__ __device__ constexpr int tri_index(int bi, int bj) {
  return bi * RB - bi * (bi - 1) / 2 + (bj - bi);
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}

// Sum over the 16 lanes of a DPP row; every lane of the row gets the same bits.
__device__ __forceinline__ float row16_sum(float x) {
  x = dpp_add<0xB1>(x);   // quad_perm [1, 0, 3, 2]
  x = dpp_add<0x4E>(x);   // quad_perm [2, 3, 0, 1]
  x = dpp_add<0x141>(x);  // row_half_mirror: quad 0 <-> 1, 2 <-> 3
  x = dpp_add<0x140>(x);  // row_mirror: half 0 <-> half 1
  return x;
}

// Sum of the values of lanes 0, 16, 32, 48 (the C == 0 lanes), in that order.
__device__ __forceinline__ float c0_lanes_sum(float x) {
  const int b = __builtin_bit_cast(int, x);
  return (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)) +
          __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16))) +
         (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32)) +
          __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48)));
}

}  // namespace sn
