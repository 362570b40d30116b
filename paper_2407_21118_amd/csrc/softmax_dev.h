// Wavefront primitives of the softmax over tokens (value kernel pv.hip, attention kernel attend16.hip): a lane holds one
// token of a set of 32, the halves of the wavefront hold different heads.
#pragma once

#include "palu_dev.h"

namespace palu {

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// lane ^ 16 inside each half of the wavefront
__device__ __forceinline__ float swap16(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
}
// Maximum over the 32 lanes of a wavefront half; the result is in all 32 lanes.  The numbers (no NaN among
// them) are compared as integers of the same order (negative floats have their low 31 bits inverted): an
// integer maximum with its lane move is one instruction, where fmaxf() of a moved float takes four (the move
// and its initial value, and one per operand to quiet signalling NaNs).
__device__ __forceinline__ int float_order(int b) { return b ^ ((b >> 31) & 0x7fffffff); }     // its own inverse
template <int CTRL>
__device__ __forceinline__ int dpp_peek(int v) {          // every lane has a source lane under these controls: no old value to keep
  return __builtin_amdgcn_update_dpp((int)0x80000000, v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ float half_wave_max(float f) {
  int v = float_order(__builtin_bit_cast(int, f));
  v = max(v, dpp_peek<0xB1>(v));      // quad_perm [1,0,3,2]
  v = max(v, dpp_peek<0x4E>(v));      // quad_perm [2,3,0,1]
  v = max(v, dpp_peek<0x141>(v));     // row_half_mirror
  v = max(v, dpp_peek<0x140>(v));     // row_mirror
  v = max(v, __builtin_amdgcn_ds_swizzle(v, 0x401F));
  return __builtin_bit_cast(float, float_order(v));
}
__device__ __forceinline__ float half_wave_sum(float v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  v += dpp_move<0x140>(v);
  return v + swap16(v);
}

// LDS written by some lanes of this wavefront is read by others: the hardware keeps
// a wavefront's LDS operations in order, this keeps the compiler from moving them
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace palu
