// Moves between the lanes of a wave that need no LDS round trip: DPP inside rows of sixteen lanes,
// lane reads across the wave.
#pragma once

#include <hip/hip_runtime.h>

namespace sdl {
namespace {

// DPP controls used below: quad_perm [1,0,3,2] (lane ^ 1) and [2,3,0,1] (lane ^ 2), row_half_mirror
// and row_mirror (after the two quad steps of a reduction: the other quad, the other half row)
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int CTRL, int ROWS = 0xF>
__device__ inline int dpp32(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS = 0xF, typename U>
__device__ inline U dpp(U old, U v) {
  if constexpr (sizeof(U) == 4) {
    return __builtin_bit_cast(U, dpp32<CTRL, ROWS>(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v)));
  } else {
    const long long o = __builtin_bit_cast(long long, old), b = __builtin_bit_cast(long long, v);
    const int lo = dpp32<CTRL, ROWS>((int)o, (int)b);
    const int hi = dpp32<CTRL, ROWS>((int)(o >> 32), (int)(b >> 32));
    return __builtin_bit_cast(U, ((long long)hi << 32) | (unsigned int)lo);
  }
}
template <typename U>
__device__ inline U lane_read(U v, int l) {  // l uniform
  if constexpr (sizeof(U) == 4) {
    return __builtin_bit_cast(U, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
  } else {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __builtin_bit_cast(U, ((long long)hi << 32) | (unsigned int)lo);
  }
}

// lane L's value of v, within each row of sixteen lanes
template <int L, typename U>
__device__ inline U bcast16(U v) {
  if constexpr (sizeof(U) == 4) {
    return __builtin_bit_cast(U, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x150 + L, 0xF, 0xF, true));
  } else {  // row_newbcast:L
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x150 + L, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x150 + L, 0xF, 0xF, true);
    return __builtin_bit_cast(U, ((long long)hi << 32) | (unsigned int)lo);
  }
}
}  // namespace
}  // namespace sdl
