// Shared by the backward kernels (paper Alg. 2 loop body, bf16).
#pragma once
#include "burst_common.h"

namespace burst {

// Store of two neighbouring keys' values of one column per lane (lane = column lr, odd and even columns on
// neighbouring lanes) as bf16: even lanes store the first key's pair of columns, odd lanes the
// second key's, four bytes each.
__device__ __forceinline__ void store_pair_bf16(bf16* first, bf16* second, int lr, float a, float b, bool has_second) {
  const bool odd = (lr & 1) != 0;
  const float give = odd ? a : b;
  const float got = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, give), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  bf16x2 v;
  v[0] = (bf16)(odd ? got : a);
  v[1] = (bf16)(odd ? b : got);
  bf16* const p = odd ? second + (lr - 1) : first + lr;
  if (!odd || has_second) *reinterpret_cast<bf16x2*>(p) = v;
}

__device__ __forceinline__ bf16x8 cat4(bf16x4 a, bf16x4 b) {
  bf16x8 v;
  v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3];
  v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
  return v;
}

}  // namespace burst
