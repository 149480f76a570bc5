// Shared by the backward kernels (paper Alg. 2 loop body, bf16).
#pragma once
#include "burst_common.h"

namespace burst {

__device__ __forceinline__ bf16x8 cat4(bf16x4 a, bf16x4 b) {
  bf16x8 v;
  v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3];
  v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
  return v;
}

}  // namespace burst
