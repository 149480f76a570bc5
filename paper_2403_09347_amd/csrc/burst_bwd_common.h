// Shared by the backward kernels (paper Alg. 2 loop body, bf16).
#pragma once
#include "burst_rows.h"

namespace burst {

// Stores a wavefront's 32 keys of dK (times `scale`) and dV.  Layout of the accumulators: lane = column
// db*32 + lr, register r = key key0 + 8*(r/4) + 4h + r%4.  `dK`, `dV`: key 0 of the head, rows of d values,
// fp32 or, `half`, bf16.  Keys past Nc and (PAD) columns past d lie outside the buffers' range (at most
// 4 Mi rows x 512 bytes), so there is not one branch or 64-bit address in here.
// Bound by the stores, which must follow each other without a wait: with the loads of `acc` on a way of
// their own.  (As one loop, old = acc ? load : 0, the compiler waited for every store before the next: a
// workgroup of 128 keys then took 13.7 us on its 128 KB.)
// bf16: a lane holds one column of two neighbouring keys; neighbouring lanes exchange, so that even lanes
// store the first key's pair of columns and odd lanes the second key's, four bytes each.
template <int DB, bool PAD>
__device__ __forceinline__ void store_dkv(const f32x16 (&dk)[DB], const f32x16 (&dv)[DB], void* dK, void* dV, int Nc, int d,
                                          int key0, int lr, int h, float scale, int half, int acc) {
  const unsigned pitch = (unsigned)d * (half ? 2u : 4u);
  const unsigned bytes = (unsigned)Nc * pitch;
  const __amdgpu_buffer_rsrc_t krs = make_rsrc(dK, bytes), vrs = make_rsrc(dV, bytes);
  const unsigned row0 = (unsigned)(key0 + 4 * h) * pitch;
  auto key_of = [](int r) { return 8 * (r >> 2) + (r & 3); };
  if (half) {
    const bool odd = (lr & 1) != 0;
    const unsigned base = row0 + (odd ? pitch + (lr - 1) * 2u : lr * 2u);
    auto pair = [&](__amdgpu_buffer_rsrc_t rs, unsigned off, float x, float y) __attribute__((always_inline)) {
      const float give = odd ? x : y;
      const float got = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, give), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
      bf16x2 v;
      v[0] = (bf16)(odd ? got : x);
      v[1] = (bf16)(odd ? y : got);
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, off, 0, 0);
    };
#pragma unroll
    for (int db = 0; db < DB; db++) {
      const unsigned col = PAD && db * 32 + lr >= d ? 0x80000000u : base + db * 64u;   // (d is even: both lanes of a pair agree)
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        pair(krs, col + key_of(r) * pitch, scale * dk[db][r], scale * dk[db][r + 1]);
        pair(vrs, col + key_of(r) * pitch, dv[db][r], dv[db][r + 1]);
      }
    }
    return;
  }
  const unsigned base = row0 + lr * 4u;
  unsigned col[DB];
#pragma unroll
  for (int db = 0; db < DB; db++) col[db] = PAD && db * 32 + lr >= d ? 0x80000000u : base + db * 128u;
  auto put = [](__amdgpu_buffer_rsrc_t rs, unsigned off, float x) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), rs, off, 0, 0);
  };
  if (acc) {
    auto get = [](__amdgpu_buffer_rsrc_t rs, unsigned off) __attribute__((always_inline)) {
      return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
    };
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      float k_old[4][DB], v_old[4][DB];
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int db = 0; db < DB; db++) {
          k_old[j][db] = get(krs, col[db] + (8 * q4 + j) * pitch);
          v_old[j][db] = get(vrs, col[db] + (8 * q4 + j) * pitch);
        }
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int db = 0; db < DB; db++) {
          put(krs, col[db] + (8 * q4 + j) * pitch, k_old[j][db] + scale * dk[db][4 * q4 + j]);
          put(vrs, col[db] + (8 * q4 + j) * pitch, v_old[j][db] + dv[db][4 * q4 + j]);
        }
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < 16; r++)
#pragma unroll
    for (int db = 0; db < DB; db++) {
      put(krs, col[db] + key_of(r) * pitch, scale * dk[db][r]);
      put(vrs, col[db] + key_of(r) * pitch, dv[db][r]);
    }
}

// Adds the partial dK, dV of a split launch (see RowParts) in the order of the parts: one wavefront per key.  Bound by
// its reads (32 heads x 777 keys, d = 96, at most 3 parts: 57 MB in 10.8 us; four keys per wavefront 11.1).  PAD: keys whose sum is infinite or NaN are computed by themselves
// (see burst_rows.h).
template <int D, int BC, int BR, bool PAD, typename A>
__global__ void __launch_bounds__(256)
merge_dkv_kernel(A a) {
  const int lane = threadIdx.x & 63;
  const int row = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= a.parts.rows) return;
  int c = 0;
  while (c + 1 < a.n && row >= a.ch[c + 1].first_row) c++;
  const Chunk& C = a.ch[c];
  const int kvhead = (row - C.first_row) / C.span_keys, key = C.span_lo + row - C.first_row - kvhead * C.span_keys;
  const RowRange range = row_range(a.Nq, a.causal, a.window, a.q_off, C.k_off, C.Nc, key / BC * BC, BC, BR);
  const int parts = a.parts.of((range.hi - range.lo) * a.group);
  if (parts == 1) return;                          // written by its workgroup
  int d = D;
  if constexpr (PAD) d = a.d;
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  f32x2 k = {0.f, 0.f}, v = {0.f, 0.f};
  const int col = 2 * lane < d ? 2 * lane : 0;
  const size_t plane = (size_t)a.parts.rows * d;
  const float* from = a.parts.part + (size_t)row * d + col;
#pragma unroll 4
  for (int i = 0; i < parts; i++, from += 2 * plane) {
    const f32x2 x = *reinterpret_cast<const f32x2*>(from), y = *reinterpret_cast<const f32x2*>(from + plane);
    k[0] += x[0]; k[1] += x[1];
    v[0] += y[0]; v[1] += y[1];
  }
  const size_t at = ((size_t)kvhead * C.Nc + key) * d;
  if constexpr (PAD) {
    const unsigned most = larger_of(larger_of(larger_of(larger_of(0, k[0]), k[1]), v[0]), v[1]);
    if (__builtin_amdgcn_ballot_w64(most >= kInfBits) != 0) {
      const int keys[kRows] = {key, key, key};
      float gk[kRows][2], gv[kRows][2];
      keys_dkv<bf16, true>(gk, gv, a, C, kvhead, keys, lane);
      row_gradient<bf16>(C.dK, at, gk[0], a.scale, a.half, a.acc_dkv, lane, d);
      row_gradient<bf16>(C.dV, at, gv[0], 1.f, a.half, a.acc_dkv, lane, d);
      return;
    }
  }
  if (2 * lane >= d) return;
  if (a.half) {
    bf16x2 x, y;
    x[0] = (bf16)k[0]; x[1] = (bf16)k[1];
    y[0] = (bf16)v[0]; y[1] = (bf16)v[1];
    *reinterpret_cast<bf16x2*>((bf16*)C.dK + at + col) = x;
    *reinterpret_cast<bf16x2*>((bf16*)C.dV + at + col) = y;
  } else {
    f32x2* const dk = reinterpret_cast<f32x2*>((float*)C.dK + at + col);
    f32x2* const dv = reinterpret_cast<f32x2*>((float*)C.dV + at + col);
    if (a.acc_dkv) {
      const f32x2 x = *dk, y = *dv;
      k[0] += x[0]; k[1] += x[1];
      v[0] += y[0]; v[1] += y[1];
    }
    *dk = k;
    *dv = v;
  }
}
template <int D, int BC, int BR, bool PAD, typename A>
static int launch_merge_dkv(const A& a, hipStream_t stream) {
  BURST_LAUNCH((merge_dkv_kernel<D, BC, BR, PAD, A>), dim3((unsigned)((a.parts.rows + 3) / 4)), dim3(256), 0, stream, a);
  return launch_status();
}
// (after the chunks; all chunks of the call without flags where its walks are cut)
template <typename A>
static void set_row_parts(A& a, const BwdIo& io) {
  a.parts = io.parts != nullptr ? io.parts->parts : RowParts{nullptr, 1, 1, 1, 0};
  for (int i = 0; i < a.n && a.parts.splits > 1; i++) {
    const RowSpan& s = io.parts->span[i];
    a.ch[i].first_row = s.first; a.ch[i].span_lo = s.lo; a.ch[i].span_keys = s.keys;
  }
}

__device__ __forceinline__ bf16x8 cat4(bf16x4 a, bf16x4 b) {
  bf16x8 v;
  v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3];
  v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
  return v;
}

}  // namespace burst
