// One query row (forward, dQ) or one key (dK, dV) at a time, by one wavefront with scalar FMAs: what the matrix-core
// kernels of burst_generic.hip and of the padded builds of burst_plain_mfma.h fall back to where their accumulators come
// out infinite or NaN.  A matrix product multiplies every pair of its operands, also where one of the two is a
// zero that stands for "nothing": a hidden pair, the rows and columns of padding, the lower terms of a probability
// split into three bf16 numbers.  0 x inf is NaN, so one infinite value could reach rows that do not see it, and inf
// could become NaN in a row that does.  Here hidden pairs are skipped and every product is the one of the formula.
// Finite accumulators need no second look: inf and NaN do not go away in a sum, nor when it is scaled.
// Cost: nothing but the test at the end of a workgroup; with it, the time these calls took before they ran on the matrix
// cores (rows at some 9 G pairs/s: 8 heads of 700 x 700, d = 128, all of them NaN: 0.45 / 0.5 / 1.9 ms for the three
// kernels instead of 48 / 64 / 91 us).
#pragma once
#include "burst_common.h"

namespace burst {

// Largest magnitude so far, as an integer: infinities and NaN are not below kInfBits.  (Integers and an opaque move,
// because the compiler may assume that no float is a NaN.)
constexpr unsigned kInfBits = 0x7f800000u;
__device__ __forceinline__ unsigned larger_of(unsigned so_far, float x) {
  unsigned b = __builtin_bit_cast(unsigned, x);
  asm("" : "+v"(b));
  b &= 0x7fffffffu;
  return b > so_far ? b : so_far;
}

__device__ __forceinline__ float wave_max(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

template <typename A>
__device__ __forceinline__ bool pair_visible(const A& a, const Chunk& C, int head, int row, int key) {
  const long long qp = a.q_off + row, kp = C.k_off + key;
  if (a.causal && kp > qp) return false;
  if (a.window > 0 && kp <= qp - a.window) return false;
  return C.bmask == nullptr ||
         C.bmask[(size_t)head * C.bhstride + (size_t)(row / a.bsize) * C.bpitch + key / a.bsize] != 0;
}
template <typename T>
__device__ __forceinline__ float row_dot(const T* x, const T* y, int d) {
  float s = 0.f;
#pragma unroll 1
  for (int t = 0; t < d; t++) s = __builtin_fmaf((float)x[t], (float)y[t], s);
  return s;
}
// acc += f x row, columns lane and lane + 64
template <typename T>
__device__ __forceinline__ void row_add(float (&acc)[2], float f, const T* row, int lane, int d) {
  if (lane < d) acc[0] = __builtin_fmaf(f, (float)row[lane], acc[0]);
  if (lane + 64 < d) acc[1] = __builtin_fmaf(f, (float)row[lane + 64], acc[1]);
}

struct RowState { float m, l, o[2]; };             // o: columns lane and lane + 64
__device__ __forceinline__ RowState row_state(bool fresh, const float* O_acc, const float* m, const float* l, size_t sr, int d, int lane) {
  RowState st = {BURST_NEG_INF, 0.f, {0.f, 0.f}};
  if (!fresh && m[sr] != BURST_NEG_INF) {          // (a row that has seen nothing may hold anything)
    st.m = m[sr]; st.l = l[sr];
    row_add(st.o, 1.f, O_acc + sr * d, lane, d);
  }
  return st;
}
// The tiles [first, last) of 64 keys of the sequence that `tiles_of` (chunk -> range) makes of the chunks.
template <typename T, typename A, typename F>
__device__ __forceinline__ void row_forward(RowState& st, const A& a, int head, int row, int lane, F tiles_of, int first, int last) {
  const T* const q = (const T*)a.Q + a.lay.q_base(head) + (size_t)row * a.lay.qs_r;
  int at = 0;
#pragma unroll 1
  for (int i = 0; i < a.n; i++) {
    const Chunk& C = a.ch[i];
    const size_t base = C.kv_base(head / a.group, a.lay.kv_heads);
    const T* const K = (const T*)C.K + base;
    const T* const V = (const T*)C.V + base;
    RowState c = {BURST_NEG_INF, 0.f, {0.f, 0.f}};
    int lo, hi;
    tiles_of(C, lo, hi);
#pragma unroll 1
    for (int t = lo; t < hi; t++, at++) {
      if (at < first || at >= last) continue;
      const int key = t * 64 + lane;
      const bool vis = key < C.Nc && pair_visible(a, C, head, row, key);
      const float s = vis ? product(row_dot(q, K + (size_t)key * C.ks_r, a.d), a.scale) : BURST_NEG_INF;
      const float m_new = fmaxf(c.m, wave_max(s)), ref = m_new == BURST_NEG_INF ? 0.f : m_new;
      const float p = vis ? fast_exp2((s - ref) * kLog2e) : 0.f, alpha = fast_exp2((c.m - ref) * kLog2e);
      c.l = c.l * alpha + wave_sum(p);
      c.o[0] *= alpha; c.o[1] *= alpha;
      c.m = m_new;
      for (unsigned long long left = __builtin_amdgcn_ballot_w64(vis); left != 0; left &= left - 1) {
        const int k = __builtin_ctzll(left);
        row_add(c.o, __shfl(p, k), V + (size_t)(t * 64 + k) * C.ks_r, lane, a.d);
      }
    }
    if (c.m == BURST_NEG_INF) continue;            // no key of the chunk: the state stays
    const float m_new = fmaxf(st.m, c.m);          // Alg. 1 merge step
    const float fa = fast_exp2((st.m - m_new) * kLog2e), fb = fast_exp2((c.m - m_new) * kLog2e);
#pragma unroll
    for (int j = 0; j < 2; j++) st.o[j] = (fa == 0.f ? 0.f : fa * st.o[j]) + fb * c.o[j];
    st.l = (fa == 0.f ? 0.f : fa * st.l) + fb * c.l;
    st.m = m_new;
  }
}
// The state, and (out: the row's output, or null) its last two steps of Alg. 1.
template <typename T>
__device__ __forceinline__ void row_store(const RowState& st, bool fresh, float* O_acc, float* m, float* l, T* out, float* lse,
                                          size_t sr, int d, int lane) {
  const bool some = st.l > 0.f;
  const float inv = some ? 1.0f / st.l : 0.f;
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const int col = lane + 64 * j;
    if (col >= d) continue;
    if (O_acc != nullptr && (fresh || st.m != BURST_NEG_INF)) O_acc[sr * d + col] = st.o[j];
    if (out != nullptr) out[col] = (T)(some ? st.o[j] * inv : 0.f);
  }
  if (lane != 0) return;
  if (O_acc != nullptr && (fresh || st.m != BURST_NEG_INF)) { m[sr] = st.m; l[sr] = st.l; }
  if (out != nullptr) lse[sr] = some ? st.m + __logf(st.l) : BURST_NEG_INF;
}

// dQ of one row without its factor `scale`: every `splits`-th tile of TILE keys of the sequence, from the one at `split`
template <typename T, int TILE, typename A, typename F>
__device__ __forceinline__ void row_dq(float (&dq)[2], const A& a, int head, int row, int lane, F tiles_of, int split, int splits) {
  const size_t sr = (size_t)head * a.Nq + row, qr = a.lay.q_base(head) + (size_t)row * a.lay.qs_r;
  const T* const q = (const T*)a.Q + qr;
  const T* const g = (const T*)a.dO + qr;
  const float lse = a.lse[sr], D = a.D[sr];
  dq[0] = dq[1] = 0.f;
  if (lse == BURST_NEG_INF) return;
  int at = 0;
#pragma unroll 1
  for (int i = 0; i < a.n; i++) {
    const Chunk& C = a.ch[i];
    const size_t base = C.kv_base(head / a.group, a.lay.kv_heads);
    const T* const K = (const T*)C.K + base;
    const T* const V = (const T*)C.V + base;
    int lo, hi;
    tiles_of(C, lo, hi);
#pragma unroll 1
    for (int t = lo; t < hi; t++, at++) {
      if (at % splits != split) continue;
      const int key = t * TILE + lane;
      const bool vis = lane < TILE && key < C.Nc && pair_visible(a, C, head, row, key);
      float ds = 0.f;
      if (vis) {
        const float s = row_dot(q, K + (size_t)key * C.ks_r, a.d);
        ds = fast_exp2(above(s, a.scale, lse) * kLog2e) * (row_dot(g, V + (size_t)key * C.ks_r, a.d) - D);
      }
      for (unsigned long long left = __builtin_amdgcn_ballot_w64(vis); left != 0; left &= left - 1) {
        const int k = __builtin_ctzll(left);
        row_add(dq, __shfl(ds, k), K + (size_t)(t * TILE + k) * C.ks_r, lane, a.d);
      }
    }
  }
}

// dK (without its factor `scale`) and dV of one key, over all query heads of its group
template <typename T, typename A>
__device__ __forceinline__ void key_dkv(float (&dk)[2], float (&dv)[2], const A& a, const Chunk& C, int kvhead, int key, int lane) {
  const size_t kr = C.kv_base(kvhead, a.lay.kv_heads) + (size_t)key * C.ks_r;
  const T* const k = (const T*)C.K + kr;
  const T* const v = (const T*)C.V + kr;
  dk[0] = dk[1] = dv[0] = dv[1] = 0.f;
#pragma unroll 1
  for (int head = kvhead * a.group; head < (kvhead + 1) * a.group; head++) {
    const T* const Q = (const T*)a.Q + a.lay.q_base(head);
    const T* const G = (const T*)a.dO + a.lay.q_base(head);
#pragma unroll 1
    for (int r0 = 0; r0 < a.Nq; r0 += 64) {
      const int row = r0 + lane;
      const size_t sr = (size_t)head * a.Nq + row;
      const bool vis = row < a.Nq && pair_visible(a, C, head, row, key) && a.lse[sr] != BURST_NEG_INF;
      float p = 0.f, ds = 0.f;
      if (vis) {
        const float s = row_dot(Q + (size_t)row * a.lay.qs_r, k, a.d);
        p = fast_exp2(above(s, a.scale, a.lse[sr]) * kLog2e);
        ds = p * (row_dot(G + (size_t)row * a.lay.qs_r, v, a.d) - a.D[sr]);
      }
      for (unsigned long long left = __builtin_amdgcn_ballot_w64(vis); left != 0; left &= left - 1) {
        const int j = __builtin_ctzll(left);
        const size_t at = (size_t)(r0 + j) * a.lay.qs_r;
        row_add(dv, __shfl(p, j), G + at, lane, a.d);
        row_add(dk, __shfl(ds, j), Q + at, lane, a.d);
      }
    }
  }
}
// A gradient row times f: fp32, added to what is there (acc), or (half) of type T
template <typename T>
__device__ __forceinline__ void row_gradient(void* base, size_t at, const float (&g)[2], float f, int half, int acc, int lane, int d) {
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const int col = lane + 64 * j;
    if (col >= d) continue;
    if (half) ((T*)base)[at + col] = (T)(f * g[j]);
    else ((float*)base)[at + col] = (acc ? ((float*)base)[at + col] : 0.f) + f * g[j];
  }
}

}  // namespace burst
