// Query rows (forward, dQ) or keys (dK, dV) by themselves, a few at a time by one wavefront with scalar FMAs: what the matrix-core
// kernels of burst_generic.hip and of the padded builds of burst_plain_mfma.h fall back to where their accumulators come
// out infinite or NaN.  A matrix product multiplies every pair of its operands, also where one of the two is a
// zero that stands for "nothing": a hidden pair, the rows and columns of padding, the lower terms of a probability
// split into three bf16 numbers.  0 x inf is NaN, so one infinite value could reach rows that do not see it, and inf
// could become NaN in a row that does.  Here hidden pairs are skipped and every product is the one of the formula.
// Finite accumulators need no second look: inf and NaN do not go away in a sum, nor when it is scaled.
// Cost: the test at the end of a workgroup; where it strikes, forward / dQ / dK+dV of inputs that are NaN throughout take
// 0.55 / 0.76 / 0.96 ms (fp32, 8 heads of 700 x 700, d = 128; ordinary inputs 50 / 67 / 95 us, the scalar kernels that had these
// calls before 0.49 / 0.59 / 2.4 ms) and 3.1 / 4.8 / 5.2 ms (bf16, 32 heads of 777 causal rows, d = 96; 34 / 36 / 61 us, 1.2 /
// 1.1 / 4.3 ms): bound by the latency of one wavefront per SIMD.  Three rows share a pass over the other side: one row took
// 2.9 / 4.1 / 5.1 ms of the first call, four 0.45 / 0.61 / 0.78 ms, but at four the ordinary fp32 dK+dV spills ten registers
// more (95 -> 98 us).
#pragma once
#include "burst_common.h"

namespace burst {

// The kernel's arguments (its only parameter), read again from where they lie: the fall-back must not keep them in
// registers through the loops before it.
template <typename A>
__device__ __forceinline__ const A& args_again() {
  auto p = (const A __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const A*)p;
}

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
// bits 0 .. n - 1 of 32 (none for n <= 0)
__device__ __forceinline__ unsigned first_bits(int n) { return n >= 32 ? 0xffffffffu : n > 0 ? (1u << n) - 1u : 0u; }
// Rows (of query or key) are taken kRows at a time, so that the other side is read once for all of them.
constexpr int kRows = 3;
// The next of the rows (bits of `left`, counted from `base`) that are to be computed; fewer than kRows: the first one again.
__device__ __forceinline__ int next_rows(unsigned& left, int base, int (&row)[kRows]) {
  int n = 0;
#pragma unroll
  for (int r = 0; r < kRows; r++) {
    row[r] = left != 0 ? base + __builtin_ctz(left) : row[0];
    n += left != 0;
    left &= left - 1;
  }
  return n;
}
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
// columns lane and lane + 64 of a row
template <typename T>
__device__ __forceinline__ void row_load(float (&x)[2], const T* row, int lane, int d) {
  x[0] = lane < d ? (float)row[lane] : 0.f;
  x[1] = lane + 64 < d ? (float)row[lane + 64] : 0.f;
}
// products of the rows x with the lane's own row y (WIDE: rows that start on 16 bytes and are a multiple of 16 bytes long)
template <typename T, bool WIDE>
__device__ __forceinline__ void row_dots(float (&s)[kRows], const float (&x)[kRows][2], const T* y, int d) {
#pragma unroll
  for (int r = 0; r < kRows; r++) s[r] = 0.f;
#pragma unroll
  for (int half = 0; half < 2; half++)
#pragma unroll 1
    for (int t = 0, end = min(64, d - 64 * half); t < end; t += 8) {
      float v[8];
      if constexpr (WIDE) {
        constexpr int E = 16 / sizeof(T);
        typedef __attribute__((ext_vector_type(E))) T vec;
#pragma unroll
        for (int u = 0; u < 8; u += E) {
          const vec x8 = *reinterpret_cast<const vec*>(y + 64 * half + min(t + u, end - E));
#pragma unroll
          for (int j = 0; j < E; j++) v[u + j] = (float)x8[j];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = (float)y[64 * half + min(t + j, end - 1)];
      }
#pragma unroll
      for (int j = 0; j < 8; j++)
        if (t + j < end)
#pragma unroll
          for (int r = 0; r < kRows; r++) s[r] = __builtin_fmaf(lane_value(x[r][half], t + j), v[j], s[r]);
    }
}
// acc[r] += sum over the lanes k in seen[r] of f[r] (of lane k) x row k of `rows` (rows past `last` are not in any seen)
template <typename T>
__device__ __forceinline__ void row_sums(float (&acc)[kRows][2], const float (&f)[kRows], const unsigned long long (&seen)[kRows],
                                         const T* rows, long long pitch, int last, int lane, int d) {
#pragma unroll 1
  for (int k0 = 0; k0 <= min(last, 63); k0 += 8) {
    float x[8][2];
#pragma unroll
    for (int j = 0; j < 8; j++) row_load(x[j], rows + (size_t)min(k0 + j, last) * pitch, lane, d);
#pragma unroll
    for (int j = 0; j < 8; j++)
#pragma unroll
      for (int r = 0; r < kRows; r++)
        if ((seen[r] >> (k0 + j)) & 1) {
          const float one = lane_value(f[r], k0 + j);
          acc[r][0] = __builtin_fmaf(one, x[j][0], acc[r][0]);
          acc[r][1] = __builtin_fmaf(one, x[j][1], acc[r][1]);
        }
  }
}

struct RowState { float m, l, o[2]; };             // o: columns lane and lane + 64
__device__ __forceinline__ RowState row_state(bool fresh, const float* O_acc, const float* m, const float* l, size_t sr, int d, int lane) {
  RowState st = {BURST_NEG_INF, 0.f, {0.f, 0.f}};
  if (!fresh && m[sr] != BURST_NEG_INF) {          // (a row that has seen nothing may hold anything)
    st.m = m[sr]; st.l = l[sr];
    row_load(st.o, O_acc + sr * d, lane, d);
  }
  return st;
}
// The tiles [first, last) of 64 keys of the sequence that `tiles_of` (chunk -> range) makes of the chunks.
template <typename T, bool WIDE, typename A, typename F>
__device__ __forceinline__ void rows_forward(RowState (&st)[kRows], const A& a, int head, const int (&row)[kRows], int lane, F tiles_of,
                                             int first, int last) {
  float q[kRows][2];
#pragma unroll
  for (int r = 0; r < kRows; r++) row_load(q[r], (const T*)a.Q + a.lay.q_base(head) + (size_t)row[r] * a.lay.qs_r, lane, a.d);
  int at = 0;
#pragma unroll 1
  for (int i = 0; i < a.n; i++) {
    const Chunk& C = a.ch[i];
    const size_t base = C.kv_base(head / a.group, a.lay.kv_heads);
    const T* const K = (const T*)C.K + base;
    const T* const V = (const T*)C.V + base;
    float m[kRows], l[kRows], o[kRows][2];
#pragma unroll
    for (int r = 0; r < kRows; r++) { m[r] = BURST_NEG_INF; l[r] = o[r][0] = o[r][1] = 0.f; }
    int lo, hi;
    tiles_of(C, lo, hi);
#pragma unroll 1
    for (int t = lo; t < hi; t++, at++) {
      if (at < first || at >= last) continue;
      const int key = t * 64 + lane;
      float p[kRows];
      unsigned long long seen[kRows];
      row_dots<T, WIDE>(p, q, K + (size_t)min(key, C.Nc - 1) * C.ks_r, a.d);
#pragma unroll
      for (int r = 0; r < kRows; r++) {
        const bool vis = key < C.Nc && pair_visible(a, C, head, row[r], key);
        const float x = vis ? product(p[r], a.scale) : BURST_NEG_INF;
        const float m_new = fmaxf(m[r], wave_max(x)), ref = m_new == BURST_NEG_INF ? 0.f : m_new;
        const float alpha = fast_exp2((m[r] - ref) * kLog2e);
        p[r] = vis ? fast_exp2((x - ref) * kLog2e) : 0.f;
        l[r] = l[r] * alpha + wave_sum(p[r]);
        o[r][0] *= alpha; o[r][1] *= alpha;
        m[r] = m_new;
        seen[r] = __builtin_amdgcn_ballot_w64(vis);
      }
      row_sums(o, p, seen, V + (size_t)t * 64 * C.ks_r, C.ks_r, C.Nc - 1 - t * 64, lane, a.d);
    }
#pragma unroll
    for (int r = 0; r < kRows; r++) {
      if (m[r] == BURST_NEG_INF) continue;         // no key of the chunk: the state stays
      const float m_new = fmaxf(st[r].m, m[r]);    // Alg. 1 merge step
      const float fa = fast_exp2((st[r].m - m_new) * kLog2e), fb = fast_exp2((m[r] - m_new) * kLog2e);
#pragma unroll
      for (int j = 0; j < 2; j++) st[r].o[j] = (fa == 0.f ? 0.f : fa * st[r].o[j]) + fb * o[r][j];
      st[r].l = (fa == 0.f ? 0.f : fa * st[r].l) + fb * l[r];
      st[r].m = m_new;
    }
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

// dQ of the rows without its factor `scale`: every `splits`-th tile of TILE keys of the sequence, from the one at `split`
template <typename T, bool WIDE, int TILE, typename A, typename F>
__device__ __forceinline__ void rows_dq(float (&dq)[kRows][2], const A& a, int head, const int (&row)[kRows], int lane, F tiles_of, int split,
                                        int splits) {
  float q[kRows][2], g[kRows][2], lse[kRows], D[kRows];
#pragma unroll
  for (int r = 0; r < kRows; r++) {
    const size_t sr = (size_t)head * a.Nq + row[r], at = a.lay.q_base(head) + (size_t)row[r] * a.lay.qs_r;
    row_load(q[r], (const T*)a.Q + at, lane, a.d);
    row_load(g[r], (const T*)a.dO + at, lane, a.d);
    lse[r] = a.lse[sr]; D[r] = a.D[sr];
    dq[r][0] = dq[r][1] = 0.f;
  }
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
      float x[kRows], ds[kRows];
      unsigned long long seen[kRows];
      row_dots<T, WIDE>(x, q, K + (size_t)min(key, C.Nc - 1) * C.ks_r, a.d);
      row_dots<T, WIDE>(ds, g, V + (size_t)min(key, C.Nc - 1) * C.ks_r, a.d);
#pragma unroll
      for (int r = 0; r < kRows; r++) {
        const bool vis = lane < TILE && key < C.Nc && lse[r] != BURST_NEG_INF && pair_visible(a, C, head, row[r], key);
        ds[r] = vis ? fast_exp2(above(x[r], a.scale, lse[r]) * kLog2e) * (ds[r] - D[r]) : 0.f;
        seen[r] = __builtin_amdgcn_ballot_w64(vis);
      }
      row_sums(dq, ds, seen, K + (size_t)t * TILE * C.ks_r, C.ks_r, min(TILE, C.Nc - t * TILE) - 1, lane, a.d);
    }
  }
}

// dK (without its factor `scale`) and dV of the keys, over all query heads of their group
template <typename T, bool WIDE, typename A>
__device__ __forceinline__ void keys_dkv(float (&dk)[kRows][2], float (&dv)[kRows][2], const A& a, const Chunk& C, int kvhead,
                                         const int (&key)[kRows], int lane) {
  float k[kRows][2], v[kRows][2];
#pragma unroll
  for (int r = 0; r < kRows; r++) {
    const size_t at = C.kv_base(kvhead, a.lay.kv_heads) + (size_t)key[r] * C.ks_r;
    row_load(k[r], (const T*)C.K + at, lane, a.d);
    row_load(v[r], (const T*)C.V + at, lane, a.d);
    dk[r][0] = dk[r][1] = dv[r][0] = dv[r][1] = 0.f;
  }
#pragma unroll 1
  for (int head = kvhead * a.group; head < (kvhead + 1) * a.group; head++) {
    const T* const Q = (const T*)a.Q + a.lay.q_base(head);
    const T* const G = (const T*)a.dO + a.lay.q_base(head);
#pragma unroll 1
    for (int r0 = 0; r0 < a.Nq; r0 += 64) {
      const int row = r0 + lane, there = min(row, a.Nq - 1);
      const float lse = a.lse[(size_t)head * a.Nq + there], D = a.D[(size_t)head * a.Nq + there];
      unsigned long long seen[kRows], any = 0;
#pragma unroll
      for (int r = 0; r < kRows; r++) {
        seen[r] = __builtin_amdgcn_ballot_w64(row < a.Nq && lse != BURST_NEG_INF && pair_visible(a, C, head, there, key[r]));
        any |= seen[r];
      }
      if (any == 0) continue;
      float p[kRows], ds[kRows];
      row_dots<T, WIDE>(p, k, Q + (size_t)there * a.lay.qs_r, a.d);
      row_dots<T, WIDE>(ds, v, G + (size_t)there * a.lay.qs_r, a.d);
#pragma unroll
      for (int r = 0; r < kRows; r++) {
        p[r] = fast_exp2(above(p[r], a.scale, lse) * kLog2e);
        ds[r] = p[r] * (ds[r] - D);
      }
      const size_t first = (size_t)r0 * a.lay.qs_r;
      row_sums(dv, p, seen, G + first, a.lay.qs_r, a.Nq - 1 - r0, lane, a.d);
      row_sums(dk, ds, seen, Q + first, a.lay.qs_r, a.Nq - 1 - r0, lane, a.d);
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
