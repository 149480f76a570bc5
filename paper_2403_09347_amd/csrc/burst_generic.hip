// Forward and backward for every call that the bf16 MFMA kernels do not take: fp32 tensors, bf16
// head dimensions that are no multiple of 8, slices or chunks beyond the 32-bit addressing of those
// kernels.  Same mathematics (paper Alg. 1 loop body + merge, Alg. 2 block pair), all of it in fp32
// on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products, fp32 accumulation).
//
// What they are built around: the fp32 matrix rate (157 TFLOP/s nominal, 153 measured for a large product), 64
// cycles per MFMA, so that operand traffic is small beside it.  Hence no LDS tiles and no barriers
// in the loops: a wavefront owns 32 query rows (or 32 keys), keeps their operands and accumulators in
// registers and reads the other side's 32-row tiles straight from memory, each operand while the
// MFMAs of the one before it run.  The wavefronts of a workgroup share one row block and take its
// tiles in turn (their partial results meet in LDS at the end, in a fixed order): a slice of 256
// rows would otherwise keep 8 of the chip's 1024 SIMDs busy.
// Measured per launch, forward / dQ / dK+dV, against one wavefront per row with scalar FMAs (the form
// these kernels replace): fp32, 8 heads of 700 x 700 without a mask, d = 128: 448 / 522 / 1927 -> 48 / 64 / 91 us
// (42 / 47 / 44 TFLOP/s, less than a third of the fp32 matrix rate: 176 row blocks for 256 CUs, one wavefront per SIMD, and
// operands whose 32 rows are as many cache lines per load); fp32, one head of 256 x 256, d = 64: 48 / 46 / 93 ->
// 15 / 18 / 27 us; bf16, d = 96, 32 heads of 777 x 777, before these calls went to the padded kernels of
// burst_plain_mfma.h: 1208 / 1070 / 4308 -> 272 / 480 / 587 us.
// Accumulators that come out infinite or NaN: see burst_rows.h.
//
// Operand layouts of v_mfma_f32_32x32x2_f32 (lane = 32 h + lr): A holds [m = lr][k = h], B holds
// [k = h][n = lr], one value each; D register r holds [m = 8 (r / 4) + 4 h + r % 4][n = lr].
//  - Contractions over d read four consecutive d per lane (d = 8 ks + 4 h + j); MFMA j of step ks
//    contracts d = 8 ks + j (h = 0) and 8 ks + 4 + j (h = 1) on both sides.
//  - A score register r is the B operand (forward, dQ) or A operand (dK, dV) of the second product as
//    it stands: its two keys (rows), of h = 0 and h = 1, are the two k of that MFMA.
//  - The other operand of the second product is a row of V, K, dO or Q spread over lr: block db of
//    lane lr is column col_of(db, lr).
#include "burst_bwd_common.h"

namespace burst {

struct GenArgs {
  const void* Q; const void* dO;
  float* O_acc; float* m; float* l;               // forward state
  void* O_out; float* lse_out;                    // O_out != nullptr: the state is final after this launch
  const float* lse; const float* D;               // backward inputs
  void* dQ;                                       // fp32, or T (half), as dK and dV
  int half;
  int Nq, d, BH;
  int causal, fresh;                              // fresh: the state before the launch is the initial one
  float scale;
  long long q_off;
  long long window;
  int bsize;                                      // edge of block flags, a multiple of 64
  Layout lay;                                     // strides of Q, dO, O_out
  int group;                                      // query heads per key/value head
  int acc_dq, acc_dkv;
  int blocks;                                     // forward, dQ: 32-row blocks per head
  int n;                                          // chunks
  Chunk ch[kMaxChunks];
  // SPLIT: a block's tiles are shared by the wavefronts of several workgroups, whose partial results another launch merges
  float* part; int splits;                        // forward: [split][rows][d] O, then m and l, each [split][rows]; dQ: [split][rows][d]
  RowParts parts;                                 // dK/dV
};

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int reg_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// How one call shape reads its rows.  VEC: fp32 with d a multiple of 4 (rows then start on 16 bytes).
template <typename T, int D, bool VEC>
struct Rows {
  static constexpr int NK = D / 8;                // four-wide operand pieces of a row
  static constexpr int NB = D / 32;               // 32-wide blocks of d
  static constexpr bool PACKED = VEC && D != 96;  // columns NB lr .. NB lr + NB - 1 in one load
  static __device__ __forceinline__ int col_of(int db, int lr) { return PACKED ? NB * lr + db : 32 * db + lr; }
  // columns 8 ks + 4 h .. + 3.  Past d: whatever the row's last columns hold (the other operand, `fixed`
  // below, is zero there).
  static __device__ __forceinline__ f32x4 piece(const T* row, int col, int d) {
    f32x4 v;
    if constexpr (VEC) {
      v = *reinterpret_cast<const f32x4*>(row + min(col, d - 4));
    } else {
#pragma unroll
      for (int j = 0; j < 4; j++) v[j] = (float)row[min(col + j, d - 1)];
    }
    return v;
  }
  // the same, zero past d and in rows that do not exist
  static __device__ __forceinline__ f32x4 fixed(const T* row, int col, int d, bool ok) {
    f32x4 v = piece(row, col, d);
#pragma unroll
    for (int j = 0; j < 4; j++) v[j] = (ok && col + j < d) ? v[j] : 0.f;
    return v;
  }
  // block columns of lane lr (past d: anything, such columns are never stored)
  static __device__ __forceinline__ void spread(const T* row, int lr, int d, float (&v)[NB]) {
    if constexpr (PACKED) {
      typedef __attribute__((ext_vector_type(NB))) float vec;
      if constexpr (NB == 1) v[0] = row[min(lr, d - 1)];
      else {
        const vec x = *reinterpret_cast<const vec*>(row + min(NB * lr, d - NB));
#pragma unroll
        for (int db = 0; db < NB; db++) v[db] = x[db];
      }
    } else {
#pragma unroll
      for (int db = 0; db < NB; db++) v[db] = (float)row[min(32 * db + lr, d - 1)];
    }
  }
};

// Query tiles (32 rows) that see keys [key0, key0 + 32) of the chunk.
__device__ __forceinline__ void row_tiles(const GenArgs& a, const Chunk& C, int key0, int& lo, int& hi) {
  lo = 0; hi = (a.Nq + 31) >> 5;
  if (a.causal) {
    const long long first = C.k_off + key0 - a.q_off;
    if (first >= a.Nq) lo = hi;
    else if (first > 0) lo = (int)(first >> 5);
  }
  if (a.window > 0) {
    const long long last = C.k_off + min(key0 + 31, C.Nc - 1) + a.window - 1 - a.q_off;
    if (last < 0) hi = 0;
    else if ((last >> 5) + 1 < hi) hi = (int)(last >> 5) + 1;
  }
}
// A 32 x 32 tile lies in one block of the flags (their edge is a multiple of 64).
__device__ __forceinline__ bool tile_flag(const GenArgs& a, const Chunk& C, int head, int row0, int key0) {
  if (C.bmask == nullptr) return true;
  return C.bmask[(size_t)head * C.bhstride + (size_t)(row0 / a.bsize) * C.bpitch + key0 / a.bsize] != 0;
}
// The key tiles that rows [row0, row0 + 32) see, chunk after chunk, every `every`-th of them: the share of one
// wavefront.
template <typename T>
struct KeyWalk {
  int c, t, lo, hi;                               // chunk, tile, its chunk's visible range
  const T* K; const T* V;                         // of the chunk, this head
  long long ks_r, k_off;
  int Nc;
  __device__ __forceinline__ bool to(const GenArgs& a, int head, int row0, int step, int every) {
    t += step;
    for (;;) {
      while (t >= hi) {
        const int past = t - hi;
        if (++c >= a.n) return false;
        const Chunk& C = a.ch[c];
        Nc = C.Nc; k_off = C.k_off; ks_r = C.ks_r;
        lo = 0; hi = (Nc + 31) >> 5;
        if (a.causal) {
          const long long last = a.q_off + min(row0 + 31, a.Nq - 1) - k_off;   // last visible key
          if (last < 0) hi = 0;
          else if ((last >> 5) + 1 < hi) hi = (int)(last >> 5) + 1;
        }
        if (a.window > 0) {
          const long long first = a.q_off + row0 - a.window + 1 - k_off;
          if (first >= Nc) lo = hi;
          else if (first > 0) lo = (int)(first >> 5);
        }
        hi = max(hi, lo);
        const size_t base = C.kv_base(head / a.group, a.lay.kv_heads);
        K = (const T*)C.K + base; V = (const T*)C.V + base;
        t = lo + past;
      }
      if (tile_flag(a, a.ch[c], head, row0, t * 32)) return true;
      t += every;
    }
  }
};

// Barrier of the workgroup; whether `odd` holds in a lane of any of its wavefronts (flags: W words of LDS).
template <int W>
__device__ __forceinline__ bool any_wave_odd(float* flags, int w, int lane, bool odd) {
  int* const f = reinterpret_cast<int*>(flags);
  const int mine = __builtin_amdgcn_ballot_w64(odd) != 0;
  if (lane == 0) f[w] = mine;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int i = 0; i < W; i++) any |= f[i];
  return __builtin_amdgcn_readfirstlane(any) != 0;
}

// The share of wavefront w of a block's 32 rows or keys.
template <int W>
__device__ __forceinline__ unsigned share(int w) { return ((1u << (32 / W)) - 1u) << (w * (32 / W)); }

// ---------------------------------------------------------------------------- forward
template <typename T, int D, bool VEC, int W, bool SPLIT>
__global__ void __launch_bounds__(64 * W, W / 4)
fwd_generic_kernel(GenArgs a) {
  using R = Rows<T, D, VEC>;
  constexpr int NB = R::NB, NK = R::NK;
  extern __shared__ __attribute__((aligned(16))) float gsh[];          // [W][NB][16][64] partial O^T, then [W][32] m, l
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int head, blk, split = 0;
  if (!locate_block(blockIdx.x, a.BH, SPLIT ? a.blocks * a.splits : a.blocks, head, blk)) return;
  if constexpr (SPLIT) {
    split = blk % a.splits; blk /= a.splits;
  }
  if (a.causal) blk = a.blocks - 1 - blk;          // later blocks see more keys: the long ones start first
  const int every = SPLIT ? W * a.splits : W;      // wavefronts that share the block
  const int row0 = blk * 32, row = row0 + lr;

  f32x16 o[NB];
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[db][r] = 0.f;
  float m_run = BURST_NEG_INF, lsum = 0.f;        // reference max, sum over this lane's keys

  KeyWalk<T> at;
  at.c = -1; at.t = at.lo = at.hi = 0;
  bool more = at.to(a, head, row0, SPLIT ? split * W + w : w, every);
  if (more) {
    f32x4 qf[NK], kf[NK];
    const T* Qr = (const T*)a.Q + a.lay.q_base(head) + (size_t)min(row, a.Nq - 1) * a.lay.qs_r;
#pragma unroll
    for (int ks = 0; ks < NK; ks++) qf[ks] = R::fixed(Qr, 8 * ks + 4 * h, a.d, row < a.Nq);
    auto load_k = [&]() __attribute__((always_inline)) {
      const T* kr = at.K + (size_t)min(at.t * 32 + lr, at.Nc - 1) * at.ks_r;
#pragma unroll
      for (int ks = 0; ks < NK; ks++) kf[ks] = R::piece(kr, 8 * ks + 4 * h, a.d);
    };
    load_k();
    while (more) {
      const int key0 = at.t * 32, Nc = at.Nc;
      const long long k_off = at.k_off, ks_r = at.ks_r;
      const T* const Kh = at.K;
      const T* const Vh = at.V;
      more = at.to(a, head, row0, every, every);
      float vf[16][NB];
      auto load_v = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
        for (int r = r0; r < r0 + 8; r++)
          R::spread(Vh + (size_t)min(key0 + reg_row(r, h), Nc - 1) * ks_r, lr, a.d, vf[r]);
      };
      load_v(0);
      __builtin_amdgcn_sched_barrier(0);
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < NK; ks++)
#pragma unroll
        for (int j = 0; j < 4; j++) s = mfma_f32(kf[ks][j], qf[ks][j], s);
      __builtin_amdgcn_sched_barrier(0);
      load_v(8);
      // masks: register r holds key key0 + 4 h + cpart; visible iff cpart in [lim_lo, lim]
      const long long dd = (a.q_off - k_off) + row - ((long long)key0 + 4 * h);
      int lim = min(64, Nc - 1 - (key0 + 4 * h)), lim_lo = -1;
      if (a.causal) lim = (int)min((long long)lim, dd < -1 ? -1LL : dd);
      if (a.window > 0) { const long long dl = dd - a.window + 1; lim_lo = (int)(dl < -1 ? -1 : dl > 64 ? 64 : dl); }
      float v = BURST_NEG_INF;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int cpart = 8 * (r >> 2) + (r & 3);
        s[r] = (cpart <= lim && cpart >= lim_lo) ? product(s[r], a.scale) : BURST_NEG_INF;
        v = fmaxf(v, s[r]);
      }
      const float m_new = fmaxf(m_run, max_both_halves(v)), ref = m_new == BURST_NEG_INF ? 0.f : m_new;
      const float alpha = fast_exp2((m_run - ref) * kLog2e);
      m_run = m_new;
      lsum *= alpha;
#pragma unroll
      for (int db = 0; db < NB; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[db][r] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; r++) { s[r] = fast_exp2((s[r] - ref) * kLog2e); lsum += s[r]; }
      // O^T += V^T P^T
#pragma unroll
      for (int r = 0; r < 8; r++)
#pragma unroll
        for (int db = 0; db < NB; db++) o[db] = mfma_f32(vf[r][db], s[r], o[db]);
      __builtin_amdgcn_sched_barrier(0);
      if (more) load_k();
#pragma unroll
      for (int r = 8; r < 16; r++)
#pragma unroll
        for (int db = 0; db < NB; db++) o[db] = mfma_f32(vf[r][db], s[r], o[db]);
    }
  }
  // the wavefronts' partial results meet in LDS
  float* const ml = gsh + W * NB * 1024;
  unsigned most = larger_of(0, lsum);              // a wavefront with an infinity or NaN says so by its row sums
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) most = larger_of(most, o[db][r]);
  const bool odd = __builtin_amdgcn_ballot_w64(row < a.Nq && most >= kInfBits) != 0;
  const float l_half = odd ? -BURST_NEG_INF : sum_both_halves(lsum);
  if (h == 0) { ml[w * 64 + lr] = m_run; ml[w * 64 + 32 + lr] = l_half; }
  __syncthreads();
  float mg = BURST_NEG_INF, lg = 0.f;
#pragma unroll
  for (int i = 0; i < W; i++) mg = fmaxf(mg, ml[i * 64 + lr]);
  const float mref = mg == BURST_NEG_INF ? 0.f : mg;
#pragma unroll
  for (int i = 0; i < W; i++) lg += ml[i * 64 + 32 + lr] * fast_exp2((ml[i * 64 + lr] - mref) * kLog2e);
  if (!SPLIT && __builtin_amdgcn_ballot_w64(row < a.Nq && larger_of(0, lg) >= kInfBits) != 0) {   // (alike in all wavefronts) the block's rows by themselves, see burst_rows.h
    for (unsigned left = first_bits(a.Nq - row0) & share<W>(w); left != 0;) {
      int rows[kRows];
      const int n = next_rows(left, row0, rows);
      RowState st[kRows];
#pragma unroll
      for (int r = 0; r < kRows; r++) st[r] = row_state(a.fresh, a.O_acc, a.m, a.l, (size_t)head * a.Nq + rows[r], a.d, lane);
      rows_forward<T, VEC>(st, args_again<GenArgs>(), head, rows, lane, [](const Chunk& C, int& lo, int& hi) { lo = 0; hi = (C.Nc + 63) >> 6; }, 0, 0x7fffffff);
#pragma unroll
      for (int r = 0; r < kRows; r++)
        if (r < n)
          row_store<T>(st[r], a.fresh, a.O_acc, a.m, a.l, a.O_out == nullptr ? nullptr : (T*)a.O_out + a.lay.q_base(head) + (size_t)rows[r] * a.lay.qs_r,
                       a.lse_out, (size_t)head * a.Nq + rows[r], a.d, lane);
    }
    return;
  }
  const float own = fast_exp2((m_run - mref) * kLog2e);
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) gsh[((w * NB + db) * 16 + r) * 64 + lane] = o[db][r] * own;
  __syncthreads();
  if constexpr (SPLIT) {                           // the partial state (an l that is no finite number: see merge_fwd_generic_kernel)
    if (row >= a.Nq) return;
    const size_t rows = (size_t)a.BH * a.Nq, pr = (size_t)split * rows + (size_t)head * a.Nq + row;
    if (w == 0 && h == 0) {
      float* const pm = a.part + (size_t)a.splits * rows * a.d;
      pm[pr] = mg;
      pm[(size_t)a.splits * rows + pr] = lg;
    }
#pragma unroll
    for (int rr = 0; rr < 16 / W; rr++) {
      const int r = w * (16 / W) + rr, mrow = reg_row(r, h);
#pragma unroll
      for (int db = 0; db < NB; db++) {
        float v = 0.f;
#pragma unroll
        for (int i = 0; i < W; i++) v += gsh[((i * NB + db) * 16 + r) * 64 + lane];
        const int col = R::col_of(db, mrow);
        if (col < a.d) a.part[pr * a.d + col] = v;
      }
    }
    return;
  }
  const bool saw = mg != BURST_NEG_INF;
  if (row >= a.Nq || (!saw && !a.fresh && a.O_out == nullptr)) return;   // rows that saw no key keep their state
  const size_t sr = (size_t)head * a.Nq + row;
  const float m_old = a.fresh ? BURST_NEG_INF : a.m[sr], l_old = a.fresh ? 0.f : a.l[sr];
  const float m_new = fmaxf(m_old, mg), ref = m_new == BURST_NEG_INF ? 0.f : m_new;
  const float fa = fast_exp2((m_old - ref) * kLog2e), fb = fast_exp2((mg - ref) * kLog2e);
  const float l_new = (fa == 0.f ? 0.f : fa * l_old) + fb * lg;
  __syncthreads();                                 // every wavefront has read the row's old m and l
  if (w == 0 && h == 0) {
    if (a.O_acc != nullptr && (saw || a.fresh)) { a.m[sr] = m_new; a.l[sr] = l_new; }
    if (a.O_out != nullptr) a.lse_out[sr] = l_new > 0.f ? m_new + __logf(l_new) : BURST_NEG_INF;
  }
  const float inv = l_new > 0.f ? 1.0f / l_new : 0.f;
  float* const orow = a.O_acc + sr * a.d;
  T* const out = a.O_out == nullptr ? nullptr : (T*)a.O_out + a.lay.q_base(head) + (size_t)row * a.lay.qs_r;
#pragma unroll
  for (int rr = 0; rr < 16 / W; rr++) {
    const int r = w * (16 / W) + rr, mrow = reg_row(r, h);
#pragma unroll
    for (int db = 0; db < NB; db++) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < W; i++) v += gsh[((i * NB + db) * 16 + r) * 64 + lane];
      const int col = R::col_of(db, mrow);
      if (col < a.d) {
        const float x = (fa == 0.f ? 0.f : fa * orow[col]) + fb * v;
        if (a.O_acc != nullptr && (saw || a.fresh)) orow[col] = x;
        if (out != nullptr) out[col] = (T)(l_new > 0.f ? x * inv : 0.f);
      }
    }
  }
}

// ---------------------------------------------------------------------------- backward, dQ
template <typename T, int D, bool VEC, int W, bool SPLIT>
__global__ void __launch_bounds__(64 * W, VEC && D <= 64 ? 2 : 1)   // (256 registers do at d = 64: two wavefronts per SIMD)
bwd_dq_generic_kernel(GenArgs a) {
  using R = Rows<T, D, VEC>;
  constexpr int NB = R::NB, NK = R::NK;
  extern __shared__ __attribute__((aligned(16))) float gsh[];          // [W][NB][16][64] partial dQ^T, then [W] flags
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int head, blk, split = 0;
  if (!locate_block(blockIdx.x, a.BH, SPLIT ? a.blocks * a.splits : a.blocks, head, blk)) return;
  if constexpr (SPLIT) {
    split = blk % a.splits; blk /= a.splits;
  }
  if (a.causal) blk = a.blocks - 1 - blk;          // later blocks see more keys: the long ones start first
  const int every = SPLIT ? W * a.splits : W;      // wavefronts that share the block
  const int row0 = blk * 32, row = row0 + lr;
  const bool ok = row < a.Nq;
  const size_t sr = (size_t)head * a.Nq + min(row, a.Nq - 1);

  f32x16 dq[NB];
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) dq[db][r] = 0.f;
  KeyWalk<T> at;
  at.c = -1; at.t = at.lo = at.hi = 0;
  bool more = at.to(a, head, row0, SPLIT ? split * W + w : w, every);
  if (more) {
    f32x4 qf[NK], gf[NK], kf[NK];
    const size_t qrow = a.lay.q_base(head) + (size_t)min(row, a.Nq - 1) * a.lay.qs_r;
#pragma unroll
    for (int ks = 0; ks < NK; ks++) {
      qf[ks] = R::fixed((const T*)a.Q + qrow, 8 * ks + 4 * h, a.d, ok);
      gf[ks] = R::fixed((const T*)a.dO + qrow, 8 * ks + 4 * h, a.d, ok);
    }
    const float lv = ok ? a.lse[sr] : BURST_NEG_INF;
    const float nlse = lv == BURST_NEG_INF ? BURST_NEG_INF : -lv;   // -inf: P = 0
    const float nD = ok ? -a.D[sr] : 0.f;
    auto load_k = [&]() __attribute__((always_inline)) {
      const T* kr = at.K + (size_t)min(at.t * 32 + lr, at.Nc - 1) * at.ks_r;
#pragma unroll
      for (int ks = 0; ks < NK; ks++) kf[ks] = R::piece(kr, 8 * ks + 4 * h, a.d);
    };
    load_k();
    while (more) {
      const int key0 = at.t * 32, Nc = at.Nc;
      const long long k_off = at.k_off, ks_r = at.ks_r;
      const T* const Kh = at.K;
      const T* const Vh = at.V;
      more = at.to(a, head, row0, every, every);
      f32x4 vf[NK];
      const T* vr = Vh + (size_t)min(key0 + lr, Nc - 1) * ks_r;
#pragma unroll
      for (int ks = 0; ks < NK; ks++) vf[ks] = R::piece(vr, 8 * ks + 4 * h, a.d);
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = nD; }
#pragma unroll
      for (int ks = 0; ks < NK; ks++)
#pragma unroll
        for (int j = 0; j < 4; j++) s = mfma_f32(kf[ks][j], qf[ks][j], s);
      __builtin_amdgcn_sched_barrier(0);
      float kt[16][NB];
      auto load_kt = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
        for (int r = r0; r < r0 + 8; r++)
          R::spread(Kh + (size_t)min(key0 + reg_row(r, h), Nc - 1) * ks_r, lr, a.d, kt[r]);
        __builtin_amdgcn_sched_barrier(0);
      };
      load_kt(0);
#pragma unroll
      for (int ks = 0; ks < NK; ks++)
#pragma unroll
        for (int j = 0; j < 4; j++) dp = mfma_f32(vf[ks][j], gf[ks][j], dp);
      __builtin_amdgcn_sched_barrier(0);
      load_kt(8);
      const long long dd = (a.q_off - k_off) + row - ((long long)key0 + 4 * h);
      int lim = min(64, Nc - 1 - (key0 + 4 * h)), lim_lo = -1;
      if (a.causal) lim = (int)min((long long)lim, dd < -1 ? -1LL : dd);
      if (a.window > 0) { const long long dl = dd - a.window + 1; lim_lo = (int)(dl < -1 ? -1 : dl > 64 ? 64 : dl); }
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int cpart = 8 * (r >> 2) + (r & 3);
        const float p = fast_exp2(above(s[r], a.scale, -nlse) * kLog2e);
        dp[r] = (cpart <= lim && cpart >= lim_lo) ? p * dp[r] : 0.f;   // dS^T
      }
      // dQ^T += K^T dS^T
#pragma unroll
      for (int r = 0; r < 8; r++)
#pragma unroll
        for (int db = 0; db < NB; db++) dq[db] = mfma_f32(kt[r][db], dp[r], dq[db]);
      __builtin_amdgcn_sched_barrier(0);
      if (more) load_k();
#pragma unroll
      for (int r = 8; r < 16; r++)
#pragma unroll
        for (int db = 0; db < NB; db++) dq[db] = mfma_f32(kt[r][db], dp[r], dq[db]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) gsh[((w * NB + db) * 16 + r) * 64 + lane] = dq[db][r];
  unsigned most = 0;
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) most = larger_of(most, dq[db][r]);
  if (any_wave_odd<W>(gsh + W * NB * 1024, w, lane, ok && most >= kInfBits) && !SPLIT) {   // the block's rows by themselves, see burst_rows.h
    for (unsigned left = first_bits(a.Nq - row0) & share<W>(w); left != 0;) {
      int rows[kRows];
      const int n = next_rows(left, row0, rows);
      float g[kRows][2];
      rows_dq<T, VEC, 64>(g, args_again<GenArgs>(), head, rows, lane, [](const Chunk& C, int& lo, int& hi) { lo = 0; hi = (C.Nc + 63) >> 6; }, 0, 1);
#pragma unroll
      for (int r = 0; r < kRows; r++)
        if (r < n) row_gradient<T>(a.dQ, ((size_t)head * a.Nq + rows[r]) * a.d, g[r], a.scale, a.half, a.acc_dq, lane, a.d);
    }
    return;
  }
  if (!ok) return;
  float* const out = (float*)a.dQ + sr * a.d;
  T* const out16 = (T*)a.dQ + sr * a.d;
#pragma unroll
  for (int rr = 0; rr < 16 / W; rr++) {
    const int r = w * (16 / W) + rr, mrow = reg_row(r, h);
#pragma unroll
    for (int db = 0; db < NB; db++) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < W; i++) v += gsh[((i * NB + db) * 16 + r) * 64 + lane];
      const int col = R::col_of(db, mrow);
      if (col >= a.d) continue;
      if constexpr (SPLIT) a.part[((size_t)split * a.BH * a.Nq + sr) * a.d + col] = a.scale * v;
      else if (a.half) out16[col] = (T)(a.scale * v);
      else out[col] = (a.acc_dq ? out[col] : 0.f) + a.scale * v;
    }
  }
}

// ---------------------------------------------------------------------------- backward, dK dV
// Lane = key; score register r = query row reg_row(r, h) of the tile.
template <typename T, int D, bool VEC, int W, bool SPLIT>
__global__ void __launch_bounds__(64 * W, W / 4)
bwd_dkv_generic_kernel(GenArgs a) {
  using R = Rows<T, D, VEC>;
  constexpr int NB = R::NB, NK = R::NK;
  extern __shared__ __attribute__((aligned(16))) float gsh[];          // [W][NB][16][64] partial dK, then dV; [W] flags
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int ci = 0;                                      // the workgroups of all chunks, chunk after chunk
  while (ci + 1 < a.n && (int)blockIdx.x >= a.ch[ci + 1].first_block) ci++;
  const Chunk& C = a.ch[ci];
  const int Nc = C.Nc;
  int kvhead, blk, part = 0, parts = 1;
  if constexpr (SPLIT) {
    if (!locate_part((int)blockIdx.x - C.first_block, a.BH / a.group, (Nc + 31) >> 5, a.parts.splits, kvhead, blk, part)) return;
  } else {
    if (!locate_block((int)blockIdx.x - C.first_block, a.BH / a.group, (Nc + 31) >> 5, kvhead, blk)) return;
  }
  const int key0 = blk * 32, key = key0 + lr;
  int lo, hi;
  row_tiles(a, C, key0, lo, hi);
  const int per_head = hi - lo, total = max(per_head, 0) * a.group;   // walk positions: the tiles of all heads of the group
  if constexpr (SPLIT) {
    parts = a.parts.of(total);
    if (part >= parts) return;
  }
  const int every = SPLIT ? W * parts : W;         // wavefronts that share the walk
  auto place = [&](int n, int& head, int& tile) __attribute__((always_inline)) {
    const int g = n / per_head;
    head = kvhead * a.group + g;
    tile = lo + n - g * per_head;
  };
  auto seek = [&](int n) {
    while (n < total) {
      int head, tile;
      place(n, head, tile);
      if (tile_flag(a, C, head, tile * 32, key0)) break;
      n += every;
    }
    return n;
  };

  f32x16 dk[NB], dv[NB];
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) { dk[db][r] = 0.f; dv[db][r] = 0.f; }
  int n = seek(SPLIT ? part * W + w : w);
  if (n < total) {
    f32x4 kf[NK], vf[NK];
    const size_t krow = C.kv_base(kvhead, a.lay.kv_heads) + (size_t)min(key, Nc - 1) * C.ks_r;
#pragma unroll
    for (int ks = 0; ks < NK; ks++) {
      kf[ks] = R::fixed((const T*)C.K + krow, 8 * ks + 4 * h, a.d, key < Nc);
      vf[ks] = R::fixed((const T*)C.V + krow, 8 * ks + 4 * h, a.d, key < Nc);
    }
    // A tile is eight groups of MFMAs (S, dP, dV, dK, two halves each); every group's operands are
    // requested one group ahead, which is all that fits beside the resident operands and
    // accumulators (256 registers at d = 128).
    constexpr int HK = NK / 2;
    f32x4 pa[HK], pb[HK];                         // pieces of Q or dO rows: first and second half of a contraction over d
    float ra[8][NB], rb[8][NB];                   // spread rows of dO or Q: first and second half of a contraction over rows
    auto pieces = [&](f32x4 (&dst)[HK], const T* rowp, int half) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < HK; i++) dst[i] = R::piece(rowp, 8 * (half * HK + i) + 4 * h, a.d);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto rows8 = [&](float (&dst)[8][NB], const T* base, int row0, int half) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 8; i++)
        R::spread(base + (size_t)min(row0 + reg_row(8 * half + i, h), a.Nq - 1) * a.lay.qs_r, lr, a.d, dst[i]);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto over_d = [&](f32x16& acc, const f32x4 (&x)[HK], const f32x4 (&y)[NK], int half) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < HK; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc = mfma_f32(x[i][j], y[half * HK + i][j], acc);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto over_rows = [&](f32x16 (&acc)[NB], const f32x16& x, const float (&y)[8][NB], int half) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 8; i++)
#pragma unroll
        for (int db = 0; db < NB; db++) acc[db] = mfma_f32(x[8 * half + i], y[i][db], acc[db]);
      __builtin_amdgcn_sched_barrier(0);
    };
    int head, tile;
    place(n, head, tile);
    const T* qrow = (const T*)a.Q + a.lay.q_base(head) + (size_t)min(tile * 32 + lr, a.Nq - 1) * a.lay.qs_r;
    pieces(pa, qrow, 0);
    while (n < total) {
      const int nn = seek(n + every), row0 = tile * 32;
      const T* Qh = (const T*)a.Q + a.lay.q_base(head);
      const T* Gh = (const T*)a.dO + a.lay.q_base(head);
      const T* grow = Gh + (size_t)min(row0 + lr, a.Nq - 1) * a.lay.qs_r;
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = 0.f; }
      pieces(pb, qrow, 1);
      over_d(s, pa, kf, 0);
      pieces(pa, grow, 0);
      over_d(s, pb, kf, 1);
      float lrow[16], drow[16];
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const size_t sr = (size_t)head * a.Nq + min(row0 + reg_row(r, h), a.Nq - 1);
        lrow[r] = a.lse[sr];
        drow[r] = a.D[sr];
      }
      pieces(pb, grow, 1);
      over_d(dp, pa, vf, 0);
      rows8(ra, Gh, row0, 0);
      over_d(dp, pb, vf, 1);
      rows8(rb, Gh, row0, 1);
      // masks: register r holds row row0 + 4 h + cpart; visible iff cpart in [lim_lo, lim]
      const long long dd = (C.k_off - a.q_off) + key - ((long long)row0 + 4 * h);   // key position - row position at cpart 0
      int lim = min(64, a.Nq - 1 - (row0 + 4 * h)), lim_lo = -1;
      if (a.causal) lim_lo = (int)(dd < -1 ? -1 : dd > 64 ? 64 : dd);
      if (a.window > 0) { const long long dl = dd + a.window - 1; lim = (int)min((long long)lim, dl < -1 ? -1LL : dl); }
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int cpart = 8 * (r >> 2) + (r & 3);
        const bool vis = cpart <= lim && cpart >= lim_lo && lrow[r] != BURST_NEG_INF;
        const float p = fast_exp2(above(s[r], a.scale, lrow[r]) * kLog2e);
        dp[r] = vis ? p * (dp[r] - drow[r]) : 0.f;
        s[r] = vis ? p : 0.f;
      }
      // dV += P^T dO, dK += dS^T Q
      over_rows(dv, s, ra, 0);
      rows8(ra, Qh, row0, 0);
      over_rows(dv, s, rb, 1);
      rows8(rb, Qh, row0, 1);
      over_rows(dk, dp, ra, 0);
      if (nn < total) {
        place(nn, head, tile);
        qrow = (const T*)a.Q + a.lay.q_base(head) + (size_t)min(tile * 32 + lr, a.Nq - 1) * a.lay.qs_r;
        pieces(pa, qrow, 0);
      }
      over_rows(dk, dp, rb, 1);
      n = nn;
    }
  }
  unsigned most = 0;
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) most = larger_of(larger_of(most, dk[db][r]), dv[db][r]);
  if (any_wave_odd<W>(gsh + W * NB * 1024, w, lane, most >= kInfBits) && parts == 1) {   // (parts: the merging launch sees to it)
      // the block's keys by themselves, see burst_rows.h
    for (unsigned left = first_bits(Nc - key0) & share<W>(w); left != 0;) {
      int keys[kRows];
      const int n = next_rows(left, key0, keys);
      float gk[kRows][2], gv[kRows][2];
      keys_dkv<T, VEC>(gk, gv, args_again<GenArgs>(), C, kvhead, keys, lane);
#pragma unroll
      for (int r = 0; r < kRows; r++) {
        if (r >= n) continue;
        const size_t at = ((size_t)kvhead * Nc + keys[r]) * a.d;
        row_gradient<T>(C.dK, at, gk[r], a.scale, a.half, a.acc_dkv, lane, a.d);
        row_gradient<T>(C.dV, at, gv[r], 1.f, a.half, a.acc_dkv, lane, a.d);
      }
    }
    return;
  }
  // lane = column, registers = keys; the two sums use the same LDS one after the other
#pragma unroll
  for (int which = 0; which < 2; which++) {
    if (which) __syncthreads();
#pragma unroll
    for (int db = 0; db < NB; db++)
#pragma unroll
      for (int r = 0; r < 16; r++) gsh[((w * NB + db) * 16 + r) * 64 + lane] = which ? dv[db][r] : dk[db][r];
    __syncthreads();
    float* const to = SPLIT ? a.parts.part + ((size_t)(2 * part + which) * a.parts.rows + C.first_row) * a.d : nullptr;
    void* const base = parts > 1 ? (void*)to : which ? C.dV : C.dK;
    const float f = which ? 1.f : a.scale;
    const int half = parts > 1 ? 0 : a.half, acc = parts > 1 ? 0 : a.acc_dkv;
#pragma unroll
    for (int rr = 0; rr < 16 / W; rr++) {
      const int r = w * (16 / W) + rr, k = key0 + reg_row(r, h);
      if (k >= Nc) continue;
      float* const out = (float*)base + ((size_t)kvhead * Nc + k) * a.d;
      T* const out16 = (T*)base + ((size_t)kvhead * Nc + k) * a.d;
#pragma unroll
      for (int db = 0; db < NB; db++) {
        float v = 0.f;
#pragma unroll
        for (int i = 0; i < W; i++) v += gsh[((i * NB + db) * 16 + r) * 64 + lane];
        const int col = R::col_of(db, lr);
        if (col >= a.d) continue;
        if (half) out16[col] = (T)(f * v);
        else out[col] = (acc ? out[col] : 0.f) + f * v;
      }
    }
  }
}

// ---------------------------------------------------------------------------- merging (SPLIT): one wavefront per row
// Rows whose sum is infinite or NaN are computed by themselves (see burst_rows.h).
template <typename T, bool VEC>
__global__ void __launch_bounds__(256)
merge_fwd_generic_kernel(GenArgs a) {
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rows = (long long)a.BH * a.Nq;
  if (row >= rows) return;
  const int head = (int)(row / a.Nq), at = (int)(row - (long long)head * a.Nq);
  const float* const pm = a.part + (size_t)a.splits * rows * a.d;
  const float* const pl = pm + (size_t)a.splits * rows;
  const int mine = min(lane, a.splits - 1);        // (at most 64 splits)
  const float m_part = pm[(size_t)mine * rows + row], l_part = pl[(size_t)mine * rows + row];
  const float m = wave_max(m_part), ref = m == BURST_NEG_INF ? 0.f : m;
  const float f = fast_exp2((m_part - ref) * kLog2e);
  float o[2] = {0.f, 0.f}, l = 0.f;
#pragma unroll 4
  for (int i = 0; i < a.splits; i++) {
    float x[2];
    row_load(x, a.part + ((size_t)i * rows + row) * a.d, lane, a.d);
    const float fi = lane_value(f, i);
    o[0] = __builtin_fmaf(fi, x[0], o[0]);
    o[1] = __builtin_fmaf(fi, x[1], o[1]);
    l = __builtin_fmaf(fi, lane_value(l_part, i), l);
  }
  RowState st[kRows];
  st[0] = row_state(a.fresh, a.O_acc, a.m, a.l, row, a.d, lane);
  const unsigned most = larger_of(larger_of(larger_of(0, l), o[0]), o[1]);
  if (__builtin_amdgcn_ballot_w64(most >= kInfBits) != 0) {
    const int again[kRows] = {at, at, at};
    st[1] = st[2] = st[0];
    rows_forward<T, VEC>(st, a, head, again, lane, [](const Chunk& C, int& lo, int& hi) { lo = 0; hi = (C.Nc + 63) >> 6; }, 0, 0x7fffffff);
  } else if (m != BURST_NEG_INF) {                 // Alg. 1 merge step
    const float m_new = fmaxf(st[0].m, m);
    const float fa = fast_exp2((st[0].m - m_new) * kLog2e), fb = fast_exp2((m - m_new) * kLog2e);
#pragma unroll
    for (int j = 0; j < 2; j++) st[0].o[j] = (fa == 0.f ? 0.f : fa * st[0].o[j]) + fb * o[j];
    st[0].l = (fa == 0.f ? 0.f : fa * st[0].l) + fb * l;
    st[0].m = m_new;
  }
  row_store<T>(st[0], a.fresh, a.O_acc, a.m, a.l, a.O_out == nullptr ? nullptr : (T*)a.O_out + a.lay.q_base(head) + (size_t)at * a.lay.qs_r,
               a.lse_out, row, a.d, lane);
}
template <typename T, bool VEC>
__global__ void __launch_bounds__(256)
merge_dq_generic_kernel(GenArgs a) {
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rows = (long long)a.BH * a.Nq;
  if (row >= rows) return;
  float g[kRows][2] = {}, scale = 1.f;
#pragma unroll 4
  for (int i = 0; i < a.splits; i++) {
    float x[2];
    row_load(x, a.part + ((size_t)i * rows + row) * a.d, lane, a.d);
    g[0][0] += x[0];
    g[0][1] += x[1];
  }
  if (__builtin_amdgcn_ballot_w64(larger_of(larger_of(0, g[0][0]), g[0][1]) >= kInfBits) != 0) {
    const int head = (int)(row / a.Nq), at = (int)(row - (long long)head * a.Nq);
    const int again[kRows] = {at, at, at};
    rows_dq<T, VEC, 64>(g, a, head, again, lane, [](const Chunk& C, int& lo, int& hi) { lo = 0; hi = (C.Nc + 63) >> 6; }, 0, 1);
    scale = a.scale;
  }
  row_gradient<T>(a.dQ, row * a.d, g[0], scale, a.half, a.acc_dq, lane, a.d);
}
template <typename T, bool VEC>
__global__ void __launch_bounds__(256)
merge_dkv_generic_kernel(GenArgs a) {
  const int lane = threadIdx.x & 63;
  const int row = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= a.parts.rows) return;
  int c = 0;
  while (c + 1 < a.n && row >= a.ch[c + 1].first_row) c++;
  const Chunk& C = a.ch[c];
  const int kvhead = (row - C.first_row) / C.Nc, key = row - C.first_row - kvhead * C.Nc;
  int lo, hi;
  row_tiles(a, C, key & ~31, lo, hi);
  const int parts = a.parts.of(max(hi - lo, 0) * a.group);
  if (parts == 1) return;                          // written by its workgroup
  float gk[kRows][2] = {}, gv[kRows][2] = {}, scale = 1.f;
#pragma unroll 4
  for (int i = 0; i < parts; i++) {
    float x[2], y[2];
    row_load(x, a.parts.part + ((size_t)(2 * i) * a.parts.rows + row) * a.d, lane, a.d);
    row_load(y, a.parts.part + ((size_t)(2 * i + 1) * a.parts.rows + row) * a.d, lane, a.d);
#pragma unroll
    for (int j = 0; j < 2; j++) { gk[0][j] += x[j]; gv[0][j] += y[j]; }
  }
  const unsigned most = larger_of(larger_of(larger_of(larger_of(0, gk[0][0]), gk[0][1]), gv[0][0]), gv[0][1]);
  if (__builtin_amdgcn_ballot_w64(most >= kInfBits) != 0) {
    const int again[kRows] = {key, key, key};
    keys_dkv<T, VEC>(gk, gv, a, C, kvhead, again, lane);
    scale = a.scale;
  }
  const size_t at = ((size_t)kvhead * C.Nc + key) * a.d;
  row_gradient<T>(C.dK, at, gk[0], scale, a.half, a.acc_dkv, lane, a.d);
  row_gradient<T>(C.dV, at, gv[0], 1.f, a.half, a.acc_dkv, lane, a.d);
}

// ---------------------------------------------------------------------------- launchers
static void make_args(GenArgs& a, const KParams& p, const Chunk* ch, int n) {
  a.Nq = p.Nq; a.d = p.d; a.BH = p.B * p.H;
  a.causal = p.causal; a.scale = p.scale; a.q_off = p.q_off; a.window = p.window;
  a.bsize = p.bsize; a.group = p.group; a.lay = p.lay;
  a.n = n;
  for (int i = 0; i < n; i++) a.ch[i] = ch[i];
}

enum { GEN_FWD, GEN_DQ, GEN_DKV };
template <int KIND, typename T, int D, bool VEC, int W, bool SPLIT = false>
static int gen_launch(GenArgs& a, long long grid, hipStream_t s) {
  const unsigned lds = (W * (D / 32) * 1024 + (KIND == GEN_FWD ? W * 64 : W)) * 4;
  void (*kernel)(GenArgs);
  if constexpr (KIND == GEN_FWD) kernel = fwd_generic_kernel<T, D, VEC, W, SPLIT>;
  else if constexpr (KIND == GEN_DQ) kernel = bwd_dq_generic_kernel<T, D, VEC, W, SPLIT>;
  else kernel = bwd_dkv_generic_kernel<T, D, VEC, W, SPLIT>;
  static DeviceOnce lds_opt_in;
  const int st = lds_opt_in.run([&] {
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess ? BURST_OK : BURST_ERR_LAUNCH;
  });
  if (st != BURST_OK) return st;
  BURST_LAUNCH(kernel, dim3((unsigned)grid), dim3(64 * W), lds, s, a);
  return launch_status();
}
// Padded head dimension: the next multiple of 32.  With eight wavefronts per workgroup (two per
// SIMD; the registers allow it up to 64) a row block's tiles are walked in half the time; that pays
// while there are fewer row blocks than CUs.
template <int KIND>
static int gen_split(GenArgs& a, long long grid, hipStream_t s) {      // (fp32, d a multiple of 4)
  const int st = a.d <= 32 ? gen_launch<KIND, float, 32, true, 4, true>(a, grid, s) : a.d <= 64 ? gen_launch<KIND, float, 64, true, 4, true>(a, grid, s)
               : a.d <= 96 ? gen_launch<KIND, float, 96, true, 4, true>(a, grid, s) : gen_launch<KIND, float, 128, true, 4, true>(a, grid, s);
  if (st != BURST_OK) return st;
  const long long rows = KIND == GEN_DKV ? a.parts.rows : (long long)a.BH * a.Nq;
  void (*merge)(GenArgs);
  if constexpr (KIND == GEN_FWD) merge = merge_fwd_generic_kernel<float, true>;
  else if constexpr (KIND == GEN_DQ) merge = merge_dq_generic_kernel<float, true>;
  else merge = merge_dkv_generic_kernel<float, true>;
  BURST_LAUNCH(merge, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, a);
  return launch_status();
}
template <int KIND>
static int gen_dispatch(GenArgs& a, int dtype, hipStream_t s) {
  long long grid = 0, rows = 0;
  if (KIND == GEN_DKV) {
    for (int i = 0; i < a.n; i++) {
      const long long blocks = ((long long)a.ch[i].Nc + 31) / 32;
      a.ch[i].first_block = (int)grid;
      a.ch[i].first_row = (int)rows;               // (used by split launches only, which are small)
      rows += (long long)(a.BH / a.group) * a.ch[i].Nc;
      grid += a.parts.splits > 1 ? part_grid(a.BH / a.group, blocks, a.parts.splits) : grid_blocks(a.BH / a.group, blocks);
      if (grid > 0x7fffff00LL) return BURST_ERR_SHAPE;
    }
  } else {
    a.blocks = (int)(((long long)a.Nq + 31) / 32);
    grid = grid_blocks(a.BH, (long long)a.blocks * a.splits);
  }
  if (grid > 0x7fffff00LL) return BURST_ERR_SHAPE;
  if (grid == 0) return BURST_OK;
  if (KIND == GEN_DKV ? a.parts.splits > 1 : a.splits > 1) {
    if (dtype != BURST_F32 || a.d % 4 != 0 || a.ch[0].bmask != nullptr || a.splits > 64) return BURST_ERR_SHAPE;
    return gen_split<KIND>(a, grid, s);
  }
  const bool few = grid <= 256;
  if (dtype == BURST_F32 && a.d % 4 == 0) {
    if (a.d <= 32) return few ? gen_launch<KIND, float, 32, true, 8>(a, grid, s) : gen_launch<KIND, float, 32, true, 4>(a, grid, s);
    if (a.d <= 64) return few ? gen_launch<KIND, float, 64, true, 8>(a, grid, s) : gen_launch<KIND, float, 64, true, 4>(a, grid, s);
    if (a.d <= 96) return gen_launch<KIND, float, 96, true, 4>(a, grid, s);
    return gen_launch<KIND, float, 128, true, 4>(a, grid, s);
  }
  if (dtype == BURST_F32) return a.d <= 64 ? gen_launch<KIND, float, 64, false, 4>(a, grid, s) : gen_launch<KIND, float, 128, false, 4>(a, grid, s);
  return a.d <= 64 ? gen_launch<KIND, bf16, 64, false, 4>(a, grid, s) : gen_launch<KIND, bf16, 128, false, 4>(a, grid, s);
}

// n <= kMaxChunks chunks.
int launch_fwd_generic(const KParams& p, int dtype, const FwdIo& io, const Chunk* ch, int n, hipStream_t s) {
  GenArgs a = {};
  make_args(a, p, ch, n);
  a.Q = io.Q; a.O_acc = io.O_acc; a.m = io.m; a.l = io.l; a.O_out = io.O_out; a.lse_out = io.lse;
  a.part = io.part; a.splits = io.splits > 1 ? io.splits : 1;
  a.fresh = io.fresh;
  return gen_dispatch<GEN_FWD>(a, dtype, s);
}
static void bwd_args(GenArgs& a, const KParams& p, const BwdIo& io, const Chunk* ch, int n) {
  make_args(a, p, ch, n);
  a.Q = io.Q; a.dO = io.dO; a.lse = io.lse; a.D = io.D; a.dQ = io.dQ; a.half = io.half; a.acc_dq = io.acc_dq; a.acc_dkv = io.acc_dkv;
  a.part = io.part; a.splits = io.splits > 1 ? io.splits : 1;
  a.parts = row_parts(io, ch, n, a.BH / a.group);
}
int launch_bwd_dq_generic(const KParams& p, int dtype, const BwdIo& io, const Chunk* ch, int n, hipStream_t s) {
  GenArgs a = {};
  bwd_args(a, p, io, ch, n);
  return gen_dispatch<GEN_DQ>(a, dtype, s);
}
int launch_bwd_dkv_generic(const KParams& p, int dtype, const BwdIo& io, const Chunk* ch, int n, hipStream_t s) {
  GenArgs a = {};
  bwd_args(a, p, io, ch, n);
  return gen_dispatch<GEN_DKV>(a, dtype, s);
}

}  // namespace burst
