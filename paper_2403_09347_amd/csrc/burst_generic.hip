// Forward and backward for every call that the bf16 MFMA kernels do not take: fp32 tensors, bf16
// head dimensions that are no multiple of 8, slices or chunks beyond the 32-bit addressing of those
// kernels.  Same mathematics (paper Alg. 1 loop body + merge, Alg. 2 block pair), all of it in fp32
// on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products, fp32 accumulation).
//
// What they are built around: the fp32 matrix rate (157 TFLOP/s nominal, 153 measured for a large product), 64
// cycles per MFMA, so that operand traffic is small beside it.  A wavefront owns 32 query rows (or 32 keys), keeps their
// operands and accumulators in registers and walks the other side in 32-row tiles: fp32 through LDS of its own, without
// barriers (LdsTile); other types and strides straight from memory, each operand while the MFMAs of the one before it
// run.  The wavefronts of a workgroup share one row block and take its tiles in turn (their partial results meet in LDS at
// the end, in a fixed order): a slice of 256 rows would otherwise keep 8 of the chip's 1024 SIMDs busy.  Where that is not
// enough several workgroups share a block (SPLIT).
// Measured per launch, forward / dQ / dK+dV, fp32, with operands from memory / through LDS: 8 heads of 700 rows x 1400 causal keys,
// d = 128, 71 / 104 / 121 -> 68 / 89 / 100 us; 4 x 1000 x 3000, d = 64, 53 / 63 / 112 -> 51 / 60 / 85; 8 x 1000 x 4000, d = 32,
// 67 / 82 / 134 -> 61 / 71 / 100.  What is left at 700 rows: 176 row blocks for 256 CUs, of unequal length, one wavefront
// per SIMD, and about 12 us a workgroup before and after its tiles.
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
  int order;                                      // see grid_order
  int n;                                          // chunks
  Chunk ch[kMaxChunks];
  // SPLIT: a block's tiles are shared by the wavefronts of several workgroups, whose partial results another launch merges
  const void* O;                                  // dQ, VEC: D is computed from it and written (nullptr: D is there)
  float* part; int splits;                        // forward: [split][rows][d] O, then m and l, each [split][rows]; dQ: [split][rows][d]
  RowParts parts;                                 // dK/dV
};

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int reg_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// How one call shape reads its rows.  VEC: fp32 with d a multiple of 4 (see fp32_tiles), whose tiles come through LDS but where
// gen_dispatch says otherwise.
template <typename T, int D, bool VEC>
struct Rows {
  static constexpr int NK = D / 8;                // four-wide operand pieces of a row
  static constexpr int NB = D / 32;               // 32-wide blocks of d
  static constexpr bool PACKED = VEC && D != 96;  // columns NB lr .. NB lr + NB - 1 in one read
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
    if constexpr (PACKED && NB > 1) {
      typedef __attribute__((ext_vector_type(NB))) float vec;
      const vec x = *reinterpret_cast<const vec*>(row + min(NB * lr, d - NB));
#pragma unroll
      for (int db = 0; db < NB; db++) v[db] = x[db];
    } else {
#pragma unroll
      for (int db = 0; db < NB; db++) v[db] = (float)row[min(32 * db + lr, d - 1)];
    }
  }
};

// VEC: a wavefront's tiles of the other side, 32 rows of D floats, come by DMA into LDS of its own (no barriers): read from
// memory directly, the four-wide pieces of 32 rows are as many cache lines per load, each fetched again for the next piece.
// Two tiles per wavefront (K and V, or Q and dO); each is refilled as soon as the last product that reads it has been issued, a
// phase or more ahead of its next use.  Granule g (four floats) of row r sits at slot g ^ (r & 15) (D = 32, 96: & 7), so that
// reads of one granule of 16 rows use all banks (D = 96: two rows each).  Rows and columns that do not exist are zero.
template <int D>
struct LdsTile {
  static constexpr int G = D / 4, LOADS = D / 8, BYTES = 32 * D * 4;   // wave-wide loads of a tile
  static __device__ __forceinline__ int off(int row, int g) { return (row * G + (g ^ (row & (G % 16 == 0 ? 15 : 7)))) * 16; }
  // byte offsets of the lane's granules in a tensor (outside any tile for columns past d)
  static __device__ __forceinline__ void sources(int (&at)[LOADS], int lane, unsigned pitch, int d) {
#pragma unroll
    for (int il = 0; il < LOADS; il++) {
      const int flat = il * 64 + lane, row = flat / G, g = (flat % G) ^ (row & (G % 16 == 0 ? 15 : 7));
      at[il] = 4 * g < d ? (int)(row * pitch) + g * 16 : (int)0x80000000u;
    }
  }
  // rows: how many of the 32 exist
  static __device__ __forceinline__ void fetch(unsigned lds, const float* first, int rows, unsigned pitch, int d, const int (&at)[LOADS]) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(first, (unsigned)(min(rows, 32) - 1) * pitch + 4u * d);
#pragma unroll
    for (int il = 0; il < LOADS; il++) dma_b128_to_lds(rs, lds + il * 1024u, at[il]);
  }
  static __device__ __forceinline__ f32x4 piece(const char* t, int row, int g) { return *reinterpret_cast<const f32x4*>(t + off(row, g)); }
  // block columns of lane lr (Rows::col_of)
  static __device__ __forceinline__ void spread(const char* t, int row, int lr, float (&v)[D / 32]) {
    constexpr int NB = D / 32;
    if constexpr (D == 96) {
#pragma unroll
      for (int db = 0; db < NB; db++) v[db] = *reinterpret_cast<const float*>(t + off(row, 8 * db + (lr >> 2)) + (lr & 3) * 4);
    } else {
      typedef __attribute__((ext_vector_type(NB))) float vec;
      const char* const p = t + off(row, NB * lr >> 2) + (NB * lr & 3) * 4;
      if constexpr (NB == 1) v[0] = *reinterpret_cast<const float*>(p);
      else {
        const vec x = *reinterpret_cast<const vec*>(p);
#pragma unroll
        for (int db = 0; db < NB; db++) v[db] = x[db];
      }
    }
  }
};
// at most N loads outstanding; LDS reads below stay below
template <int N>
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}
// the LDS reads above have been answered
__device__ __forceinline__ void wait_reads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0)
}

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

// Floats of LDS per wavefront: its two tiles, and at the end its partial results.
template <int D, bool VEC>
constexpr int wave_floats() { return VEC ? 64 * D : 32 * D; }

// ---------------------------------------------------------------------------- forward
// LDS: tiles come through LDS (VEC).
template <typename T, int D, bool VEC, int W, bool SPLIT, bool LDS>
__global__ void __launch_bounds__(64 * W, W / 4)
fwd_generic_kernel(GenArgs a) {
  using R = Rows<T, D, VEC>;
  constexpr int NB = R::NB, NK = R::NK, WS = wave_floats<D, LDS>();
  extern __shared__ __attribute__((aligned(16))) float gsh[];          // per wavefront: tiles, then [NB][16][64] partial O^T; [W][32] m, l
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int head, blk, split = 0;
  if (!locate_block(blockIdx.x, a.BH, SPLIT ? a.blocks * a.splits : a.blocks, head, blk, a.order)) return;
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
  if (LDS && more) {
    if constexpr (LDS) {
    using L = LdsTile<D>;
    char* const kl = reinterpret_cast<char*>(gsh) + w * 2 * L::BYTES;
    char* const vl = kl + L::BYTES;
    const unsigned kd = lds_addr(kl), vd = lds_addr(vl);
    f32x4 qf[NK];
    const T* Qr = (const T*)a.Q + a.lay.q_base(head) + (size_t)min(row, a.Nq - 1) * a.lay.qs_r;
#pragma unroll
    for (int ks = 0; ks < NK; ks++) qf[ks] = R::fixed(Qr, 8 * ks + 4 * h, a.d, row < a.Nq);
    wait_loads<0>();                               // (no load of the compiler's own in the loop: it would wait for the DMA too)
    int src[L::LOADS];
    unsigned pitch = (unsigned)at.ks_r * 4u;
    L::sources(src, lane, pitch, a.d);
    auto fetch = [&](unsigned to, const T* base) __attribute__((always_inline)) {
      if (pitch != (unsigned)at.ks_r * 4u) {       // (chunks of another pitch)
        pitch = (unsigned)at.ks_r * 4u;
        L::sources(src, lane, pitch, a.d);
      }
      L::fetch(to, base + (size_t)at.t * 32 * at.ks_r, at.Nc - at.t * 32, pitch, a.d, src);
    };
    fetch(kd, at.K);
    fetch(vd, at.V);
    while (more) {
      const int key0 = at.t * 32, Nc = at.Nc;
      const long long k_off = at.k_off;
      more = at.to(a, head, row0, every, every);
      wait_loads<L::LOADS>();                      // K; V may be on its way
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < NK; ks++) {
        const f32x4 kf = L::piece(kl, lr, 2 * ks + h);
#pragma unroll
        for (int j = 0; j < 4; j++) s = mfma_f32(kf[j], qf[ks][j], s);
      }
      wait_reads();
      if (more) fetch(kd, at.K);
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
      if (more) wait_loads<L::LOADS>();            // V; the next K may be on its way
      else wait_loads<0>();
      // O^T += V^T P^T
#pragma unroll
      for (int r = 0; r < 16; r++) {
        float vf[NB];
        L::spread(vl, reg_row(r, h), lr, vf);
#pragma unroll
        for (int db = 0; db < NB; db++) o[db] = mfma_f32(vf[db], s[r], o[db]);
      }
      wait_reads();
      if (more) fetch(vd, at.V);
    }
    }
  } else if (more) {
    if constexpr (!LDS) {
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
  }
  // the wavefronts' partial results meet in LDS
  float* const ml = gsh + W * WS;
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
    for (int r = 0; r < 16; r++) gsh[w * WS + (db * 16 + r) * 64 + lane] = o[db][r] * own;
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
        for (int i = 0; i < W; i++) v += gsh[i * WS + (db * 16 + r) * 64 + lane];
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
      for (int i = 0; i < W; i++) v += gsh[i * WS + (db * 16 + r) * 64 + lane];
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
  constexpr int NB = R::NB, NK = R::NK, WS = wave_floats<D, VEC>();
  extern __shared__ __attribute__((aligned(16))) float gsh[];          // per wavefront: tiles, then [NB][16][64] partial dQ^T; [W] flags
  const int lane = threadIdx.x & 63, lr = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int head, blk, split = 0;
  if (!locate_block(blockIdx.x, a.BH, SPLIT ? a.blocks * a.splits : a.blocks, head, blk, a.order)) return;
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
  float nD = 0.f;                                  // minus D
  if (VEC && a.O != nullptr) {                     // (every wavefront for itself)
    // in the order of bwd_prepare_kernel's sums, which is a tree over 16-byte pieces: the same bits.  (As two chains of
    // d / 2 products the largest error of D against 64 bits was 2.3 times as large at d = 128.)
    constexpr int L2 = D <= 32 ? 4 : 8;            // pairs of pieces that bwd_prepare_kernel has lanes for
    const size_t from = a.lay.q_base(head) + (size_t)min(row, a.Nq - 1) * a.lay.qs_r;
    float x[L2] = {};
#pragma unroll
    for (int ks = 0; ks < NK; ks++) {
      const f32x4 g = R::fixed((const T*)a.dO + from, 8 * ks + 4 * h, a.d, ok), o = R::fixed((const T*)a.O + from, 8 * ks + 4 * h, a.d, ok);
#pragma unroll
      for (int j = 0; j < 4; j++) x[ks % L2] = fma_in_order(o[j], g[j], x[ks % L2]);
    }
#pragma unroll
    for (int off = L2 / 2; off > 0; off >>= 1)
#pragma unroll
      for (int ks = 0; ks < off; ks++) x[ks] = add_in_order(x[ks], x[ks + off]);
    const float sum = sum_both_halves(x[0]);
    nD = -sum;
    if (ok && h == 0 && w == 0) const_cast<float*>(a.D)[sr] = sum;
  } else if (ok) {
    nD = -a.D[sr];
  }
  KeyWalk<T> at;
  at.c = -1; at.t = at.lo = at.hi = 0;
  bool more = at.to(a, head, row0, SPLIT ? split * W + w : w, every);
  if (VEC && more) {
    if constexpr (VEC) {
    using L = LdsTile<D>;
    char* const kl = reinterpret_cast<char*>(gsh) + w * 2 * L::BYTES;
    char* const vl = kl + L::BYTES;
    const unsigned kd = lds_addr(kl), vd = lds_addr(vl);
    f32x4 qf[NK], gf[NK];
    const size_t qrow = a.lay.q_base(head) + (size_t)min(row, a.Nq - 1) * a.lay.qs_r;
#pragma unroll
    for (int ks = 0; ks < NK; ks++) {
      qf[ks] = R::fixed((const T*)a.Q + qrow, 8 * ks + 4 * h, a.d, ok);
      gf[ks] = R::fixed((const T*)a.dO + qrow, 8 * ks + 4 * h, a.d, ok);
    }
    const float lv = ok ? a.lse[sr] : BURST_NEG_INF;
    const float nlse = lv == BURST_NEG_INF ? BURST_NEG_INF : -lv;   // -inf: P = 0
    wait_loads<0>();
    int src[L::LOADS];
    unsigned pitch = (unsigned)at.ks_r * 4u;
    L::sources(src, lane, pitch, a.d);
    auto fetch = [&](unsigned to, const T* base) __attribute__((always_inline)) {
      if (pitch != (unsigned)at.ks_r * 4u) {       // (chunks of another pitch)
        pitch = (unsigned)at.ks_r * 4u;
        L::sources(src, lane, pitch, a.d);
      }
      L::fetch(to, base + (size_t)at.t * 32 * at.ks_r, at.Nc - at.t * 32, pitch, a.d, src);
    };
    fetch(vd, at.V);
    fetch(kd, at.K);
    while (more) {                                 // V's product first: K, which is read last, has that long to arrive
      const int key0 = at.t * 32, Nc = at.Nc;
      const long long k_off = at.k_off;
      more = at.to(a, head, row0, every, every);
      wait_loads<L::LOADS>();
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = nD; }
#pragma unroll
      for (int ks = 0; ks < NK; ks++) {
        const f32x4 vf = L::piece(vl, lr, 2 * ks + h);
#pragma unroll
        for (int j = 0; j < 4; j++) dp = mfma_f32(vf[j], gf[ks][j], dp);
      }
      wait_reads();
      if (more) {
        fetch(vd, at.V);
        wait_loads<L::LOADS>();
      } else {
        wait_loads<0>();
      }
#pragma unroll
      for (int ks = 0; ks < NK; ks++) {
        const f32x4 kf = L::piece(kl, lr, 2 * ks + h);
#pragma unroll
        for (int j = 0; j < 4; j++) s = mfma_f32(kf[j], qf[ks][j], s);
      }
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
      for (int r = 0; r < 16; r++) {
        float kt[NB];
        L::spread(kl, reg_row(r, h), lr, kt);
#pragma unroll
        for (int db = 0; db < NB; db++) dq[db] = mfma_f32(kt[db], dp[r], dq[db]);
      }
      wait_reads();
      if (more) fetch(kd, at.K);
    }
    }
  } else if (more) {
    if constexpr (!VEC) {
    f32x4 qf[NK], gf[NK], kf[NK];
    const size_t qrow = a.lay.q_base(head) + (size_t)min(row, a.Nq - 1) * a.lay.qs_r;
#pragma unroll
    for (int ks = 0; ks < NK; ks++) {
      qf[ks] = R::fixed((const T*)a.Q + qrow, 8 * ks + 4 * h, a.d, ok);
      gf[ks] = R::fixed((const T*)a.dO + qrow, 8 * ks + 4 * h, a.d, ok);
    }
    const float lv = ok ? a.lse[sr] : BURST_NEG_INF;
    const float nlse = lv == BURST_NEG_INF ? BURST_NEG_INF : -lv;   // -inf: P = 0
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
  }
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) gsh[w * WS + (db * 16 + r) * 64 + lane] = dq[db][r];
  unsigned most = 0;
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) most = larger_of(most, dq[db][r]);
  if (any_wave_odd<W>(gsh + W * WS, w, lane, ok && most >= kInfBits) && !SPLIT) {   // the block's rows by themselves, see burst_rows.h
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
      for (int i = 0; i < W; i++) v += gsh[i * WS + (db * 16 + r) * 64 + lane];
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
  constexpr int NB = R::NB, NK = R::NK, WS = wave_floats<D, VEC>();
  extern __shared__ __attribute__((aligned(16))) float gsh[];          // per wavefront: tiles, then [NB][16][64] partial dK, then dV; statistics, then flags
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
    if (!locate_block((int)blockIdx.x - C.first_block, a.BH / a.group, (Nc + 31) >> 5, kvhead, blk, C.order)) return;
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
  if (VEC && n < total) {
    if constexpr (VEC) {
    f32x4 kf[NK], vf[NK];
    const size_t krow = C.kv_base(kvhead, a.lay.kv_heads) + (size_t)min(key, Nc - 1) * C.ks_r;
#pragma unroll
    for (int ks = 0; ks < NK; ks++) {
      kf[ks] = R::fixed((const T*)C.K + krow, 8 * ks + 4 * h, a.d, key < Nc);
      vf[ks] = R::fixed((const T*)C.V + krow, 8 * ks + 4 * h, a.d, key < Nc);
    }
    using L = LdsTile<D>;
    char* const ql = reinterpret_cast<char*>(gsh) + w * 2 * L::BYTES;
    char* const gl = ql + L::BYTES;
    const float* const stat = reinterpret_cast<const float*>(reinterpret_cast<const char*>(gsh) + W * 2 * L::BYTES + w * 512);   // lse, then D, of the tile's rows
    const unsigned qd = lds_addr(ql), gd = lds_addr(gl), sd = lds_addr(stat);
    wait_loads<0>();
    int src[L::LOADS];
    const unsigned pitch = (unsigned)a.lay.qs_r * 4u;
    L::sources(src, lane, pitch, a.d);
    int head, tile;
    place(n, head, tile);
    auto fetch = [&](unsigned to, const void* x) __attribute__((always_inline)) {
      L::fetch(to, (const T*)x + a.lay.q_base(head) + (size_t)tile * 32 * a.lay.qs_r, a.Nq - tile * 32, pitch, a.d, src);
    };
    auto fetch_g = [&]() __attribute__((always_inline)) {
      fetch(gd, a.dO);
      const size_t sr = (size_t)head * a.Nq + tile * 32;
      const unsigned bytes = 4u * min(32, a.Nq - tile * 32);
      dma_b32_to_lds(make_rsrc(a.lse + sr, bytes), sd, lr * 4);
      dma_b32_to_lds(make_rsrc(a.D + sr, bytes), sd + 256, lr * 4);
    };
    fetch_g();
    fetch(qd, a.Q);
    while (n < total) {                            // dO's product first: Q, which is read last, has that long to arrive
      const int row0 = tile * 32;
      const int nn = seek(n + every);
      const bool more = nn < total;
      if (more) place(nn, head, tile);
      wait_loads<L::LOADS>();
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < NK; ks++) {
        const f32x4 x = L::piece(gl, lr, 2 * ks + h);
#pragma unroll
        for (int j = 0; j < 4; j++) dp = mfma_f32(x[j], vf[ks][j], dp);
      }
      wait_loads<0>();
#pragma unroll
      for (int ks = 0; ks < NK; ks++) {
        const f32x4 x = L::piece(ql, lr, 2 * ks + h);
#pragma unroll
        for (int j = 0; j < 4; j++) s = mfma_f32(x[j], kf[ks][j], s);
      }
      float lrow[16], drow[16];
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(stat + 8 * q4 + 4 * h), d4 = *reinterpret_cast<const f32x4*>(stat + 64 + 8 * q4 + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; j++) { lrow[4 * q4 + j] = l4[j]; drow[4 * q4 + j] = d4[j]; }
      }
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
#pragma unroll
      for (int r = 0; r < 16; r++) {
        float x[NB];
        L::spread(gl, reg_row(r, h), lr, x);
#pragma unroll
        for (int db = 0; db < NB; db++) dv[db] = mfma_f32(s[r], x[db], dv[db]);
      }
      wait_reads();
      if (more) fetch_g();
#pragma unroll
      for (int r = 0; r < 16; r++) {
        float x[NB];
        L::spread(ql, reg_row(r, h), lr, x);
#pragma unroll
        for (int db = 0; db < NB; db++) dk[db] = mfma_f32(dp[r], x[db], dk[db]);
      }
      wait_reads();
      if (more) fetch(qd, a.Q);
      n = nn;
    }
    }
  } else if (n < total) {
    if constexpr (!VEC) {
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
  }
  unsigned most = 0;
#pragma unroll
  for (int db = 0; db < NB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) most = larger_of(larger_of(most, dk[db][r]), dv[db][r]);
  if (any_wave_odd<W>(gsh + W * WS + (VEC ? 128 * W : 0), w, lane, most >= kInfBits) && parts == 1) {   // (parts: the merging launch sees to it)
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
      for (int r = 0; r < 16; r++) gsh[w * WS + (db * 16 + r) * 64 + lane] = which ? dv[db][r] : dk[db][r];
    __syncthreads();
    // the head's keys: partial ones of the chunk's span, or the chunk's own
    void* base = which ? C.dV : C.dK;
    size_t first = (size_t)kvhead * Nc;
    if (SPLIT && parts > 1) { base = a.parts.at(part, which, C, kvhead, a.d); first = -(size_t)C.span_lo; }
    const float f = which ? 1.f : a.scale;
    const int half = parts > 1 ? 0 : a.half, acc = parts > 1 ? 0 : a.acc_dkv;
#pragma unroll
    for (int rr = 0; rr < 16 / W; rr++) {
      const int r = w * (16 / W) + rr, k = key0 + reg_row(r, h);
      if (k >= Nc) continue;
      float* const out = (float*)base + (first + k) * a.d;
      T* const out16 = (T*)base + (first + k) * a.d;
#pragma unroll
      for (int db = 0; db < NB; db++) {
        float v = 0.f;
#pragma unroll
        for (int i = 0; i < W; i++) v += gsh[i * WS + (db * 16 + r) * 64 + lane];
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
  for (int i = 0; i < a.splits; i += 4) {          // (four splits' loads together)
    float x[4][2];
#pragma unroll
    for (int j = 0; j < 4; j++) row_load(x[j], a.part + ((size_t)min(i + j, a.splits - 1) * rows + row) * a.d, lane, a.d);
#pragma unroll
    for (int j = 0; j < 4; j++) {
      if (i + j >= a.splits) break;
      const float fi = lane_value(f, i + j);
      o[0] = __builtin_fmaf(fi, x[j][0], o[0]);
      o[1] = __builtin_fmaf(fi, x[j][1], o[1]);
      l = __builtin_fmaf(fi, lane_value(l_part, i + j), l);
    }
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
  const int kvhead = (row - C.first_row) / C.span_keys, key = C.span_lo + row - C.first_row - kvhead * C.span_keys;
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
template <int KIND, typename T, int D, bool VEC, int W, bool SPLIT = false, bool LDS = VEC>
static int gen_launch(GenArgs& a, long long grid, hipStream_t s) {
  const unsigned lds = (W * wave_floats<D, LDS>() + (KIND == GEN_FWD ? W * 64 : KIND == GEN_DKV && VEC ? W * 129 : W)) * 4;
  void (*kernel)(GenArgs);
  if constexpr (KIND == GEN_FWD) kernel = fwd_generic_kernel<T, D, VEC, W, SPLIT, LDS>;
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
static int gen_dispatch(GenArgs& a, const KParams& p, int dtype, hipStream_t s) {
  long long grid = 0;
  if (KIND == GEN_DKV) {
    for (int i = 0; i < a.n; i++) {
      const long long blocks = ((long long)a.ch[i].Nc + 31) / 32;
      a.ch[i].first_block = (int)grid;
      grid += a.parts.splits > 1 ? part_grid(a.BH / a.group, blocks, a.parts.splits) : grid_blocks(a.BH / a.group, blocks);
      if (grid > 0x7fffff00LL) return BURST_ERR_SHAPE;
    }
  } else {
    a.blocks = (int)(((long long)a.Nq + 31) / 32);
    grid = grid_blocks(a.BH, (long long)a.blocks * a.splits);
  }
  if (grid > 0x7fffff00LL) return BURST_ERR_SHAPE;
  if (grid == 0) return BURST_OK;
  if (KIND == GEN_DKV)
    for (int i = 0; i < a.n && a.parts.splits == 1; i++) a.ch[i].order = keys_order(p, a.ch[i], a.n, a.BH / a.group, 32, 32, 1);
  else a.order = grid_order(a.BH, (long long)a.blocks * a.splits, unequal_rows(p, a.ch, a.n, 32), 1);
  if (KIND == GEN_DKV ? a.parts.splits > 1 : a.splits > 1) {
    if (dtype != BURST_F32 || !fp32_tiles(a.d, a.lay, a.ch, a.n) || a.ch[0].bmask != nullptr || a.splits > 64) return BURST_ERR_SHAPE;
    return gen_split<KIND>(a, grid, s);
  }
  const bool few = grid <= 256;
  if (dtype == BURST_F32 && fp32_tiles(a.d, a.lay, a.ch, a.n)) {
    if (a.d <= 32) return few ? gen_launch<KIND, float, 32, true, 8>(a, grid, s) : gen_launch<KIND, float, 32, true, 4>(a, grid, s);
    if (a.d <= 64) return few ? gen_launch<KIND, float, 64, true, 8>(a, grid, s) : gen_launch<KIND, float, 64, true, 4>(a, grid, s);
    if constexpr (KIND == GEN_FWD) {
      // One tile a wavefront at most: nothing is fetched ahead, and LDS for two tiles a wavefront leaves a CU one workgroup.  Through
      // LDS / from memory, us, d = 128: 1 x 512 rows x 64 keys 14.4 / 13.4, 32 x 805 x 41 72.3 / 69.3; d = 96, 8 x 1213 x 100 26.0 / 25.1; at d = 64
      // 14.5 / 15.9, and with 7 tiles, d = 128, 20.0 / 20.6.
      long long tiles = 0;
      for (int i = 0; i < a.n; i++) tiles += ((long long)a.ch[i].Nc + 31) / 32;
      if (a.d > 64 && tiles <= 4)
        return a.d <= 96 ? gen_launch<KIND, float, 96, true, 4, false, false>(a, grid, s) : gen_launch<KIND, float, 128, true, 4, false, false>(a, grid, s);
    }
    if (a.d <= 96) return gen_launch<KIND, float, 96, true, 4>(a, grid, s);
    return gen_launch<KIND, float, 128, true, 4>(a, grid, s);
  }
  if (a.O != nullptr) return BURST_ERR_SHAPE;      // (the kernels below leave D to bwd_prepare)
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
  return gen_dispatch<GEN_FWD>(a, p, dtype, s);
}
static void bwd_args(GenArgs& a, const KParams& p, const BwdIo& io, const Chunk* ch, int n) {
  make_args(a, p, ch, n);
  a.Q = io.Q; a.dO = io.dO; a.lse = io.lse; a.D = io.D; a.dQ = io.dQ; a.half = io.half; a.acc_dq = io.acc_dq; a.acc_dkv = io.acc_dkv; a.O = io.O;
  a.part = io.part; a.splits = io.splits > 1 ? io.splits : 1;
  set_row_parts(a, io);
}
int launch_bwd_dq_generic(const KParams& p, int dtype, const BwdIo& io, const Chunk* ch, int n, hipStream_t s) {
  GenArgs a = {};
  bwd_args(a, p, io, ch, n);
  return gen_dispatch<GEN_DQ>(a, p, dtype, s);
}
int launch_bwd_dkv_generic(const KParams& p, int dtype, const BwdIo& io, const Chunk* ch, int n, hipStream_t s) {
  GenArgs a = {};
  bwd_args(a, p, io, ch, n);
  a.O = nullptr;
  return gen_dispatch<GEN_DKV>(a, p, dtype, s);
}

}  // namespace burst
