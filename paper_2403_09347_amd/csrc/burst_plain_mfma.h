// Plainly written MFMA kernels for the forward chunk step (paper Alg. 1 loop body, tiled as in
// Sec. 2.4) and the two halves of the backward block pair (Alg. 2 loop body), bf16, with the head
// dimension a compile-time constant.  This header is the source of six kernel families; each is
// built by a small translation unit that defines BURST_SMALL_D (head dimension), BURST_SMALL_NS
// (namespace) and, optionally, BURST_SMALL_DKV_WAVES before including it:
//   burst_d64_mfma.hip    d = 64, namespace burst::d64, all three kernels
//   burst_d128_plain.hip  d = 128, namespace burst::d128p, all three kernels, the dK/dV one with
//                         two wavefronts (64 keys) per workgroup (BURST_SMALL_DKV_WAVES = 2)
//   burst_d{32,64,96,128}_pad.hip   every other multiple of 8 below 128, padded to the next of these
//                         widths (BURST_SMALL_PAD), namespaces burst::d32x .. d128x; P and dS with 24 bits; at 128 the dK/dV kernel
//                         with eight wavefronts (BURST_SMALL_DKV_WAVES = 8)
//
// Same mathematics, operand orientations and register layouts as the hand-scheduled d = 128
// kernels (S^T = K Q^T with one query row per lane for the forward and dQ side, S = Q K^T with one
// key per lane for the dK/dV side; P and dS leave the accumulators already in the layout the next
// MFMA wants), but written plainly: one wavefront owns 32 rows (or keys), alone or halving every tile with another
// wavefront (see walk_rows in burst_api.hip), a step runs its phases
// one after the other with compiler-scheduled MFMAs in VGPR accumulators, tiles are
// double-buffered in LDS by DMA with one barrier per tile, and two workgroups share a CU so that
// one's vector work overlaps the other's matrix work.  At d = 64 a tile has half the matrix work
// per score of d = 128 and the same softmax work, so these kernels are bound by the vector unit;
// the hand-interleaved schedules of the d = 128 kernels would buy little here.
//
// LDS tile layout at d = 64: rows of 128 bytes (8 granules of 16 bytes); granule g of row r sits
// at slot g ^ ((r >> 1) & 7), which makes the 128-bit operand reads of 32 consecutive rows
// conflict-free.  At d = 128: the layout of burst_common.h.
#pragma once
#if !defined(BURST_SMALL_D) || !defined(BURST_SMALL_NS)
#error "define BURST_SMALL_D and BURST_SMALL_NS before including burst_plain_mfma.h"
#endif
#include <cmath>
#include "burst_bwd_common.h"
#include "burst_rows.h"

namespace burst {
namespace BURST_SMALL_NS {

// BURST_SMALL_PAD: the call's head dimension is any multiple of 8 up to BURST_SMALL_D (a.d).  Columns
// past it are zero in registers and in LDS (the DMA asks for them outside the buffer, which writes
// zeros and moves nothing) and are never stored.  Rows then lie in LDS with the pitch of the next
// layout there is, 64 or 128 columns.
#ifdef BURST_SMALL_PAD
constexpr bool S_PAD = true;
#else
constexpr bool S_PAD = false;
#endif
constexpr int S_D = BURST_SMALL_D;
constexpr int S_ROWB = S_D <= 64 ? 128 : 256;     // bytes per row in LDS
static_assert(S_PAD || S_ROWB == 2 * S_D, "a head dimension without an LDS layout of its own needs BURST_SMALL_PAD");
constexpr int S_KS = S_D / 16;                    // k-steps of a contraction over d
constexpr int S_DB = S_D / 32;                    // 32-wide blocks of d
constexpr int S_RPL = 1024 / S_ROWB;              // tile rows per wave-wide DMA load
constexpr int S_GPR = S_ROWB / 16;                // granules per row
constexpr float S_LAZY = S_PAD ? 8.0f * kLn2 : 8.0f;   // largest P allowed before the max is raised: 2^8

struct FwdArgsLite {
  const bf16* Q;
  float* O_acc; float* m; float* l;
  bf16* O_out; float* lse;                       // O_out != nullptr: final after this launch
  float* part;                                   // partial states (splits > 1)
  int Nq, H, group;                              // H counts batch x heads
  int causal, fresh;
  float c, scale;                                // c = scale * log2(e)
  long long q_off, window;
  int bsize;
  int blocks_per_head, splits, order;            // order: see grid_order
  int d;                                         // head dimension (S_D unless S_PAD)
  int n;                                         // chunks
  Layout lay;                                    // strides of Q and O_out
  Chunk ch[kMaxChunks];
};
struct BwdArgsLite {
  const bf16* Q; const bf16* dO;
  const float* lse; const float* D;
  void* dQ;                                      // fp32, or bf16 (half), as dK and dV
  int half;
  float* part;                                   // partial dQ (splits > 1)
  int Nq, H, group;                              // H counts batch x heads (dQ: query heads, dK/dV: key/value heads)
  int causal, acc_dq, acc_dkv;
  float c, scale, log2_scale;
  long long q_off, window;
  int bsize;
  int blocks_per_head, splits, order;
  int d, n;
  int per;                                       // dK/dV: workgroups of every chunk (chunk_at)
  RowParts parts;                                // dK/dV
  Layout lay;
  Chunk ch[kMaxChunks];
  const bf16* O;                                 // dQ: D is computed from it and written (nullptr: D is there)
};

__device__ __forceinline__ int s_swz(int row) { return S_ROWB == 128 ? ((row >> 1) & 7) : row_code(row); }
__device__ __forceinline__ int s_off(int row, int granule) {
  return row * S_ROWB + ((granule ^ s_swz(row)) << 4);
}
// DMA of `rows8` groups of 8 tile rows: one wave-wide load moves 8 rows (1024 bytes); lane i
// fills LDS slot i & 7 of row i >> 3 of the group and asks for the granule that belongs there.
// (pitch: bytes between rows of the tensor in HBM; granules past the head dimension are asked for
// 2 GiB further on, which no buffer of a padded call reaches: launchers check its span)
__device__ __forceinline__ int s_dma_off(int group, int lane, unsigned pitch, int d) {
  const int row = group * S_RPL + lane / S_GPR, granule = (lane % S_GPR) ^ s_swz(row);
  if (S_PAD && granule * 8 >= d) return (int)0x80000000u;
  return (int)(row * pitch + (granule << 4));
}
// bytes a buffer descriptor must cover for `rows` rows `pitch` bytes apart
__device__ __forceinline__ unsigned s_span(int rows, unsigned pitch, int d) {
  return rows > 0 ? (unsigned)(rows - 1) * pitch + (unsigned)(2 * d) : 0u;
}
// addresses of the transposing reads of a 16-row group (see the d = 128 forward kernel): the
// 16-lane group (h, dh) reads rows 8*sx + 4*h + (0..3), columns db*32 + dh*16 + (0..15)
__device__ __forceinline__ void s_taddr(int lane, int (&taddr)[S_DB][2]) {
  const int j16 = lane & 15, dh = (lane >> 4) & 1, h = lane >> 5;
#pragma unroll
  for (int db = 0; db < S_DB; db++)
#pragma unroll
    for (int sx = 0; sx < 2; sx++)
      taddr[db][sx] = s_off(8 * sx + 4 * h + (j16 >> 2), db * 4 + 2 * dh + ((j16 & 3) >> 1)) + (j16 & 1) * 8;
}
__device__ __forceinline__ bf16x8 s_load8(const bf16* p, bool ok) {
  bf16x8 z;
#pragma unroll
  for (int t = 0; t < 8; t++) z[t] = (bf16)0.0f;
  return ok ? *reinterpret_cast<const bf16x8*>(p) : z;
}
// A pair of probabilities (or dS) as bf16 operands of the second products: S_TERMS terms that add up to
// the fp32 values, in elements t and t + 1 of the fragments.  One term where the inputs' 8 bits are the measure of a
// probability as well (d = 64, 128, as in the hand-scheduled kernels).  The padded builds serve calls that had
// fp32 probabilities in the generic kernels and keep all 24 bits: three terms, each remainder exact, three
// MFMAs.  32 heads of 777 causal rows, d = 96, call with gradients: 80 us with one term, 114 us with three (121 us with
// s_units and the check of burst_rows.h; 1375 us on the generic kernels); a walk's dV differs from 64 bits by 1.6e-3 with one term, 5.7e-7 with three (5.8e-7
// on the generic kernels).
constexpr int S_TERMS = S_PAD ? 3 : 1;
// Units of scores, maxima and lse: log2 (one fma per exponent), or natural in the padded builds, where s x scale is rounded
// before the maximum or lse is taken from it, as in the forward that made them: a row's largest key has exponent 0 exactly,
// however large its score.  (In log2 units the product with log2 e rounds once more: at scores of 2^20 a
// probability of 1 is up to 4 % off, and from 2^31 on it comes out as 0 or infinity.)
__device__ __forceinline__ float s_units(float s, float scale, float c) { return S_PAD ? product(s, scale) : s * c; }
__device__ __forceinline__ float s_exp(float s, float scale, float c, float nref) {   // nref: minus the reference in these units
  return S_PAD ? fast_exp2(above(s, scale, -nref) * kLog2e) : fast_exp2(__builtin_fmaf(s, c, nref));
}
__device__ __forceinline__ float s_raise(float& m_st, float& cm, float mx, float l) {
  return S_PAD ? raise_reference_natural(m_st, cm, mx, l) : raise_reference(m_st, cm, mx, l);
}
// DOT: remainders by dot products instead of a shift or mask and a subtraction (all but the dense 128-wide forward, 86 / 89 us at 32 x 2048
// causal rows: its vector unit is not what bounds it).
template <bool DOT = true>
__device__ __forceinline__ void s_terms(bf16x8 (&out)[S_TERMS], int t, float x, float y) {
  unsigned c1 = 0x0000bf80u, c2 = 0xbf800000u;     // (-1, 0) and (0, -1), in registers: as an inline constant -1.0 has no packed meaning to rely on
  asm("" : "+s"(c1), "+s"(c2));
  const bf16x2 first = __builtin_bit_cast(bf16x2, c1), second = __builtin_bit_cast(bf16x2, c2);
#pragma unroll
  for (int i = 0; i < S_TERMS; i++) {
    bf16x2 pk;
    pk[0] = (bf16)x; pk[1] = (bf16)y;
    out[i][t] = pk[0]; out[i][t + 1] = pk[1];
    if (!DOT) {
      x -= (float)pk[0]; y -= (float)pk[1];
    } else if (i + 1 < S_TERMS) {                  // x - pk[0], y - pk[1]: one instruction each, exact (below 2^-126 nothing, as by subtraction)
      x = __builtin_amdgcn_fdot2_f32_bf16(pk, first, x, false);
      y = __builtin_amdgcn_fdot2_f32_bf16(pk, second, y, false);
    }
  }
}
// acc += a x (the sum of b's terms) and acc += (the sum of a's terms) x b, the smallest terms first
__device__ __forceinline__ f32x16 s_mfma_terms_b(bf16x8 a, const bf16x8 (&b)[S_TERMS], f32x16 acc) {
#pragma unroll
  for (int i = S_TERMS - 1; i >= 0; i--) acc = mfma32(a, b[i], acc);
  return acc;
}
__device__ __forceinline__ f32x16 s_mfma_terms_a(const bf16x8 (&a)[S_TERMS], bf16x8 b, f32x16 acc) {
#pragma unroll
  for (int i = S_TERMS - 1; i >= 0; i--) acc = mfma32(a[i], b, acc);
  return acc;
}
// Calls with block flags (paper Sec. 2.6) run the SPARSE instantiations: wavefront 0 first writes
// the list of tiles that at least one wavefront of the workgroup can see into LDS (tile index plus
// one bit per wavefront, list[0] = count), the loop then walks that list, and a wavefront whose bit
// is clear skips the tile.  A walk over several chunks writes a list per chunk when it gets there: all
// wavefronts have then read the last entry of the one before.
constexpr int S_MAX_LIST = 4096;                  // entries; longer masked calls take the generic kernels
template <typename F>
__device__ __forceinline__ int s_build_list(int* list, int w, int lane, int t_lo, int t_hi, F bits_of) {
  __syncthreads();                                // (the count of the list before may still be on its way)
  if (w == 0) {
    int n = 0;
    for (int base = t_lo; base < t_hi; base += 64) {
      const int t = base + lane;
      int bits = 0;
      if (t < t_hi) bits = bits_of(t);
      const unsigned long long bal = __builtin_amdgcn_ballot_w64(bits != 0);
      if (bits != 0) {
        const int pos = n + __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
        list[1 + pos] = t | (bits << 20);
      }
      n += __builtin_popcountll(bal);
    }
    if (lane == 0) list[0] = n;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(list[0]);
}

// ------------------------------------------------------------------------------- forward
// NW wavefronts of 32 query rows per workgroup.  Four; two for block flags 64 wide (SPARSE), whose lists of visible tiles
// then hold what the workgroup's 64 rows see and nothing else, so that no wavefront waits for another's tiles.  Such a
// workgroup takes 32 keys a tile instead of 64, so that as many wavefronts share a CU's LDS.
constexpr int sf_keys(int NW) { return NW == 2 ? 32 : 64; }
// KG = 2: the four wavefronts are two row blocks times two halves of every tile's keys; the halves' states meet in LDS at the
// end.  Half the rows a workgroup make twice the workgroups, and each wavefront walks half as many scores: a causal call that fits the
// chip once is bound by its longest wavefronts, alone on their SIMDs, whose vector and matrix work do not overlap.  32 heads of
// 777 causal rows, d = 96: 31 -> 23 us (dQ 37 -> 24); 32 of 1000, d = 64: 21 -> 15 (27 -> 18).  Rule and more sizes: walk_rows.
template <bool SPARSE, int NW, int KG>
__global__ void __launch_bounds__(64 * NW, 2)     // (second figure: wavefronts per SIMD)
burst_fwd_d64_kernel(FwdArgsLite a) {
  constexpr int RW = NW / KG, SF_BR = 32 * RW;    // row blocks, query rows per workgroup
  constexpr int SF_BC = sf_keys(NW), SF_TILE = SF_BC * S_ROWB;   // keys per tile
  constexpr int KB = SF_BC / 32 / KG;             // 32-key blocks of a wavefront's share of a tile
  __shared__ __attribute__((aligned(16))) char smem[4 * SF_TILE];   // K[2], V[2]
  extern __shared__ int s_list[];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, lr = lane & 31, h = lane >> 5;
  const int d = S_PAD ? a.d : S_D;
  int head, qb, split = 0;
  if (!locate_block(blockIdx.x, a.H, a.blocks_per_head * a.splits, head, qb, a.order)) return;
  if (a.splits > 1) { split = qb % a.splits; qb /= a.splits; }
  if (a.causal) qb = a.blocks_per_head - 1 - qb;   // later blocks see more keys: the long ones start first
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int rw = KG == 1 ? wu : wu % RW, koff = KG == 1 ? 0 : wu / RW * (32 * KB);   // row block; first key of the share
  const int q0 = qb * SF_BR + (KG == 1 ? w : rw) * 32, row = q0 + lr;
  const int kvhead = head / a.group;
  const unsigned lds0 = lds_addr(smem);

  // The chunks' visible tiles (or list entries) form one sequence, walked with the next tile in flight across the
  // chunk boundaries.  splits > 1: this workgroup takes one of that many runs of it, of equal length.
  constexpr int NL = SF_BC / S_RPL / NW;          // wave-wide loads per wavefront and tile
  auto tiles_of = [&](const Chunk& C, int& lo, int& hi) __attribute__((always_inline)) {   // that some row of the workgroup sees
    lo = 0; hi = (C.Nc + SF_BC - 1) / SF_BC;
    if (a.window > 0) {                            // keys before the window of the first row
      const long long first = a.q_off + (long long)qb * SF_BR - a.window + 1 - C.k_off;
      if (first >= C.Nc) lo = hi;
      else if (first > 0) lo = (int)(first / SF_BC);
    }
    if (a.causal) {                                // keys after the last row
      const long long last = a.q_off + min(qb * SF_BR + SF_BR, a.Nq) - 1 - C.k_off;
      if (last < 0) hi = lo;
      else if (last / SF_BC + 1 < hi) hi = (int)(last / SF_BC) + 1;
    }
    hi = max(hi, lo);
  };
  int c = -1, ft = 0, lo = 0, hi = 0;             // chunk, position in it, first and end position
  int left = 0x7fffffff;                          // tiles of the run from the one that `advance` finds next
  if constexpr (!SPARSE)
    if (a.splits > 1) {
      int all = 0;
      for (int i = 0; i < a.n; i++) {
        tiles_of(a.ch[i], lo, hi);
        all += hi - lo;
      }
      lo = hi = 0;
      ft = all * split / a.splits;                 // (at most 512 runs of 32 x 2^16 tiles)
      left = all * (split + 1) / a.splits - ft;
    }
  int f_tile = 0, f_bits = 0xf, f_Nc = 0;         // the tile that was fetched last
  long long f_koff = 0;
  bool f_first = false;                           // ... is the first one of its chunk
  unsigned ktile = 0;
  int goff[NL];
  __amdgpu_buffer_rsrc_t krs = make_rsrc(nullptr, 0), vrs = krs;
  auto advance = [&](int step) __attribute__((always_inline)) {
    if (--left < 0) return false;
    ft += step;
    while (ft >= hi) {
      const int past = ft - hi;
      if (++c >= a.n) return false;
      const Chunk& C = a.ch[c];
      f_Nc = C.Nc; f_koff = C.k_off;
      tiles_of(C, lo, hi);
      if (hi > lo) {
        const unsigned kpitch = (unsigned)C.ks_r * 2u;           // bytes between key rows
        const size_t base = C.kv_base(kvhead, a.lay.kv_heads);
        krs = make_rsrc((const bf16*)C.K + base, s_span(f_Nc, kpitch, d));
        vrs = make_rsrc((const bf16*)C.V + base, s_span(f_Nc, kpitch, d));
        ktile = kpitch * SF_BC;
#pragma unroll
        for (int il = 0; il < NL; il++) goff[il] = s_dma_off(w * NL + il, lane, kpitch, d);
        if constexpr (SPARSE) {
          const uint8_t* const bm = C.bmask + (size_t)head * C.bhstride;
          hi = s_build_list(s_list, w, lane, lo, hi, [&](int t) {
            int bits = 0;
#pragma unroll
            for (int ww = 0; ww < NW; ww++) {
              const int row0 = qb * SF_BR + ww * 32;
              if (row0 < a.Nq && bm[(size_t)(row0 / a.bsize) * C.bpitch + (t * SF_BC) / a.bsize] != 0) bits |= 1 << ww;
            }
            return bits;
          });
          lo = 0;
        }
      }
      ft = lo + past;
    }
    f_first = ft == lo;
    f_tile = ft;
    if constexpr (SPARSE) {
      const int e = __builtin_amdgcn_readfirstlane(s_list[1 + ft]);
      f_tile = e & 0xfffff;
      f_bits = e >> 20;
    }
    return true;
  };
  auto fetch = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int il = 0; il < NL; il++) {
      dma_b128_to_lds(krs, lds0 + buf * SF_TILE + (unsigned)(wu * NL + il) * 1024u, (int)((unsigned)f_tile * ktile) + goff[il]);
      dma_b128_to_lds(vrs, lds0 + (2 + buf) * SF_TILE + (unsigned)(wu * NL + il) * 1024u, (int)((unsigned)f_tile * ktile) + goff[il]);
    }
  };
  bool have = advance(0);
  // nothing visible: the state stays as it is, unless this launch has to produce it
  if (!have && !a.fresh && a.O_out == nullptr) return;
  if (have) fetch(0);

  bf16x8 qf[S_KS];
  const bf16* Qh = a.Q + a.lay.q_base(head);
#pragma unroll
  for (int ks = 0; ks < S_KS; ks++) qf[ks] = s_load8(Qh + (size_t)row * a.lay.qs_r + ks * 16 + h * 8, row < a.Nq && (!S_PAD || ks * 16 + h * 8 < d));
  // The state in registers: O^T accumulators, reference maximum (m_st as it is stored, cm the chunk's: see
  // raise_reference), and the row sum over this lane's keys.
  const size_t srow = (size_t)head * a.Nq + (row < a.Nq ? row : 0);
  f32x16 o[S_DB];
#pragma unroll
  for (int db = 0; db < S_DB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[db][r] = 0.f;
  float m_st = BURST_NEG_INF, cm = BURST_NEG_INF, lsum = 0.f;
  if (!a.fresh && row < a.Nq) {
    m_st = a.m[srow];
    if (m_st != BURST_NEG_INF) {                   // (a row that has seen nothing may hold anything)
      if (h == 0) lsum = a.l[srow];
      const float* orow = a.O_acc + srow * d;
#pragma unroll
      for (int db = 0; db < S_DB; db++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) {
          if (S_PAD && db * 32 + 8 * q4 >= d) continue;
          const f32x4 v = *reinterpret_cast<const f32x4*>(orow + db * 32 + 8 * q4 + 4 * h);
#pragma unroll
          for (int b = 0; b < 4; b++) o[db][4 * q4 + b] = v[b];
        }
    }
  }
  // A new chunk: what a store of the state and a load by the next launch do to it (to the row sum; m_st comes back
  // as it was), so that a walk gives the same bits whether its chunks come in one launch or one by one.
  auto settle = [&]() __attribute__((always_inline)) {
    const float both = sum_both_halves(lsum);
    lsum = h == 0 ? both : 0.f;
    cm = BURST_NEG_INF;
  };

  int kaddr[S_KS], taddr[S_DB][2];
#pragma unroll
  for (int ks = 0; ks < S_KS; ks++) kaddr[ks] = s_off(lr, 2 * ks + h);
  s_taddr(lane, taddr);
  const long long wave_first_q = a.q_off + qb * SF_BR + rw * 32, wave_last_q = wave_first_q + 31;   // (scalar)
  bf16x2 ones;
  ones[0] = (bf16)1.0f; ones[1] = (bf16)1.0f;

  // The scores of a wavefront's share of a tile (from key `first` on), masked, and the row's maximum of them (see s_units).
  auto scores = [&](const char* kl, int first, int Nc, long long k_off, f32x16 (&s)[KB]) __attribute__((always_inline)) {
    // S^T = K Q^T: register r of key block kb = key first + kb*32 + 8*(r/4) + 4h + r%4
#pragma unroll
    for (int kb = 0; kb < KB; kb++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[kb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < S_KS; ks++)
#pragma unroll
      for (int kb = 0; kb < KB; kb++)
        s[kb] = mfma32(lds_read_b128(kl, kb * 32 * S_ROWB + kaddr[ks]), qf[ks], s[kb]);
    const long long tile_first_k = k_off + first;
    const bool need_mask = ((a.causal != 0) & (tile_first_k + 32 * KB - 1 > wave_first_q)) |   // (no short circuits: one branch)
                           ((a.window > 0) & (tile_first_k < wave_last_q - a.window + 1)) | (first + 32 * KB > Nc);
    if (need_mask) {
      const long long dd = (a.q_off - k_off) + (q0 + lr) - ((long long)first + 4 * h);
      const int tail = Nc - 1 - (first + 4 * h);
      int lim = a.causal ? (int)(dd < -1 ? -1 : (dd > 64 ? 64 : dd)) : 64;
      lim = lim < tail ? lim : tail;
      const long long dl = dd - a.window + 1;
      const int lim_lo = a.window > 0 ? (int)(dl < -1 ? -1 : (dl > 64 ? 64 : dl)) : -1;
#pragma unroll
      for (int kb = 0; kb < KB; kb++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int cpart = kb * 32 + 8 * (r >> 2) + (r & 3);
          if (!(cpart <= lim && cpart >= lim_lo)) s[kb][r] = BURST_NEG_INF;
        }
    }
    float v = s[0][0];
#pragma unroll
    for (int kb = 0; kb < KB; kb++)
#pragma unroll
      for (int r = 0; r < 16; r++) v = fmaxf(v, s[kb][r]);
    return s_units(max_both_halves(v), a.scale, a.c);
  };
  bool begun = false, unset = true;                // unset: some row has no reference in this chunk yet (KG > 1)
  // A run that begins inside a chunk takes the chunk's references from its first tile like every other run (one more
  // K tile and its scores per run).
  if constexpr (!SPARSE)
    if (have && !f_first) {
#pragma unroll
      for (int il = 0; il < NL; il++)
        dma_b128_to_lds(krs, lds0 + SF_TILE + (unsigned)(wu * NL + il) * 1024u, (int)((unsigned)lo * ktile) + goff[il]);
      __builtin_amdgcn_s_waitcnt(0x0070);          // vmcnt(0), lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      f32x16 s[KB];
      float mx = scores(smem + SF_TILE, lo * SF_BC, f_Nc, f_koff, s);
      if constexpr (KG > 1) mx = fmaxf(mx, scores(smem + SF_TILE + 32 * KB * S_ROWB, lo * SF_BC + 32 * KB, f_Nc, f_koff, s));
      s_raise(m_st, cm, mx, 0.f);
      if constexpr (KG > 1) unset = __builtin_amdgcn_ballot_w64(row < a.Nq && cm == BURST_NEG_INF) != 0;
    }
  for (int buf = 0; have; buf ^= 1) {
    const int kt = f_tile, Nc = f_Nc;
    const long long k_off = f_koff;
    const bool mine = ((f_bits >> wu) & 1) != 0, first = f_first;
    __builtin_amdgcn_s_waitcnt(0x0070);            // vmcnt(0), lgkmcnt(0): the tile landed, reads of the one before are done
    __builtin_amdgcn_s_barrier();
    have = advance(1);
    if (have) fetch(buf ^ 1);
    if (first && begun) {
      settle();
      unset = true;
    }
    begun = true;
    if (!mine) continue;                           // block flags hide the tile from this wavefront's rows
    const char* kl = smem + buf * SF_TILE + koff * S_ROWB;
    const char* vl = smem + (2 + buf) * SF_TILE + koff * S_ROWB;
    f32x16 s[KB];
    float mx = scores(kl, kt * SF_BC + koff, Nc, k_off, s);
    // A row's first reference in a chunk is its maximum in the whole tile: its probabilities then do not depend on the groups
    // (under a window they do on the workgroup's rows, which its first tile follows).
    if (KG > 1 && unset) {
      const int other = koff ^ (32 * KB);
      f32x16 t[KB];
      const float m2 = scores(smem + buf * SF_TILE + other * S_ROWB, kt * SF_BC + other, Nc, k_off, t);
      mx = cm == BURST_NEG_INF ? fmaxf(mx, m2) : mx;
      unset = __builtin_amdgcn_ballot_w64(row < a.Nq && fmaxf(mx, cm) == BURST_NEG_INF) != 0;
    }
    if (__builtin_amdgcn_ballot_w64(mx > cm + S_LAZY) != 0) {   // a chunk's first reference, or raised (rare)
      const float alpha = s_raise(m_st, cm, mx, sum_both_halves(lsum));
      lsum *= alpha;
#pragma unroll
      for (int db = 0; db < S_DB; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[db][r] *= alpha;
    }
    const float nref = (m_st == BURST_NEG_INF) ? 0.f : S_PAD ? -m_st : -(m_st * kLog2e);
    bf16x8 pf[2 * KB][S_TERMS];                       // P^T fragments per 16-key group
#pragma unroll
    for (int kg = 0; kg < 2 * KB; kg++)
#pragma unroll
      for (int t = 0; t < 8; t += 2) {
        const int kb = kg >> 1, r = 8 * (kg & 1) + t;
        const float p0 = s_exp(s[kb][r], a.scale, a.c, nref), p1 = s_exp(s[kb][r + 1], a.scale, a.c, nref);
        s_terms<SPARSE || S_D <= 96>(pf[kg], t, p0, p1);
        if constexpr (S_TERMS == 1) {                // sums what the MFMA multiplies
          bf16x2 pk;
          pk[0] = pf[kg][0][t]; pk[1] = pf[kg][0][t + 1];
          lsum = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, lsum, false);
        } else {
          lsum += p0 + p1;
        }
      }
    // O^T += V^T P^T
#pragma unroll
    for (int kg = 0; kg < 2 * KB; kg++)
#pragma unroll
      for (int db = 0; db < S_DB; db++) {
        const bf16x4 va = lds_read_tr(vl, kg * 16 * S_ROWB + taddr[db][0]);
        const bf16x4 vb = lds_read_tr(vl, kg * 16 * S_ROWB + taddr[db][1]);
        o[db] = s_mfma_terms_b(cat4(va, vb), pf[kg], o[db]);
      }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);

  float l_all = sum_both_halves(lsum);
  if constexpr (KG > 1) {                          // [row block][db][q4][lane] O^T, then [row block][m, l][row]
    static_assert(KG == 2 && RW * (128 * S_D + 256) <= 4 * SF_TILE, "the other half's state fits the tiles");
    f32x4* const so = reinterpret_cast<f32x4*>(smem) + rw * S_DB * 4 * 64 + lane;
    float* const ml = reinterpret_cast<float*>(smem) + RW * S_D * 32 + rw * 64 + lr;
    __syncthreads();                               // (all have read the last tile; a barrier that the writes below do not cross)
    if (koff != 0) {
#pragma unroll
      for (int db = 0; db < S_DB; db++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) so[(db * 4 + q4) * 64] = f32x4{o[db][4 * q4], o[db][4 * q4 + 1], o[db][4 * q4 + 2], o[db][4 * q4 + 3]};
      if (h == 0) { ml[0] = m_st; ml[32] = l_all; }
    }
    __syncthreads();
    if (koff != 0) return;
    const float m1 = ml[0], l1 = ml[32], both = fmaxf(m_st, m1), ref = both == BURST_NEG_INF ? 0.f : both;
    // (in the units of the probabilities, and 1 where a half's reference is the larger one)
    const float f0 = fast_exp2(S_PAD ? (m_st - ref) * kLog2e : product(m_st, kLog2e) - product(ref, kLog2e));
    const float f1 = fast_exp2(S_PAD ? (m1 - ref) * kLog2e : product(m1, kLog2e) - product(ref, kLog2e));
    m_st = both;
    l_all = l_all * f0 + l1 * f1;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const f32x4 v = so[(db * 4 + q4) * 64];
#pragma unroll
        for (int b = 0; b < 4; b++) o[db][4 * q4 + b] = o[db][4 * q4 + b] * f0 + v[b] * f1;
      }
  }
  if constexpr (S_PAD) {                           // rows with an infinity or NaN, by themselves (see burst_rows.h)
    unsigned most = larger_of(0, l_all);
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int r = 0; r < 16; r++) most = larger_of(most, o[db][r]);
    const unsigned long long bal = __builtin_amdgcn_ballot_w64(row < a.Nq && most >= kInfBits);
    const unsigned redo = (unsigned)bal | (unsigned)(bal >> 32);
    if (redo != 0) {
      int first = 0, last = 0x7fffffff;
      if (a.splits > 1) {
        int all = 0;
        for (int i = 0; i < a.n; i++) {
          tiles_of(a.ch[i], lo, hi);
          all += hi - lo;
        }
        first = all * split / a.splits;
        last = all * (split + 1) / a.splits;
      }
      for (unsigned left = redo; left != 0;) {
        int rows[kRows];
        const int n = next_rows(left, qb * SF_BR + rw * 32, rows);
        RowState st[kRows];
#pragma unroll
        for (int r = 0; r < kRows; r++) st[r] = row_state(a.fresh, a.O_acc, a.m, a.l, (size_t)head * a.Nq + rows[r], d, lane);
        if constexpr (SF_BC == 64) rows_forward<bf16, true>(st, args_again<FwdArgsLite>(), head, rows, lane, tiles_of, first, last);
        else rows_forward<bf16, true>(st, args_again<FwdArgsLite>(), head, rows, lane, [](const Chunk& C, int& l, int& h) { l = 0; h = (C.Nc + 63) >> 6; }, 0, 0x7fffffff);
#pragma unroll
        for (int r = 0; r < kRows; r++) {
          if (r >= n) continue;
          const size_t sr = (size_t)head * a.Nq + rows[r];
          if (a.splits > 1) {
            const size_t n_rows = (size_t)a.H * a.Nq, pr = (size_t)split * n_rows + sr;
            float* const ml = a.part + (size_t)a.splits * n_rows * d;
            row_gradient<bf16>(a.part, pr * d, st[r].o, 1.f, 0, 0, lane, d);
            if (lane == 0) { ml[pr] = st[r].m; ml[(size_t)a.splits * n_rows + pr] = st[r].l; }
          } else {
            row_store<bf16>(st[r], a.fresh, a.O_acc, a.m, a.l, a.O_out == nullptr ? nullptr : a.O_out + a.lay.q_base(head) + (size_t)rows[r] * a.lay.qs_r,
                            a.lse, sr, d, lane);
          }
        }
      }
      if ((redo >> lr) & 1) return;
    }
  }
  if (row >= a.Nq) return;
  // lane (lr, h) holds row lr, columns db*32 + 8*q4 + 4h + (0..3)
  if (a.splits > 1) {                              // a partial state: [split][rows][d] O, then m (units: s_units) and l
    const size_t rows = (size_t)a.H * a.Nq, pr = (size_t)split * rows + srow;
    float* const prow = a.part + pr * d;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        if (S_PAD && db * 32 + 8 * q4 >= d) continue;
        f32x4 v;
#pragma unroll
        for (int b = 0; b < 4; b++) v[b] = o[db][4 * q4 + b];
        *reinterpret_cast<f32x4*>(prow + db * 32 + 8 * q4 + 4 * h) = v;
      }
    if (h == 0) {
      float* const ml = a.part + (size_t)a.splits * rows * d;
      ml[pr] = S_PAD ? m_st : m_st * kLog2e;
      ml[(size_t)a.splits * rows + pr] = l_all;
    }
    return;
  }
  if (a.O_acc != nullptr && (a.fresh || m_st != BURST_NEG_INF)) {   // rows that never saw a key keep their state
    float* const orow = a.O_acc + srow * d;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        if (S_PAD && db * 32 + 8 * q4 >= d) continue;
        f32x4 v;
#pragma unroll
        for (int b = 0; b < 4; b++) v[b] = o[db][4 * q4 + b];
        *reinterpret_cast<f32x4*>(orow + db * 32 + 8 * q4 + 4 * h) = v;
      }
    if (h == 0) { a.m[srow] = m_st; a.l[srow] = l_all; }
  }
  if (a.O_out != nullptr) {                        // Alg. 1, last two steps
    const float inv = l_all > 0.f ? 1.0f / l_all : 0.f;
    bf16* const out = a.O_out + a.lay.q_base(head) + (size_t)row * a.lay.qs_r;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        if (S_PAD && db * 32 + 8 * q4 >= d) continue;
        bf16x4 v;
#pragma unroll
        for (int b = 0; b < 4; b++) v[b] = (bf16)(l_all > 0.f ? o[db][4 * q4 + b] * inv : 0.f);
        *reinterpret_cast<bf16x4*>(out + db * 32 + 8 * q4 + 4 * h) = v;
      }
    if (h == 0) a.lse[srow] = l_all > 0.f ? m_st + __logf(l_all) : BURST_NEG_INF;
  }
}

// ------------------------------------------------------------------------------- backward, dQ
// Builds whose dQ kernel can compute D.  (At d = 128 the host never asks for it, and the branch alone cost 3 % of walks of few
// rows: 52 rows x 6656 keys, window 1074, 34.3 / 35.2 us.)
constexpr bool S_SUMS = S_PAD || S_D == 64;
// (d = 64 fits four wavefronts per SIMD; left alone, the compiler takes 136 registers with block flags, which leaves three:
// 32 heads of 4096 x 4096 rows, 64-wide flags at density 0.5: 164 us instead of 147)
// (NW: as in the forward kernel)
template <bool SPARSE, int NW, int KG>
__global__ void __launch_bounds__(64 * NW, S_D == 64 && !S_PAD ? 4 : 2)
burst_bwd_dq_d64_kernel(BwdArgsLite a) {
  constexpr int RW = NW / KG, SQ_BR = 32 * RW;    // row blocks, query rows per workgroup
  constexpr int SQ_BC = 32 * KG, SQ_TILE = SQ_BC * S_ROWB;   // keys per tile, 32 a wavefront
  __shared__ __attribute__((aligned(16))) char smem[4 * SQ_TILE];   // K[2], V[2]
  extern __shared__ int s_list[];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, lr = lane & 31, h = lane >> 5;
  const int d = S_PAD ? a.d : S_D;
  int head, qb, split = 0;
  if (!locate_block(blockIdx.x, a.H, a.blocks_per_head * a.splits, head, qb, a.order)) return;
  if (a.splits > 1) { split = qb % a.splits; qb /= a.splits; }
  if (a.causal) qb = a.blocks_per_head - 1 - qb;   // later blocks see more keys: the long ones start first
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int rw = KG == 1 ? wu : wu % RW, koff = KG == 1 ? 0 : wu / RW * 32;   // row block; first key of the share of a tile
  const int q0 = qb * SQ_BR + (KG == 1 ? w : w % RW) * 32;
  const int row = q0 + lr;
  const bool ok = row < a.Nq;
  const size_t srow = (size_t)head * a.Nq + (ok ? row : 0);
  const int kvhead = head / a.group;
  const unsigned lds0 = lds_addr(smem);

  // The chunks' visible tiles (or list entries) form one sequence, as in the forward kernel.
  constexpr int NL = SQ_BC / S_RPL / NW;          // wave-wide loads per wavefront and tile
  auto tiles_of = [&](const Chunk& C, int& lo, int& hi) __attribute__((always_inline)) {   // that some row of the workgroup sees
    lo = 0; hi = (C.Nc + SQ_BC - 1) / SQ_BC;
    if (a.window > 0) {
      const long long first = a.q_off + (long long)qb * SQ_BR - a.window + 1 - C.k_off;
      if (first >= C.Nc) lo = hi;
      else if (first > 0) lo = (int)(first / SQ_BC);
    }
    if (a.causal) {
      const long long last = a.q_off + min(qb * SQ_BR + SQ_BR, a.Nq) - 1 - C.k_off;
      if (last < 0) hi = lo;
      else if (last / SQ_BC + 1 < hi) hi = (int)(last / SQ_BC) + 1;
    }
    hi = max(hi, lo);
  };
  int c = -1, ft = split, lo = 0, hi = 0;         // chunk, position in it, first and end position
  int f_tile = 0, f_bits = 0xf, f_Nc = 0;         // the tile that was fetched last
  long long f_koff = 0;
  unsigned ktile = 0;
  int goff[NL];
  __amdgpu_buffer_rsrc_t krs = make_rsrc(nullptr, 0), vrs = krs;
  auto advance = [&](int step) __attribute__((always_inline)) {
    ft += step;
    while (ft >= hi) {
      const int past = ft - hi;
      if (++c >= a.n) return false;
      const Chunk& C = a.ch[c];
      f_Nc = C.Nc; f_koff = C.k_off;
      tiles_of(C, lo, hi);
      if (hi > lo) {
        const unsigned kpitch = (unsigned)C.ks_r * 2u;           // bytes between key rows
        const size_t base = C.kv_base(kvhead, a.lay.kv_heads);
        krs = make_rsrc((const bf16*)C.K + base, s_span(f_Nc, kpitch, d));
        vrs = make_rsrc((const bf16*)C.V + base, s_span(f_Nc, kpitch, d));
        ktile = kpitch * SQ_BC;
#pragma unroll
        for (int il = 0; il < NL; il++) goff[il] = s_dma_off(w * NL + il, lane, kpitch, d);
        if constexpr (SPARSE) {
          const uint8_t* const bm = C.bmask + (size_t)head * C.bhstride;
          hi = s_build_list(s_list, w, lane, lo, hi, [&](int t) {
            int bits = 0;
#pragma unroll
            for (int ww = 0; ww < NW; ww++) {
              const int row0 = qb * SQ_BR + ww * 32;
              if (row0 < a.Nq && bm[(size_t)(row0 / a.bsize) * C.bpitch + (t * SQ_BC) / a.bsize] != 0) bits |= 1 << ww;
            }
            return bits;
          });
          lo = 0;
        }
      }
      ft = lo + past;
    }
    f_tile = ft;
    if constexpr (SPARSE) {
      const int e = __builtin_amdgcn_readfirstlane(s_list[1 + ft]);
      f_tile = e & 0xfffff;
      f_bits = e >> 20;
    }
    return true;
  };
  auto fetch = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int il = 0; il < NL; il++) {
      dma_b128_to_lds(krs, lds0 + buf * SQ_TILE + (unsigned)(wu * NL + il) * 1024u, (int)((unsigned)f_tile * ktile) + goff[il]);
      dma_b128_to_lds(vrs, lds0 + (2 + buf) * SQ_TILE + (unsigned)(wu * NL + il) * 1024u, (int)((unsigned)f_tile * ktile) + goff[il]);
    }
  };
  bool have = advance(0);
  if (!have && a.acc_dq && a.splits == 1 && !(S_SUMS && a.O != nullptr)) return;  // nothing visible: nothing to add
  if (have) fetch(0);
  // D of the workgroup's rows, in the order of bwd_prepare_kernel's sums: the same bits.  (Its own launch took 4.5 us of a
  // call with gradients of 64 heads x 1024 rows, d = 64.)
  float Dv = 0.f;
  if (S_SUMS && a.O != nullptr) {
    constexpr int L2 = S_D <= 32 ? 2 : S_D <= 64 ? 4 : 8;   // pairs of 16-byte pieces that bwd_prepare_kernel has lanes for
    const size_t at = a.lay.q_base(head) + (size_t)(ok ? row : 0) * a.lay.qs_r;
    float x[L2];
#pragma unroll
    for (int ks = 0; ks < L2; ks++) {
      x[ks] = 0.f;
      if (ks >= S_KS) continue;
      const bool there = ok && (!S_PAD || ks * 16 + h * 8 < d);
      const bf16x8 g = s_load8(a.dO + at + ks * 16 + h * 8, there), o = s_load8(a.O + at + ks * 16 + h * 8, there);
#pragma unroll
      for (int t = 0; t < 8; t++) x[ks] = fma_in_order((float)o[t], (float)g[t], x[ks]);
    }
#pragma unroll
    for (int off = L2 / 2; off > 0; off >>= 1)
#pragma unroll
      for (int ks = 0; ks < off; ks++) x[ks] = add_in_order(x[ks], x[ks + off]);
    Dv = sum_both_halves(x[0]);
    if (ok && h == 0 && koff == 0) const_cast<float*>(a.D)[srow] = Dv;   // (the fall-back below reads it again)
  } else if (ok) {
    Dv = a.D[srow];
  }

  // The accumulators start at the dQ that is there: scale is folded into the exponent below
  // (dS^T comes out as scale * dS^T), so they hold dQ itself and a walk gives the same bits whether its
  // chunks come in one launch or one by one.
  f32x16 dq[S_DB];
#pragma unroll
  for (int db = 0; db < S_DB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) dq[db][r] = 0.f;
  if (a.acc_dq && a.splits == 1 && ok && koff == 0) {
    const float* const orow = (const float*)a.dQ + srow * d;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        if (S_PAD && db * 32 + 8 * q4 >= d) continue;
        const f32x4 v = *reinterpret_cast<const f32x4*>(orow + db * 32 + 8 * q4 + 4 * h);
#pragma unroll
        for (int b = 0; b < 4; b++) dq[db][4 * q4 + b] = v[b];
      }
  }

  if (have) {                                      // (uniform over the workgroup)
    bf16x8 qf[S_KS], gf[S_KS];
#pragma unroll
    for (int ks = 0; ks < S_KS; ks++) {
      const size_t qrow = a.lay.q_base(head) + (size_t)(ok ? row : 0) * a.lay.qs_r;
      const bool there = ok && (!S_PAD || ks * 16 + h * 8 < d);
      qf[ks] = s_load8(a.Q + qrow + ks * 16 + h * 8, there);
      gf[ks] = s_load8(a.dO + qrow + ks * 16 + h * 8, there);
    }
    const float lv = ok ? a.lse[srow] : BURST_NEG_INF;
    // exponent offset: P scaled by `scale`; -inf: P = 0
    const float nlse2 = (lv == BURST_NEG_INF) ? BURST_NEG_INF : S_PAD ? -lv : __builtin_fmaf(-lv, kLog2e, a.log2_scale);
    auto scaled_p = [&](float x) __attribute__((always_inline)) {
      return S_PAD ? fast_exp2(__builtin_fmaf(above(x, a.scale, -nlse2), kLog2e, a.log2_scale)) : fast_exp2(__builtin_fmaf(x, a.c, nlse2));
    };
    int kaddr[S_KS], taddr[S_DB][2];
#pragma unroll
    for (int ks = 0; ks < S_KS; ks++) kaddr[ks] = s_off(lr, 2 * ks + h);
    s_taddr(lane, taddr);
    const long long wave_first_q = a.q_off + q0;

    for (int buf = 0; have; buf ^= 1) {
      const int kt = f_tile, Nc = f_Nc;
      const long long k_off = f_koff;
      const bool mine = ((f_bits >> wu) & 1) != 0;
      __builtin_amdgcn_s_waitcnt(0x0070);
      __builtin_amdgcn_s_barrier();
      have = advance(a.splits);
      if (have) fetch(buf ^ 1);
      if (!mine) continue;                         // block flags hide the tile from this wavefront's rows
      const char* kl = smem + buf * SQ_TILE + koff * S_ROWB;
      const char* vl = smem + (2 + buf) * SQ_TILE + koff * S_ROWB;
      const int first = kt * SQ_BC + koff;
      // S^T = K Q^T, dP^T = V dO^T: register r = key first + 8*(r/4) + 4h + r%4
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < S_KS; ks++) {
        s = mfma32(lds_read_b128(kl, kaddr[ks]), qf[ks], s);
        dp = mfma32(lds_read_b128(vl, kaddr[ks]), gf[ks], dp);
      }
      const long long tile_first_k = k_off + first;
      const bool need_mask = ((a.causal != 0) & (tile_first_k + 31 > wave_first_q)) |
                             ((a.window > 0) & (tile_first_k < wave_first_q + 31 - a.window + 1)) | (first + 32 > Nc);
      if (need_mask) {
        const long long dd = (a.q_off - k_off) + (q0 + lr) - ((long long)first + 4 * h);
        const int tail = Nc - 1 - (first + 4 * h);
        int lim = a.causal ? (int)(dd < -1 ? -1 : (dd > 64 ? 64 : dd)) : 64;
        lim = lim < tail ? lim : tail;
        const long long dl = dd - a.window + 1;
        const int lim_lo = a.window > 0 ? (int)(dl < -1 ? -1 : (dl > 64 ? 64 : dl)) : -1;
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int cpart = 8 * (r >> 2) + (r & 3);
          if (!(cpart <= lim && cpart >= lim_lo)) s[r] = BURST_NEG_INF;
        }
      }
      bf16x8 dsf[2][S_TERMS];                      // dS^T fragments per 16-key group
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const float p0 = scaled_p(s[r]), p1 = scaled_p(s[r + 1]);
        s_terms(dsf[r >> 3], r & 7, p0 * (dp[r] - Dv), p1 * (dp[r + 1] - Dv));
      }
      // dQ^T += K^T dS^T
#pragma unroll
      for (int kg = 0; kg < 2; kg++)
#pragma unroll
        for (int db = 0; db < S_DB; db++) {
          const bf16x4 ta = lds_read_tr(kl, kg * 16 * S_ROWB + taddr[db][0]);
          const bf16x4 tb = lds_read_tr(kl, kg * 16 * S_ROWB + taddr[db][1]);
          dq[db] = s_mfma_terms_b(cat4(ta, tb), dsf[kg], dq[db]);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
  }
  if constexpr (KG > 1) {                          // the halves' sums meet, as in the forward kernel
    static_assert(KG == 2 && RW * 128 * S_D <= 4 * SQ_TILE, "the other half's sums fit the tiles");
    f32x4* const so = reinterpret_cast<f32x4*>(smem) + rw * S_DB * 4 * 64 + lane;
    __syncthreads();                               // (all have read the last tile; a barrier that the writes below do not cross)
    if (koff != 0) {
#pragma unroll
      for (int db = 0; db < S_DB; db++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) so[(db * 4 + q4) * 64] = f32x4{dq[db][4 * q4], dq[db][4 * q4 + 1], dq[db][4 * q4 + 2], dq[db][4 * q4 + 3]};
    }
    __syncthreads();
    if (koff != 0) return;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const f32x4 v = so[(db * 4 + q4) * 64];
#pragma unroll
        for (int b = 0; b < 4; b++) dq[db][4 * q4 + b] += v[b];
      }
  }
  if constexpr (S_PAD) {                           // rows with an infinity or NaN, by themselves (see burst_rows.h)
    unsigned most = 0;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int r = 0; r < 16; r++) most = larger_of(most, dq[db][r]);
    const unsigned long long bal = __builtin_amdgcn_ballot_w64(ok && most >= kInfBits);
    const unsigned redo = (unsigned)bal | (unsigned)(bal >> 32);
    for (unsigned left = redo; left != 0;) {
      int rows[kRows];
      const int n = next_rows(left, qb * SQ_BR + rw * 32, rows);
      float g[kRows][2];
      rows_dq<bf16, true, SQ_BC>(g, args_again<BwdArgsLite>(), head, rows, lane, tiles_of, split, a.splits);
#pragma unroll
      for (int r = 0; r < kRows; r++) {
        if (r >= n) continue;
        const size_t at = ((size_t)head * a.Nq + rows[r]) * d;
        if (a.splits > 1) row_gradient<bf16>(a.part, (size_t)split * a.H * a.Nq * d + at, g[r], a.scale, 0, 0, lane, d);
        else row_gradient<bf16>(a.dQ, at, g[r], a.scale, a.half, a.acc_dq, lane, d);
      }
    }
    if ((redo >> lr) & 1) return;
  }
  if (ok && a.half && a.splits == 1) {
    bf16* const orow = (bf16*)a.dQ + srow * d;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        if (S_PAD && db * 32 + 8 * q4 >= d) continue;
        bf16x4 v;
#pragma unroll
        for (int b = 0; b < 4; b++) v[b] = (bf16)dq[db][4 * q4 + b];
        *reinterpret_cast<bf16x4*>(orow + db * 32 + 8 * q4 + 4 * h) = v;
      }
  } else if (ok) {
    float* const orow = a.splits > 1 ? a.part + ((size_t)split * a.H * a.Nq + srow) * d : (float*)a.dQ + srow * d;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        if (S_PAD && db * 32 + 8 * q4 >= d) continue;
        f32x4 v;
#pragma unroll
        for (int b = 0; b < 4; b++) v[b] = dq[db][4 * q4 + b];
        *reinterpret_cast<f32x4*>(orow + db * 32 + 8 * q4 + 4 * h) = v;
      }
  }
}

// ------------------------------------------------------------------------------- backward, dK / dV
// Wavefronts per dK/dV workgroup, 32 keys each.  Four by default.  With two (BURST_SMALL_DKV_WAVES
// = 2: the d = 128 build) a workgroup owns 64 keys, the finest block edge a call's flags can have,
// so its list of visible tiles is exactly the tiles those 64 keys are needed for, and two such
// workgroups share a CU at one wavefront per SIMD (the kernel needs more than 256 registers at
// d = 128).
#ifndef BURST_SMALL_DKV_WAVES
#define BURST_SMALL_DKV_WAVES 4
#endif
constexpr int SK_WAVES = BURST_SMALL_DKV_WAVES;

// PARTS: the walks are cut (RowParts), in an instantiation of its own: as a branch of the ordinary one it cost short walks 1 to 2 %.
// QG = 2: the wavefronts are two key blocks times two halves of every tile's rows; the halves' sums meet in LDS at the end, for the
// reasons of KG in the forward kernel (rule: dkv_parts; 32 heads of 777 causal rows, d = 96: 32 + 10 merging parts -> 34 us).
// NW wavefronts.  Eight (the 128-wide padded build): two per SIMD, a CU's only workgroup, QG = 2.  K and V of its 128 keys lie in
// LDS before the tiles: in registers they and the three terms of P and dS left room for one wavefront per SIMD (382 registers).
// 32 over 8 heads x 3001 causal rows, dK/dV with merging: 422 us so, 363 with eight (five contractions' worth of terms at 0.85 PFLOP/s
// executed); 8 x 2048, d = 120, 133 / 77.  Block flags 64 wide stay with two wavefronts of 64 keys, whose lists are exact (density 0.25, 32 over 8
// x 1000 x 2000 60 / 71; 128 wide 125 / 119, 256 wide 74 / 58).
constexpr int SK_GROUPS = SK_WAVES == 8 ? 2 : 1;  // the build's ordinary QG
constexpr int sk_keys(int NW, int QG) { return 32 * NW / QG; }   // keys per workgroup
constexpr int sk_rows(int QG) { return 32 * QG; }              // query rows per tile
template <bool SPARSE, bool PARTS, int QG, int NW>
__global__ void __launch_bounds__(64 * NW, NW >= 4 ? 2 : 1)   // (second figure: wavefronts per SIMD)
burst_bwd_dkv_d64_kernel(BwdArgsLite a) {
  constexpr bool S_KV_LDS = NW == 8;
  constexpr int KW = NW / QG, SK_BC = sk_keys(NW, QG), SK_BR = sk_rows(QG), SK_TILE = SK_BR * S_ROWB;
  constexpr int SK_Q = S_KV_LDS ? 2 * SK_BC * S_ROWB : 0;   // K, V; then the tiles
  constexpr int SK_STAT = SK_Q + 4 * SK_TILE;     // per buffer and row: -lse (see s_units), then D
  __shared__ __attribute__((aligned(16))) char smem[SK_STAT + 2 * 2 * SK_BR * 4];   // (K, V,) Q[2], dO[2], statistics[2]
  extern __shared__ int s_list[];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, lr = lane & 31, h = lane >> 5;
  const int d = S_PAD ? a.d : S_D;
  // the workgroups of all chunks, chunk after chunk
  const int chunk = chunk_at((int)blockIdx.x, a.ch, a.n, a.per);
  const Chunk& C = a.ch[chunk];
  int kvhead, kblk, part = 0;                      // a.H counts key/value heads here
  const int bid = (int)blockIdx.x - C.first_block, blocks = (C.Nc + SK_BC - 1) / SK_BC;
  if constexpr (PARTS) {
    if (!locate_part(bid, a.H, blocks, a.parts.splits, kvhead, kblk, part)) return;
  } else {
    if (!locate_block(bid, a.H, blocks, kvhead, kblk, C.order)) return;
  }
  const int Nc = C.Nc;
  const long long k_off = C.k_off;
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int kw = QG == 1 ? wu : wu % KW, qoff = QG == 1 ? 0 : wu / KW * 32;   // key block; first row of the share of a tile
  const int key_wg = kblk * SK_BC, key0 = key_wg + (QG == 1 ? w : w % KW) * 32;
  const bf16* Kh = (const bf16*)C.K + C.kv_base(kvhead, a.lay.kv_heads);
  const bf16* Vh = (const bf16*)C.V + C.kv_base(kvhead, a.lay.kv_heads);
  const unsigned qpitch = (unsigned)a.lay.qs_r * 2u;             // bytes between query rows

  // query tiles of one head to visit, then the same range for every head of the group
  const RowRange range = row_range(a.Nq, a.causal, a.window, a.q_off, k_off, Nc, key_wg, SK_BC, SK_BR);
  const int t_begin = range.lo, per_head = range.hi - range.lo;
  int nwalk = per_head * a.group, first = 0, parts = 1;   // this workgroup's tiles begin at position `first` of the walk
  if constexpr (PARTS) {
    parts = a.parts.of(nwalk);
    if (part >= parts) return;
    first = (int)((long long)nwalk * part / parts);
    nwalk = (int)((long long)nwalk * (part + 1) / parts) - first;
  }
  if constexpr (SPARSE) {                          // entries count tiles over all heads of the group
    nwalk = s_build_list(s_list, w, lane, 0, nwalk, [&](int n) {
      const int g = n / (per_head > 0 ? per_head : 1);
      const int t = t_begin + n % (per_head > 0 ? per_head : 1);
      const uint8_t* mrow = C.bmask + (size_t)(kvhead * a.group + g) * C.bhstride + (size_t)((t * SK_BR) / a.bsize) * C.bpitch;
      int bits = 0;
#pragma unroll
      for (int ww = 0; ww < KW; ww++) {
        const int k0 = key_wg + ww * 32;
        if (k0 < Nc && mrow[k0 / a.bsize] != 0) bits |= 1 << ww;
      }
      return bits;
    });
  }
  // walk position -> (query head of the group, tile, this wavefront's bit)
  auto locate = [&](int j, int& g, int& t) __attribute__((always_inline)) {
    int n = first + j, bits = 0xf;
    if constexpr (SPARSE) {
      const int e = __builtin_amdgcn_readfirstlane(s_list[1 + j]);
      n = e & 0xfffff; bits = e >> 20;
    }
    if (a.group == 1) {                            // (no division in the common case: a scalar divide is some forty instructions)
      g = 0;
      t = t_begin + n;
    } else {
      g = n / per_head;
      t = t_begin + (n - g * per_head);
    }
    return bits;
  };

  f32x16 dk[S_DB], dv[S_DB];
#pragma unroll
  for (int db = 0; db < S_DB; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) { dk[db][r] = 0.f; dv[db][r] = 0.f; }

  if (nwalk > 0) {
    bf16x8 kf[S_KS], vf[S_KS];
    if constexpr (!S_KV_LDS)
#pragma unroll
    for (int ks = 0; ks < S_KS; ks++) {
      const bool there = key0 + lr < Nc && (!S_PAD || ks * 16 + h * 8 < d);
      kf[ks] = s_load8(Kh + (size_t)(key0 + lr) * C.ks_r + ks * 16 + h * 8, there);
      vf[ks] = s_load8(Vh + (size_t)(key0 + lr) * C.ks_r + ks * 16 + h * 8, there);
    }
    int qaddr[S_KS], taddr[S_DB][2];
#pragma unroll
    for (int ks = 0; ks < S_KS; ks++) qaddr[ks] = s_off(lr, 2 * ks + h);
    s_taddr(lane, taddr);
    const unsigned lds0 = lds_addr(smem);
    constexpr int NL = SK_BR / S_RPL / NW;  // wave-wide loads per wavefront and tile
    static_assert(NL >= 1 && NL * NW * S_RPL == SK_BR, "a tile's rows must divide evenly among the wavefronts");
    int goff[NL];
#pragma unroll
    for (int il = 0; il < NL; il++) goff[il] = s_dma_off(w * NL + il, lane, qpitch, d);
    float* const stat = reinterpret_cast<float*>(smem + SK_STAT);
    // walk position n -> (query head, tile); every wavefront DMAs its rows of Q and dO.  The
    // first wavefronts also fetch the rows' statistics with plain loads issued BEFORE the
    // DMA (the wait the compiler places before their first use then does not cover the DMA) and
    // writes them to LDS at the end of the step (stat_commit).
    float stat_x = 0.f;
    auto fetch = [&](int n, int buf) __attribute__((always_inline)) {
      int g, t;
      locate(n, g, t);
      const size_t hrow = (size_t)(kvhead * a.group + g) * a.Nq;
      if (tid < 2 * SK_BR) {
        const int r = t * SK_BR + (tid & (SK_BR - 1));
        if (tid < SK_BR) stat_x = r < a.Nq ? a.lse[hrow + r] : BURST_NEG_INF;
        else stat_x = r < a.Nq ? a.D[hrow + r] : 0.f;
      }
      const size_t hbase = a.lay.q_base(kvhead * a.group + g);
      const __amdgpu_buffer_rsrc_t qrs = make_rsrc(a.Q + hbase, s_span(a.Nq, qpitch, d));
      const __amdgpu_buffer_rsrc_t grs = make_rsrc(a.dO + hbase, s_span(a.Nq, qpitch, d));
#pragma unroll
      for (int il = 0; il < NL; il++) {
        dma_b128_to_lds(qrs, lds0 + SK_Q + buf * SK_TILE + (unsigned)(wu * NL + il) * 1024u, (int)(t * SK_BR * qpitch) + goff[il]);
        dma_b128_to_lds(grs, lds0 + SK_Q + (2 + buf) * SK_TILE + (unsigned)(wu * NL + il) * 1024u, (int)(t * SK_BR * qpitch) + goff[il]);
      }
    };
    auto stat_commit = [&](int buf) __attribute__((always_inline)) {
      if (tid < SK_BR) stat[buf * 2 * SK_BR + tid] = (stat_x == BURST_NEG_INF) ? BURST_NEG_INF : S_PAD ? -stat_x : -stat_x * kLog2e;   // -inf: P = 0
      else if (tid < 2 * SK_BR) stat[buf * 2 * SK_BR + tid] = stat_x;
    };
    const long long wave_first_k = k_off + key0, wave_last_k = wave_first_k + 31;
    const long long kpos = wave_first_k + lr;

    if constexpr (S_KV_LDS) {                      // (keys past Nc, columns past d: zero; awaited with the first tile)
      constexpr int LOADS = SK_BC / S_RPL / NW;
      const unsigned kpitch = (unsigned)C.ks_r * 2u;
      const __amdgpu_buffer_rsrc_t krs = make_rsrc(Kh, s_span(Nc, kpitch, d)), vrs = make_rsrc(Vh, s_span(Nc, kpitch, d));
#pragma unroll
      for (int il = 0; il < LOADS; il++) {
        const int off = s_dma_off(w * LOADS + il, lane, kpitch, d), at = S_PAD && off < 0 ? off : (int)((unsigned)key_wg * kpitch) + off;
        dma_b128_to_lds(krs, lds0 + (unsigned)(wu * LOADS + il) * 1024u, at);
        dma_b128_to_lds(vrs, lds0 + SK_BC * S_ROWB + (unsigned)(wu * LOADS + il) * 1024u, at);
      }
    }
    fetch(0, 0);
    stat_commit(0);
    for (int n = 0; n < nwalk; n++) {
      __builtin_amdgcn_s_waitcnt(0x0070);
      __builtin_amdgcn_s_barrier();
      if (n + 1 < nwalk) fetch(n + 1, (n + 1) & 1);
      const int buf = n & 1;
      const char* ql = smem + SK_Q + buf * SK_TILE + qoff * S_ROWB;
      const char* gl = smem + SK_Q + (2 + buf) * SK_TILE + qoff * S_ROWB;
      int g_unused, t;
      const bool mine = ((locate(n, g_unused, t) >> kw) & 1) != 0;
      if (mine) {                                  // (else: block flags hide this wavefront's keys from the tile)
        // S = Q K^T, dP = dO V^T: lane = key lr, register r = row first_row + 8*(r/4) + 4h + r%4
        const int first_row = t * SK_BR + qoff;
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = 0.f; }
        if constexpr (NW == 2) {
          // One wavefront per SIMD: nobody else hides an LDS read's latency, and left alone the
          // compiler reads one fragment, waits, multiplies, sixteen times over.  All sixteen
          // fragments are requested first (the registers are there), then the MFMAs run.
          bf16x8 qa[S_KS], ga[S_KS];
#pragma unroll
          for (int ks = 0; ks < S_KS; ks++) { qa[ks] = lds_read_b128(ql, qaddr[ks]); ga[ks] = lds_read_b128(gl, qaddr[ks]); }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int ks = 0; ks < S_KS; ks++) { s = mfma32(qa[ks], kf[ks], s); dp = mfma32(ga[ks], vf[ks], dp); }
        } else if constexpr (S_KV_LDS) {
          const char* const kl = smem + kw * 32 * S_ROWB;
#pragma unroll
          for (int ks = 0; ks < S_KS; ks++) {
            s = mfma32(lds_read_b128(ql, qaddr[ks]), lds_read_b128(kl, qaddr[ks]), s);
            dp = mfma32(lds_read_b128(gl, qaddr[ks]), lds_read_b128(kl, SK_BC * S_ROWB + qaddr[ks]), dp);
          }
        } else {
#pragma unroll
          for (int ks = 0; ks < S_KS; ks++) {
            s = mfma32(lds_read_b128(ql, qaddr[ks]), kf[ks], s);
            dp = mfma32(lds_read_b128(gl, qaddr[ks]), vf[ks], dp);
          }
        }
        const long long tile_first_q = a.q_off + first_row;
        const bool need_mask = ((a.causal != 0) & (wave_last_k > tile_first_q)) |
                               ((a.window > 0) & (tile_first_q + 31 >= wave_first_k + a.window)) |
                               (S_PAD & (first_row + 32 > a.Nq));   // (rows of zeros, whose product with an infinite key is NaN)
        if (need_mask) {
          // visible iff key position <= row position (constant part >= lim) and row position <
          // key position + window (constant part <= lim2)
          const long long dd = kpos - (tile_first_q + 4 * h);
          const int lim = a.causal ? (int)(dd < -1 ? -1 : (dd > 64 ? 64 : dd)) : -1;
          const long long d2 = dd + a.window - 1;
          int lim2 = a.window > 0 ? (int)(d2 < -1 ? -1 : (d2 > 64 ? 64 : d2)) : 64;
          if (S_PAD) lim2 = min(lim2, a.Nq - 1 - (first_row + 4 * h));
#pragma unroll
          for (int r = 0; r < 16; r++) {
            const int cpart = 8 * (r >> 2) + (r & 3);
            if (!(cpart >= lim && cpart <= lim2)) s[r] = BURST_NEG_INF;
          }
        }
        // (two wavefronts per workgroup: the transposed dO and Q fragments of the last phase are
        // requested here, so that they arrive while the exponentials run)
        bf16x4 tg[2][S_DB][2], tq[2][S_DB][2];
        if constexpr (NW == 2) {
#pragma unroll
          for (int u = 0; u < 2; u++)
#pragma unroll
            for (int db = 0; db < S_DB; db++)
#pragma unroll
              for (int sx = 0; sx < 2; sx++) {
                tg[u][db][sx] = lds_read_tr(gl, u * 16 * S_ROWB + taddr[db][sx]);
                tq[u][db][sx] = lds_read_tr(ql, u * 16 * S_ROWB + taddr[db][sx]);
              }
          __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 pf[2][S_TERMS], dsf[2][S_TERMS];      // per 16-row group: A operands of dV, dK
        auto terms = [&](int u) __attribute__((always_inline)) {
#pragma unroll
          for (int q4 = 2 * u; q4 < 2 * u + 2; q4++) {
            const f32x4 nl = *reinterpret_cast<const f32x4*>(stat + buf * 2 * SK_BR + qoff + 8 * q4 + 4 * h);
            const f32x4 dr = *reinterpret_cast<const f32x4*>(stat + buf * 2 * SK_BR + SK_BR + qoff + 8 * q4 + 4 * h);
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
              const int r = 4 * q4 + j;
              const float p0 = s_exp(s[r], a.scale, a.c, nl[j]), p1 = s_exp(s[r + 1], a.scale, a.c, nl[j + 1]);
              s_terms(pf[u], r & 7, p0, p1);
              s_terms(dsf[u], r & 7, p0 * (dp[r] - dr[j]), p1 * (dp[r + 1] - dr[j + 1]));
            }
          }
        };
        // dV += P^T dO, dK += dS^T Q (dO and Q through transposing reads)
        auto products = [&](int u) __attribute__((always_inline)) {
#pragma unroll
          for (int db = 0; db < S_DB; db++) {
            bf16x8 bg, bq;
            if constexpr (NW == 2) {
              bg = cat4(tg[u][db][0], tg[u][db][1]);
              bq = cat4(tq[u][db][0], tq[u][db][1]);
            } else {
              bg = cat4(lds_read_tr(gl, u * 16 * S_ROWB + taddr[db][0]), lds_read_tr(gl, u * 16 * S_ROWB + taddr[db][1]));
              bq = cat4(lds_read_tr(ql, u * 16 * S_ROWB + taddr[db][0]), lds_read_tr(ql, u * 16 * S_ROWB + taddr[db][1]));
            }
            dv[db] = s_mfma_terms_a(pf[u], bg, dv[db]);
            dk[db] = s_mfma_terms_a(dsf[u], bq, dk[db]);
          }
        };
        terms(0);
        if constexpr (S_KV_LDS) { products(0); terms(1); }           // (fewer registers)
        else { terms(1); products(0); }
        products(1);
      }
      if (n + 1 < nwalk) stat_commit((n + 1) & 1);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    if constexpr (QG > 1) {                        // [key block][dK, dV][db][q4][lane]
      static_assert(QG == 2 && KW * 256 * S_D <= SK_STAT, "the other half's sums fit the tiles");
      f32x4* const so = reinterpret_cast<f32x4*>(smem) + kw * 2 * S_DB * 4 * 64 + lane;
      __syncthreads();                             // (all have read the last tile; a barrier that the writes below do not cross)
      if (qoff != 0) {
#pragma unroll
        for (int db = 0; db < S_DB; db++)
#pragma unroll
          for (int q4 = 0; q4 < 4; q4++) {
            so[(db * 4 + q4) * 64] = f32x4{dk[db][4 * q4], dk[db][4 * q4 + 1], dk[db][4 * q4 + 2], dk[db][4 * q4 + 3]};
            so[((S_DB + db) * 4 + q4) * 64] = f32x4{dv[db][4 * q4], dv[db][4 * q4 + 1], dv[db][4 * q4 + 2], dv[db][4 * q4 + 3]};
          }
      }
      __syncthreads();
      if (qoff == 0) {
#pragma unroll
        for (int db = 0; db < S_DB; db++)
#pragma unroll
          for (int q4 = 0; q4 < 4; q4++) {
            const f32x4 x = so[(db * 4 + q4) * 64], y = so[((S_DB + db) * 4 + q4) * 64];
#pragma unroll
            for (int b = 0; b < 4; b++) { dk[db][4 * q4 + b] += x[b]; dv[db][4 * q4 + b] += y[b]; }
          }
      }
    }
  }
  if (QG > 1 && qoff != 0) return;
  if (PARTS && parts > 1) {                        // (infinities and NaN: merge_dkv_kernel sees to them)
    store_dkv<S_DB, S_PAD>(dk, dv, a.parts.at(part, false, C, kvhead, d), a.parts.at(part, true, C, kvhead, d),
                           C.span_keys, d, key0 - C.span_lo, lr, h, a.scale, 0, 0);
    return;
  }
  if constexpr (S_PAD) {                           // keys with an infinity or NaN, and their neighbours (see burst_rows.h)
    unsigned most = 0;
#pragma unroll
    for (int db = 0; db < S_DB; db++)
#pragma unroll
      for (int r = 0; r < 16; r++) most = larger_of(larger_of(most, dk[db][r]), dv[db][r]);
    if (__builtin_amdgcn_ballot_w64(most >= kInfBits) != 0) {
      const int base = key_wg + kw * 32;
      for (unsigned left = first_bits(Nc - base); left != 0;) {
        int keys[kRows];
        const int n = next_rows(left, base, keys);
        float gk[kRows][2], gv[kRows][2];
        keys_dkv<bf16, true>(gk, gv, args_again<BwdArgsLite>(), C, kvhead, keys, lane);
#pragma unroll
        for (int r = 0; r < kRows; r++) {
          if (r >= n) continue;
          const size_t at = ((size_t)kvhead * Nc + keys[r]) * d;
          row_gradient<bf16>(C.dK, at, gk[r], a.scale, a.half, a.acc_dkv, lane, d);
          row_gradient<bf16>(C.dV, at, gv[r], 1.f, a.half, a.acc_dkv, lane, d);
        }
      }
      return;
    }
  }
  const size_t at = (size_t)kvhead * Nc * d * (a.half ? 2 : 4);
  store_dkv<S_DB, S_PAD>(dk, dv, (char*)C.dK + at, (char*)C.dV + at, Nc, d, key0, lr, h, a.scale, a.half, a.acc_dkv);
}

// ------------------------------------------------------------------------------- launchers
// Tile lists are dynamic LDS behind up to 64 KB of static tiles: the kernels that take one opt
// in to the larger total once per device.
template <typename K>
static int allow_list(K kernel, DeviceOnce& once) {
  return once.run([kernel] {
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (S_MAX_LIST + 4) * 4) ==
                   hipSuccess ? BURST_OK : BURST_ERR_LAUNCH;
  });
}
template <typename A, typename K>
static int launch_plain(K dense, K sparse, DeviceOnce& once, A& a, long long nb, long long entries, int threads, hipStream_t stream) {
  if (nb > 0x7fffffffLL) return BURST_ERR_SHAPE;
  if (nb == 0) return BURST_OK;
  if (a.ch[0].bmask != nullptr) {
    if (entries > S_MAX_LIST) return BURST_ERR_SHAPE;
    if (int st = allow_list(sparse, once); st != BURST_OK) return st;
    BURST_LAUNCH(sparse, dim3((unsigned)nb), dim3(threads), ((unsigned)entries + 4) * 4, stream, a);
  } else {
    BURST_LAUNCH(dense, dim3((unsigned)nb), dim3(threads), 0, stream, a);
  }
  return launch_status();
}

// Wavefronts of a forward or dQ workgroup: two where the flags are 64 wide (see the forward kernel).  32 heads x 4096 rows x
// 8192 keys, four / two, us: dQ, d = 128, density 0.1 166 / 134, 0.25 351 / 280, 0.5 496 / 470; d = 64 171 / 149, 270 / 253
// (0.25, 0.5); forward, d = 64, 141 / 130, 216 / 215.  In the forward at d = 128 the smaller tiles take back what the exact
// lists give (134 / 132, 274 / 266, 389 / 408): two only while all workgroups are resident at once (8 heads x 1000 rows x
// 3000 keys 44 / 35).  Four for at most 64 rows, where both have as many workgroups (8 x 64 rows x 4000 keys, forward, d = 64, 0.25, 18.0 /
// 22.3, d = 120 36 / 40), and in the forward where workgroups of four wavefronts have a CU each and equal work, on the narrow padded builds
// (d = 40, 24 x 900 x 1800, 0.1, 0.25 and 0.5 17.4 / 20.6, 29.1 / 34.8, 42.4 / 55.9) and with at most 2048 keys on the others (d = 64 13.9 / 15.6,
// 21.8 / 23.1, 30.6 / 35.0, d = 128 20.0 / 20.9, 31.2 / 32.2, 43.9 / 49.0; 6000 keys 0.87, 0.98, 1.12 of the time).  Dense flags lose
// whatever the sizes (0.9: forward 3 to 30 %, dQ up to 8 %); the host cannot see them.
static int row_waves(const KParams& p, const Chunk* ch, int n, bool forward) {
  if (ch[0].bmask == nullptr || p.bsize >= 128 || p.Nq <= 64) return 4;
  if (!forward) return 2;
  const long long heads = (long long)p.B * p.H, places = heads * ((p.Nq + 127) / 128);
  long long keys = 0;
  for (int i = 0; i < n; i++) keys += ch[i].Nc;
  if (!p.causal && places > 128 && places <= 256 && ((S_PAD && S_D <= 64) || keys <= 2048)) return 4;
  return S_D <= 64 || heads * ((p.Nq + 63) / 64) <= 1024 ? 2 : 4;
}

// n <= kMaxChunks chunks, all of them with block flags or none.
int launch_fwd(const KParams& p, const FwdIo& io, const Chunk* ch, int n, hipStream_t stream) {
  FwdArgsLite a;
  a.Q = (const bf16*)io.Q;
  a.O_acc = io.O_acc; a.m = io.m; a.l = io.l; a.O_out = (bf16*)io.O_out; a.lse = io.lse;
  a.part = io.part; a.splits = io.splits > 1 ? io.splits : 1;
  a.fresh = io.fresh || a.splits > 1;
  a.Nq = p.Nq; a.H = p.B * p.H; a.group = p.group;
  a.causal = p.causal; a.c = p.scale * kLog2e; a.scale = p.scale;
  a.q_off = p.q_off; a.window = p.window; a.bsize = p.bsize;
  a.lay = p.lay; a.d = p.d; a.n = n;
  const int nw = row_waves(p, ch, n, true), kg = io.groups == 2 && ch[0].bmask == nullptr ? 2 : 1, br = 32 * nw / kg;
  if (kg == 2 && !a.fresh) return BURST_ERR_SHAPE;   // (both groups would start from the state and count it twice)
  a.blocks_per_head = (p.Nq + br - 1) / br;
  a.order = grid_order(a.H, (long long)a.blocks_per_head * a.splits, unequal_rows(p, ch, n, br), kg == 2 && S_ROWB == 128 ? 4 : 2);
  int longest = 0;
  for (int i = 0; i < n; i++) { a.ch[i] = ch[i]; if (ch[i].Nc > longest) longest = ch[i].Nc; }
  static DeviceOnce done, done2;
  return launch_plain(kg == 2 ? burst_fwd_d64_kernel<false, 4, 2> : burst_fwd_d64_kernel<false, 4, 1>,
                      nw == 2 ? burst_fwd_d64_kernel<true, 2, 1> : burst_fwd_d64_kernel<true, 4, 1>, nw == 2 ? done2 : done, a,
                      grid_blocks(a.H, (long long)a.blocks_per_head * a.splits), (longest + sf_keys(nw) - 1) / sf_keys(nw), 64 * nw, stream);
}

static void bwd_args(BwdArgsLite& a, const KParams& p, const BwdIo& io, const Chunk* ch, int n) {
  a.Q = (const bf16*)io.Q; a.dO = (const bf16*)io.dO; a.lse = io.lse; a.D = io.D; a.dQ = io.dQ; a.half = io.half;
  a.part = io.part; a.splits = io.splits > 1 ? io.splits : 1;
  a.Nq = p.Nq; a.H = p.B * p.H; a.group = p.group;
  a.causal = p.causal; a.c = p.scale * kLog2e; a.scale = p.scale; a.log2_scale = log2f(p.scale);
  a.acc_dq = io.acc_dq; a.acc_dkv = io.acc_dkv;
  a.q_off = p.q_off; a.window = p.window; a.bsize = p.bsize;
  a.lay = p.lay; a.d = p.d; a.n = n; a.O = (const bf16*)io.O;
  for (int i = 0; i < n; i++) a.ch[i] = ch[i];
}

int launch_bwd_dq(const KParams& p, const BwdIo& io, const Chunk* ch, int n, hipStream_t stream) {
  BwdArgsLite a;
  bwd_args(a, p, io, ch, n);
  if (io.O != nullptr && !S_SUMS) return BURST_ERR_SHAPE;
  const int nw = row_waves(p, ch, n, false), kg = io.groups == 2 && ch[0].bmask == nullptr ? 2 : 1, br = 32 * nw / kg;
  a.blocks_per_head = (p.Nq + br - 1) / br;
  a.order = grid_order(a.H, (long long)a.blocks_per_head * a.splits, unequal_rows(p, ch, n, br), kg == 2 && S_ROWB == 128 ? 4 : 2);
  int longest = 0;
  for (int i = 0; i < n; i++) if (ch[i].Nc > longest) longest = ch[i].Nc;
  static DeviceOnce done, done2;
  return launch_plain(kg == 2 ? burst_bwd_dq_d64_kernel<false, 4, 2> : burst_bwd_dq_d64_kernel<false, 4, 1>,
                      nw == 2 ? burst_bwd_dq_d64_kernel<true, 2, 1> : burst_bwd_dq_d64_kernel<true, 4, 1>, nw == 2 ? done2 : done, a,
                      grid_blocks(a.H, (long long)a.blocks_per_head * a.splits), (longest + 31) / 32, 64 * nw, stream);
}

// Keys of a dK/dV workgroup, for the host's rule of splitting (two workgroups of 32-row tiles share a CU, one of 64-row tiles).
int dkv_keys() { return sk_keys(SK_WAVES, SK_GROUPS); }
int dkv_rows() { return sk_rows(SK_GROUPS); }      // rows of its tiles

int launch_bwd_dkv(const KParams& p, const BwdIo& io, const Chunk* ch, int n, hipStream_t stream) {
  BwdArgsLite a;
  bwd_args(a, p, io, ch, n);
  a.H = p.B * p.H / p.group;                       // workgroups are laid out over key/value heads
  set_row_parts(a, io);
  constexpr int G = SK_WAVES == 4 ? 2 : SK_GROUPS, FINE = SK_WAVES == 8 ? 2 : SK_WAVES;   // groups of whole walks; wavefronts for flags 64 wide
  const bool flags = ch[0].bmask != nullptr, fine = flags && p.bsize < 128;
  const int nw = fine ? FINE : SK_WAVES;
  const int groups = nw == 2 ? 1 : io.parts != nullptr && io.parts->groups == 2 && a.parts.splits == 1 && !flags ? G : SK_GROUPS, bc = sk_keys(nw, groups);
  const long long nb = chunk_grid(a.ch, n, a.H, bc, a.per, a.parts.splits);
  if (a.parts.splits > 1 && flags) return BURST_ERR_SHAPE;
  for (int i = 0; i < n && a.parts.splits == 1; i++) a.ch[i].order = keys_order(p, ch[i], n, a.H, bc, 32, nw == 8 ? 1 : 2);
  static DeviceOnce done, done2;
  const int st = launch_plain(a.parts.splits > 1 ? burst_bwd_dkv_d64_kernel<false, true, SK_GROUPS, SK_WAVES>
                              : groups == G ? burst_bwd_dkv_d64_kernel<false, false, G, SK_WAVES> : burst_bwd_dkv_d64_kernel<false, false, SK_GROUPS, SK_WAVES>,
                              nw == SK_WAVES ? burst_bwd_dkv_d64_kernel<true, false, SK_GROUPS, SK_WAVES> : burst_bwd_dkv_d64_kernel<true, false, 1, FINE>,
                              nw == SK_WAVES ? done : done2, a, nb, (long long)p.group * ((p.Nq + 31) / 32), 64 * nw, stream);
  return st != BURST_OK || a.parts.splits == 1 ? st : launch_merge_dkv<S_D, sk_keys(SK_WAVES, SK_GROUPS), sk_rows(SK_GROUPS), S_PAD>(a, stream);
}

}  // namespace BURST_SMALL_NS
}  // namespace burst
