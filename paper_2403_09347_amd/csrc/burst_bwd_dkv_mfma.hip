// Backward, dK / dV side of one block pair (paper Alg. 2 loop body) for bf16, d = 128.
//
// Key-stationary half of the split backward (see burst_bwd_dq_mfma.hip for why it is split):
//     S = Q K^T,  dP = dO V^T,  P = exp(S - lse),  dS = P o (dP - D),
//     dV += P^T dO,  dK += dS^T Q
// P is recomputed from the saved log-sum-exp; neither S, P nor dS is ever stored.
//
// One workgroup = 4 wavefronts = 128 keys of one (batch, head); a wavefront owns 32 keys:
// their K and V fragments (B operands of S and dP) and the dK / dV accumulators stay in
// registers for the whole kernel, the accumulators pinned in AGPRs.  Query rows stream through
// in tiles of 64 rows (two 32-row blocks): Q and dO tiles are DMA-ed from HBM into LDS rings two
// tiles ahead.  With S = Q K^T a lane owns one key and its registers run over query rows, so P
// and dS already have the A-operand layout of P^T dO and dS^T Q (contraction over rows); the B
// operands dO and Q come through transposing LDS reads.  lse and D are per-row, i.e. per
// register: they are staged (already scaled) in a small LDS ring and read as broadcasts.
// The 64 MFMAs of a tile run in four phases of 16, software-pipelined across the two row
// blocks so that the vector work of one block rides on the MFMAs of the other:
//   1: S, dP of block 0            2: S, dP of block 1   + P, dS of block 0
//   3: dV, dK of block 0 + P, dS of block 1              4: dV, dK of block 1 + DMA of tile t+2
// No atomics: every key row is owned by one wavefront, results are bitwise reproducible.
// A launch takes several chunks: their workgroups form one grid, chunk after chunk, so that short or
// mostly hidden chunks fill the chip together (16 chunks of 512 keys, 32 heads x 512 causal rows,
// backward: 575 us with a launch per chunk, 338 us; long chunks take the same time either way).
//
// A second shape of the same kernel has 2 wavefronts = 64 keys per workgroup and two workgroups
// per CU (NW = 2), for block flags 64 keys wide (paper Sec. 2.6): a workgroup's tile list then
// holds what its own 64 keys need and nothing else, which the 128-key shape cannot offer (a tile
// that half of its keys need costs the full time).  Two workgroups share the CU's LDS, so the
// tile ring has two slots instead of three and a tile is fetched one step ahead instead of two.
#include <algorithm>
#include "burst_bwd_common.h"

namespace burst {

constexpr int DKV_BR = 64;            // query rows per tile
constexpr int DKV_TILE_BYTES = DKV_BR * 256;
constexpr int DKV_STAT_SLOTS = 4;     // row statistics run one tile further ahead than the tiles
// Sizes and LDS layout for NW wavefronts per workgroup.
template <int NW>
struct DkvShape {
  static constexpr int BC = 32 * NW;                 // keys per workgroup
  static constexpr int SLOTS = NW == 4 ? 3 : 2;      // tile ring
  static constexpr int LPW = 16 / NW;                // DMA wave-loads per tensor and tile that a wavefront issues
  static constexpr int LDS_Q = 0;
  static constexpr int LDS_G = SLOTS * DKV_TILE_BYTES;
  static constexpr int LDS_L = 2 * SLOTS * DKV_TILE_BYTES;             // -lse / scale per row
  static constexpr int LDS_D = LDS_L + DKV_STAT_SLOTS * DKV_BR * 4;    // -D per row
  static constexpr int LDS_DUMMY = LDS_D + DKV_STAT_SLOTS * DKV_BR * 4;  // sink of the padding DMA (256 B)
  static constexpr int LDS_BYTES = LDS_DUMMY + 256;
  // block-sparse calls: most query tiles of one slice (512K rows; 128K rows where two workgroups
  // share the LDS)
  static constexpr int MAX_LIST = NW == 4 ? 8192 : 2048;
  static constexpr int LIST_BYTES = (MAX_LIST + 8) * 4;
};

struct DkvArgs {
  const bf16* Q; const bf16* dO;
  const float* lse; const float* D;
  int Nq, H, group;      // H counts batch x key/value heads; query heads per key/value head
  int causal, acc_dkv;
  int half;              // dK, dV are bf16
  float c, scale;        // c = scale * log2(e)
  long long q_off;
  long long window;      // 0 = none; else keys at positions <= query position - window are hidden
  int bsize;             // block flags: edge, a multiple of 64
  int n, per;            // chunks, all with block flags or none; workgroups of each (chunk_at)
  Layout lay;            // strides of Q and dO
  Chunk ch[kMaxChunks];
  RowParts parts;
  int items, turn;       // CHAIN: workgroups that the launch stands for; the order in which they are taken (see next_item)
};

// SPARSE: the call carries block flags (paper Sec. 2.6) or several query heads share a key/value
// head (a.group > 1: the tiles of all heads of the group are walked, `head` is then the key/value
// head; an entry also names the head of its tile, whose rows have buffer descriptors of their own,
// so that the rows past Nq of its last tile read as zeros).  The workgroup first writes the list of
// query tiles that at least one of its wavefronts' keys are visible to (tile index plus one bit per
// wavefront) into LDS and then walks that list instead of t_begin, t_begin + 1, ...; a wavefront
// whose bit is clear hides the whole tile in the masking path.  Entries past the end name a tile
// beyond the slice: its Q, dO and statistics read as zeros and contribute nothing.
// PARTS: the walks are cut (RowParts; calls without flags only).
// CHAIN: 256 workgroups, one per CU, compute the work of a.items ones each, every 256th (calls without flags or groups).
// While a block's last two tiles are computed, the K and V rows of the workgroup's next block are fetched into the
// tile slots that become free (they look like two more tiles: rows of Q and of K must lie the same distance
// apart), and the first tiles of the next block are requested before the results of this one are stored.
template <bool SPARSE, int NW, bool PARTS, bool CHAIN>
__global__ void __launch_bounds__(64 * NW, 1)
burst_bwd_dkv_kernel(DkvArgs a) {
  using Shape = DkvShape<NW>;
  constexpr int DKV_BC = Shape::BC, DKV_SLOTS = Shape::SLOTS, LPW = Shape::LPW;
  constexpr int DKV_LDS_Q = Shape::LDS_Q, DKV_LDS_G = Shape::LDS_G, DKV_LDS_L = Shape::LDS_L, DKV_LDS_D = Shape::LDS_D;
  constexpr int DKV_LDS_DUMMY = Shape::LDS_DUMMY, DKV_LDS_BYTES = Shape::LDS_BYTES;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x;
  const int w = tid >> 6, lane = tid & 63, lr = lane & 31, h = lane >> 5;
  // the workgroups of all chunks, chunk after chunk
  int chunk, head, kblk, part = 0;
  RowRange range;
  // CHAIN: the next block of keys of this workgroup that some row sees; those that none sees, before it, become zero.
  // a.turn = n > 1: the workgroups of an XCD begin at n places of their list (whole chunks apart, so that they share the
  // query tiles of one head), and hidden chunks, which are nothing but stores, are spread over the launch.  0: every
  // second round is dealt in reverse.
  int round = 0;
  auto next_item = [&](int& c, int& hd, int& kb, RowRange& r) __attribute__((always_inline)) {
    const int rounds = (a.items + 255) >> 8;
    const int rot = a.turn > 1 ? (int)(blockIdx.x >> 3) * a.turn / 32 * (rounds / a.turn) : 0;
    while (round < rounds) {
      int at = round + rot;
      if (at >= rounds) at -= rounds;
      const int id = 256 * at + (a.turn == 0 && (at & 1) ? (int)(blockIdx.x ^ 248) : (int)blockIdx.x);
      round++;
      if (id >= a.items) continue;
      c = chunk_at(id, a.ch, a.n, a.per);
      const Chunk& X = a.ch[c];
      if (!locate_block(id - X.first_block, a.H, (X.Nc + DKV_BC - 1) / DKV_BC, hd, kb)) continue;
      r = row_range(a.Nq, a.causal, a.window, a.q_off, X.k_off, X.Nc, kb * DKV_BC, DKV_BC, DKV_BR);
      if (r.lo + 1 == r.hi) r.hi++;                // (two tiles at least, for K and V behind them; no row past the range sees the keys)
      if (r.hi > r.lo) {
        c = __builtin_amdgcn_readfirstlane(c); hd = __builtin_amdgcn_readfirstlane(hd); kb = __builtin_amdgcn_readfirstlane(kb);
        r.lo = __builtin_amdgcn_readfirstlane(r.lo); r.hi = __builtin_amdgcn_readfirstlane(r.hi);
        return true;
      }
      if (!a.acc_dkv) {                            // rows of keys are contiguous in the gradients
        const size_t from = ((size_t)hd * X.Nc + (size_t)kb * DKV_BC) * (a.half ? 256 : 512);
        const unsigned bytes = (unsigned)min(DKV_BC, X.Nc - kb * DKV_BC) * (a.half ? 256u : 512u);
        const __amdgpu_buffer_rsrc_t k0 = make_rsrc((const char*)X.dK + from, bytes), v0 = make_rsrc((const char*)X.dV + from, bytes);
        typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
        const u32x4 z = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 16; i++) {             // (past the end: not stored)
          __builtin_amdgcn_raw_buffer_store_b128(z, k0, tid * 16 + i * 4096, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b128(z, v0, tid * 16 + i * 4096, 0, 0);
        }
      }
    }
    return false;
  };
  if constexpr (CHAIN) {
    if (!next_item(chunk, head, kblk, range)) return;
  } else {
    chunk = chunk_at((int)blockIdx.x, a.ch, a.n, a.per);
    const int bid = (int)blockIdx.x - a.ch[chunk].first_block, blocks = (a.ch[chunk].Nc + DKV_BC - 1) / DKV_BC;
    if constexpr (PARTS) {
      if (!locate_part(bid, a.H, blocks, a.parts.splits, head, kblk, part)) return;
    } else {
      if (!locate_block(bid, a.H, blocks, head, kblk, a.ch[chunk].order)) return;
    }
  }
  const int group = SPARSE ? a.group : 1;          // query heads that share this key/value head
  const int q_rows = group * a.Nq;                 // rows of the group's Q / dO / lse / D
  const unsigned qpitch = (unsigned)a.lay.qs_r * 2u;             // bytes between query rows
  const unsigned qtile = qpitch * DKV_BR;                        // ... between query tiles

  // (a.ch[chunk] throughout: through a pointer that changes the compiler copies the arguments to scratch memory)
  int Nc = a.ch[chunk].Nc, key_wg = kblk * DKV_BC, key0 = key_wg + w * 32;   // key0: first key of this wavefront
  long long k_off = a.ch[chunk].k_off;
  const bf16 *Qh, *Gh;                             // first query head of the group
  const float *lseh, *Dh;
  auto of_head = [&]() __attribute__((always_inline)) {
    Qh = a.Q + a.lay.q_base(head * group);
    Gh = a.dO + a.lay.q_base(head * group);
    lseh = a.lse + (size_t)head * q_rows;
    Dh = a.D + (size_t)head * q_rows;
  };
  of_head();
  auto keys_rsrc = [&](const Chunk& X, int hd, bool v) __attribute__((always_inline)) {   // keys past Nc: outside
    return make_rsrc((const bf16*)(v ? X.V : X.K) + X.kv_base(hd, a.lay.kv_heads), (unsigned)(X.Nc - 1) * (unsigned)X.ks_r * 2u + 256u);
  };

  // query tiles of a head to visit; of the walk over all of them, this workgroup's part
  if constexpr (!CHAIN) range = row_range(a.Nq, a.causal, a.window, a.q_off, k_off, Nc, key_wg, DKV_BC, DKV_BR);
  const int ntiles_all = range.hi;
  int t_begin = range.lo, first = 0, nwalk = ntiles_all - t_begin, parts = 1;   // (tiles to walk)
  if constexpr (PARTS) {
    nwalk *= group;
    parts = a.parts.of(nwalk);
    if (part >= parts) return;
    first = (int)((long long)nwalk * part / parts);
    nwalk = (int)((long long)nwalk * (part + 1) / parts) - first;
  }

  f32x16 dk[4], dv[4];     // [32-wide d block]: rows = the wavefront's 32 keys; pinned in AGPRs
#pragma unroll
  for (int db = 0; db < 4; db++)
#pragma unroll
    for (int r = 0; r < 16; r++) { dk[db][r] = 0.f; dv[db][r] = 0.f; }

  // K, V fragments (B operands: lane = key lr, 8 consecutive d; keys past Nc: outside the buffers, zero).
  // With a list they are requested before it is built, so that the two latencies overlap.
  bf16x8 kf[8], vf[8];
  auto load_kv = [&]() __attribute__((always_inline)) {
    const unsigned kpitch = (unsigned)a.ch[chunk].ks_r * 2u;
    const __amdgpu_buffer_rsrc_t krs = keys_rsrc(a.ch[chunk], head, false), vrs = keys_rsrc(a.ch[chunk], head, true);
    const unsigned off = (unsigned)(key0 + lr) * kpitch + h * 16u;
#pragma unroll
    for (int ks = 0; ks < 8; ks++) {
      kf[ks] = __builtin_bit_cast(bf16x8, buffer_load_b128(krs, (int)(off + ks * 32u)));
      vf[ks] = __builtin_bit_cast(bf16x8, buffer_load_b128(vrs, (int)(off + ks * 32u)));
    }
  };
  if constexpr (SPARSE) load_kv();
  // SPARSE: the list of visible tiles, built by wavefront 0 (64 candidate tiles per round).
  // list[0] = number of entries, list[1 + j] = tile | (wavefront bits << 16), then 4 end entries.
  int* list = reinterpret_cast<int*>(smem + DKV_LDS_BYTES);
  if constexpr (SPARSE) {
    const int end_tile = (a.Nq + DKV_BR - 1) / DKV_BR;          // a tile past the rows of the group's first head
    if (w == 0) {
      int n = 0;
      for (int g = 0; g < group; g++)
        for (int base = t_begin; base < ntiles_all; base += 64) {
          const int t = base + lane;
          int bits = 0;
          if (t < ntiles_all) {
            if (a.ch[chunk].bmask == nullptr) {
              bits = (1 << NW) - 1;
            } else {
              const uint8_t* mrow = a.ch[chunk].bmask + (size_t)(head * group + g) * a.ch[chunk].bhstride + (size_t)((t * DKV_BR) / a.bsize) * a.ch[chunk].bpitch;
#pragma unroll
              for (int ww = 0; ww < NW; ww++) {
                const int k0 = key_wg + ww * 32;
                if (k0 < Nc && mrow[k0 / a.bsize] != 0) bits |= 1 << ww;
              }
            }
          }
          const unsigned long long bal = __builtin_amdgcn_ballot_w64(bits != 0);
          if (bits != 0) {
            const int pos = n + __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
            list[1 + pos] = t | (bits << 16) | (g << 20);
          }
          n += __builtin_popcountll(bal);
        }
      if (lane < 4) list[1 + n + lane] = end_tile;
      if (lane == 0) list[0] = n;
    }
    __syncthreads();
    if constexpr (PARTS) list += first;            // (the list holds the whole walk)
    else nwalk = __builtin_amdgcn_readfirstlane(list[0]);
  } else {
    t_begin += first;
  }
  // walk position j -> its entry: the tile of its head in the low 16 bits and, SPARSE, the wavefront
  // bits (16..19) and the head of the group (20..27)
  auto entry_at = [&](int j) __attribute__((always_inline)) {
    if constexpr (SPARSE) return __builtin_amdgcn_readfirstlane(list[1 + j]);
    else return t_begin + j;
  };
  auto tile_of = [&](int e) __attribute__((always_inline)) {
    if constexpr (SPARSE) return e & 0xffff;
    else return e;
  };

  if (nwalk > 0) {
    if constexpr (!SPARSE) load_kv();
    // LDS addressing inside a 64-row tile.  A operands (128-bit): row rb*32 + lr, granule
    // 2*ks + h -> rb*8192 + (abase ^ (ks << 5)).  B operands through transposing reads:
    // rows = query rows rb*32 + u*16 + ..., cols = d.
    const int abase = lr * 256 + ((h ^ row_code(lr)) << 4);
    int taddr[4][2];
    {
      const int j16 = lane & 15, dh = (lane >> 4) & 1;
#pragma unroll
      for (int db = 0; db < 4; db++)
#pragma unroll
        for (int sx = 0; sx < 2; sx++)
          taddr[db][sx] = tile_off(8 * sx + 4 * h + (j16 >> 2), db * 4 + 2 * dh + ((j16 & 3) >> 1)) + (j16 & 1) * 8;
    }
    // DMA: a 64-row tile is 16 wave-loads of 4 rows; wavefront w issues loads LPW*w .. LPW*w + LPW-1
    const unsigned qbytes = a.Nq > 0 ? (unsigned)(a.Nq - 1) * qpitch + 256u : 0u;
    // (a descriptor per head of the group; without a list there is one head)
    auto head_of = [&](int e) __attribute__((always_inline)) { return SPARSE ? (e >> 20) & 0xff : 0; };
    auto q_rsrc = [&](int e) __attribute__((always_inline)) { return make_rsrc(Qh + (size_t)head_of(e) * a.lay.qs_h, qbytes); };
    auto g_rsrc = [&](int e) __attribute__((always_inline)) { return make_rsrc(Gh + (size_t)head_of(e) * a.lay.qs_h, qbytes); };
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const unsigned lds0 = lds_addr(smem);
    int goff[LPW];
#pragma unroll
    for (int il = 0; il < LPW; il++) {
      int row = 4 * LPW * w + 4 * il + (lane >> 4);
      goff[il] = (int)(row * qpitch + (((lane & 15) ^ row_code(row)) << 4));
    }
    // base: byte offset of the tile's first row
    auto dma_tile = [&](__amdgpu_buffer_rsrc_t rs, unsigned lds_tile, int il, unsigned base) __attribute__((always_inline)) {
      dma_b128_to_lds(rs, lds_tile + (unsigned)(wu * LPW + il) * 1024u, (int)base + goff[il]);
    };
    // Per-row statistics of a tile travel like the tiles: wavefront 0 DMAs the 64 lse values,
    // wavefront 1 the 64 D values (rows past Nq read as 0; their Q and dO rows are 0 too, so they
    // contribute nothing).  Two steps before use, wavefront 0 rewrites lse in place as
    // -lse/scale, or -inf for a row that saw nothing (then P = exp2(-inf) = 0), and wavefront
    // 1 rewrites D as -D: the S and dP accumulators START at these values, so that
    // P = exp2(c (Q K^T - lse/scale)) and dS = P o (dO V^T - D) need no subtraction in the
    // per-element vector work.  (Multiplying K by c beforehand would also remove the multiply,
    // but rounds c K to bf16 again; with few visible keys per row P is then visibly off.)  No
    // compiler-visible global load is left in the loop: its wait would drain the DMA queue.
    auto dma_rowstat = [&](int e, int slot) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t srs = make_rsrc((wu == 1 ? Dh : lseh) + (size_t)head_of(e) * a.Nq, (unsigned)a.Nq * 4u);
      // every wavefront issues exactly one such load per tile (the wait counts below rely on
      // it): 0 -> lse, 1 -> D, 2 and 3 -> a dummy copy of lse that nobody reads
      const unsigned dst = (wu == 0) ? lds0 + DKV_LDS_L + slot * DKV_BR * 4
                         : (wu == 1) ? lds0 + DKV_LDS_D + slot * DKV_BR * 4 : lds0 + DKV_LDS_DUMMY;
      dma_b32_to_lds(srs, dst, (tile_of(e) * DKV_BR + lane) * 4);
    };
    const float inv_scale = 1.0f / a.scale;
    // The same in two parts for the main loop, so that the LDS round trip hides behind MFMAs:
    // wavefronts 0 / 1 fetch their 64 values at one point of the step and write them back later.
    float stat_tmp = 0.f;
    auto rowstat_fetch = [&](int slot) __attribute__((always_inline)) {
      if (tid < 64) stat_tmp = *(reinterpret_cast<const float*>(smem + DKV_LDS_L) + slot * DKV_BR + tid);
      else if (tid < 128) stat_tmp = *(reinterpret_cast<const float*>(smem + DKV_LDS_D) + slot * DKV_BR + (tid - 64));
    };
    auto rowstat_store = [&](int slot) __attribute__((always_inline)) {
      if (tid < 64)
        *(reinterpret_cast<float*>(smem + DKV_LDS_L) + slot * DKV_BR + tid) =
            (stat_tmp == BURST_NEG_INF) ? BURST_NEG_INF : -stat_tmp * inv_scale;
      else if (tid < 128)
        *(reinterpret_cast<float*>(smem + DKV_LDS_D) + slot * DKV_BR + (tid - 64)) = -stat_tmp;
    };
    auto scale_rowstat = [&](int slot) __attribute__((always_inline)) {
      if (tid < 64) {
        float* ptr = reinterpret_cast<float*>(smem + DKV_LDS_L) + slot * DKV_BR + tid;
        float lv = *ptr;
        *ptr = (lv == BURST_NEG_INF) ? BURST_NEG_INF : -lv * inv_scale;
      } else if (tid < 128) {
        float* ptr = reinterpret_cast<float*>(smem + DKV_LDS_D) + slot * DKV_BR + (tid - 64);
        *ptr = -*ptr;
      }
    };

    // CHAIN: the next block of keys.  Its K and V rows follow the tiles of the walk as two more.
    int c_next = 0, head_next = 0, blk_next = 0;
    RowRange range_next = {0, 0};
    bool more = false;
    const bf16 *K_next = nullptr, *V_next = nullptr;
    unsigned bytes_next = 0;
    // What is fetched at walk position m (entry e): Q or K rows, dO or V rows, the offset of the first one.
    auto first_rsrc = [&](int m, int e) __attribute__((always_inline)) {
      if constexpr (CHAIN) return make_rsrc(m < nwalk ? Qh : K_next, m < nwalk ? qbytes : bytes_next);
      else return q_rsrc(e);
    };
    auto second_rsrc = [&](int m, int e) __attribute__((always_inline)) {
      if constexpr (CHAIN) return make_rsrc(m < nwalk ? Gh : V_next, m < nwalk ? qbytes : bytes_next);
      else return g_rsrc(e);
    };
    auto first_row_at = [&](int m, int e) __attribute__((always_inline)) {
      if constexpr (CHAIN) return (unsigned)(m < nwalk ? t_begin + m : 2 * blk_next + m - nwalk) * qtile;
      else return (unsigned)tile_of(e) * qtile;
    };
    // ---- prologue: tiles t_begin, t_begin + 1 into tile slots 0, 1 (two slots: the first tile
    // alone); the statistics of tiles t_begin .. t_begin + 2 into statistic slots 0 .. 2, the
    // first two scaled when they are there
    auto start_tiles = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < DKV_SLOTS - 1; t++) {
        const int e = entry_at(t);
        const unsigned base = (unsigned)tile_of(e) * qtile;
#pragma unroll
        for (int il = 0; il < LPW; il++) {
          dma_tile(q_rsrc(e), lds0 + DKV_LDS_Q + t * DKV_TILE_BYTES, il, base);
          dma_tile(g_rsrc(e), lds0 + DKV_LDS_G + t * DKV_TILE_BYTES, il, base);
        }
      }
#pragma unroll
      for (int t = 0; t < 3; t++) dma_rowstat(entry_at(t), t);
    };
    start_tiles();
    for (;;) {                                     // (CHAIN: the blocks of this workgroup; else once)
    if constexpr (CHAIN) {
      more = next_item(c_next, head_next, blk_next, range_next);
      const size_t at = a.ch[c_next].kv_base(head_next, a.lay.kv_heads);
      K_next = (const bf16*)a.ch[c_next].K + at;
      V_next = (const bf16*)a.ch[c_next].V + at;
      bytes_next = more ? (unsigned)(a.ch[c_next].Nc - 1) * qpitch + 256u : 0u;
    }
    __builtin_amdgcn_s_waitcnt(0x0070);            // vmcnt(0), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    scale_rowstat(0);
    scale_rowstat(1);
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();

    const long long wave_first_k = k_off + key0;
    const long long wave_last_k = wave_first_k + 31;
    const long long kpos = wave_first_k + lr;
    constexpr int LEAD = 6, RING = LEAD + 2;       // A-operand reads run LEAD slices ahead
    constexpr int TLEAD = 5, TRING = TLEAD + 1;    // transposed fragments run TLEAD slices ahead
                                                   // (SQ counters showed 7 % of the wave time waiting for LDS at 4 / 3)

    // S and dP accumulators of the two row blocks.  They start at -lse/scale and -D of their
    // rows (register r of a block = row 8*(r/4) + 4h + r%4: four 128-bit broadcast reads per
    // block and statistic, straight into the accumulator registers).  Block 0 of the next tile is
    // loaded while the current tile's last phases run.
    f32x16 s[2], dp[2];
    auto load_init = [&](int rb, const float* lrow, const float* drow) __attribute__((always_inline)) {
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const f32x4 lv = *reinterpret_cast<const f32x4*>(lrow + rb * 32 + 8 * q4 + 4 * h);
        const f32x4 dv = *reinterpret_cast<const f32x4*>(drow + rb * 32 + 8 * q4 + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; j++) { s[rb][4 * q4 + j] = lv[j]; dp[rb][4 * q4 + j] = dv[j]; }
      }
    };
    load_init(0, reinterpret_cast<const float*>(smem + DKV_LDS_L), reinterpret_cast<const float*>(smem + DKV_LDS_D));

    // lgkmcnt(0).  With a scalar load possibly still on its way at the loop's entry the compiler waits, in every step, for
    // all six operand reads before the first MFMA instead of for one (1 % of long walks, 2 % of short ones).
    int ahead[4];                                    // SPARSE: the entries of this tile and the next three
    if constexpr (SPARSE) {
#pragma unroll
      for (int j = 0; j < 4; j++) ahead[j] = entry_at(j);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);
    int slot = 0;
    for (int n = 0; n < nwalk; n++) {                  // n = walk position; statistic slot n & 3 holds its tile
      // this tile, the entries of the tile whose rows are fetched now and of the one whose statistics are
      int t = t_begin + n, t2 = t + DKV_SLOTS - 1, t3 = t + 3;
      bool mine = true;                                // SPARSE: this wavefront's keys are visible to the tile
      int entry4 = 0;
      if constexpr (SPARSE) {
        entry4 = list[1 + n + 4];                    // (used at the end of the step)
        t = ahead[0] & 0xffff;
        mine = ((ahead[0] >> (16 + wu)) & 1) != 0;
        t2 = ahead[DKV_SLOTS - 1];
        t3 = ahead[3];
      }
      const __amdgpu_buffer_rsrc_t qrs = first_rsrc(n + DKV_SLOTS - 1, t2), grs = second_rsrc(n + DKV_SLOTS - 1, t2);
      const unsigned base2 = first_row_at(n + DKV_SLOTS - 1, t2);
      const int slot1 = (slot == DKV_SLOTS - 1) ? 0 : slot + 1;
      // where the tile fetched in this step goes: the slot after the next tile's, or (two slots) the next tile's
      const int slot2 = DKV_SLOTS == 2 ? slot1 : (slot1 == DKV_SLOTS - 1) ? 0 : slot1 + 1;
      const char* ql = smem + DKV_LDS_Q + slot * DKV_TILE_BYTES;
      const char* gl = smem + DKV_LDS_G + slot * DKV_TILE_BYTES;
      const float* lp = reinterpret_cast<const float*>(smem + DKV_LDS_L) + (n & 3) * DKV_BR;
      const float* dp_ = reinterpret_cast<const float*>(smem + DKV_LDS_D) + (n & 3) * DKV_BR;
      const float* lp_next = reinterpret_cast<const float*>(smem + DKV_LDS_L) + ((n + 1) & 3) * DKV_BR;
      const float* dp_next = reinterpret_cast<const float*>(smem + DKV_LDS_D) + ((n + 1) & 3) * DKV_BR;
      const long long tile_first_q = a.q_off + (long long)t * DKV_BR;
      // (no branch around the MFMA phases: the AGPR-pinned accumulators must not become phi
      // values, the allocator would shuttle them through VGPRs every iteration)
      const bool need_mask = (a.causal && wave_last_k > tile_first_q) ||
                             (a.window > 0 && tile_first_q + DKV_BR - 1 >= wave_first_k + a.window) || !mine;
      {
        // A-operand read j (0..31): rb = j / 16, ks = (j / 2) % 8, even: Q fragment (for S), odd:
        // dO fragment (for dP).  S and dP alternate so that no MFMA waits for its predecessor.
        bf16x8 fq[RING];
        auto issue_read = [&](int j) __attribute__((always_inline)) {
          const int rb = j >> 4, isg = j & 1, ks = (j >> 1) & 7;
          fq[j % RING] = lds_read_b128(isg ? gl : ql, rb * 32 * 256 + (abase ^ (ks << 5)));
        };
        // transposed fragment j (0..31): rb = j / 16, u = (j / 8) % 2, db = (j / 2) % 4, then
        // 0: dO (for dV), 1: Q (for dK)
        bf16x4 tq[TRING][2];
        auto issue_tread = [&](int j) __attribute__((always_inline)) {
          const int rb = j >> 4, u = (j >> 3) & 1, db = (j >> 1) & 3, isq = j & 1;
          const char* base = isq ? ql : gl;
          const int off = (rb * 32 + u * 16) * 256;
          tq[j % TRING][0] = lds_read_tr(base, off + taddr[db][0]);
          tq[j % TRING][1] = lds_read_tr(base, off + taddr[db][1]);
        };
        bf16x8 pf[2][2], dsf[2][2];   // [row block][16-row group]: A operands of dV, dK
        // P and dS of two scores: register pair (r, r+1) of row block rb = rows 8*(r/4)+4h+r%4.
        // The work is cut in two halves, one per MFMA slice: an in-order wavefront hides only
        // what it issues between two of its own MFMAs.
        float ph0, ph1;
        auto pds_half0 = [&](int rb, int pidx) __attribute__((always_inline)) {  // pidx 0..7
          const int r = 2 * pidx;
          ph0 = fast_exp2(s[rb][r] * a.c);
          ph1 = fast_exp2(s[rb][r + 1] * a.c);
          asm volatile("" : "+v"(ph0), "+v"(ph1));   // keep the arithmetic in this slice
        };
        auto pds_half1 = [&](int rb, int pidx) __attribute__((always_inline)) {
          const int r = 2 * pidx, u = r >> 3, t8 = r & 7;
          float d0 = ph0 * dp[rb][r];
          float d1 = ph1 * dp[rb][r + 1];
          bf16x2 pk, dk2;
          pk[0] = (bf16)ph0; pk[1] = (bf16)ph1;
          dk2[0] = (bf16)d0; dk2[1] = (bf16)d1;
          // (the only consumers are MFMAs two phases later; without an anchor the compiler sinks
          // the arithmetic there, behind the mask branches)
          unsigned pu = __builtin_bit_cast(unsigned, pk), du = __builtin_bit_cast(unsigned, dk2);
          asm volatile("" : "+v"(pu), "+v"(du));
          pk = __builtin_bit_cast(bf16x2, pu); dk2 = __builtin_bit_cast(bf16x2, du);
          pf[rb][u][t8] = pk[0]; pf[rb][u][t8 + 1] = pk[1];
          dsf[rb][u][t8] = dk2[0]; dsf[rb][u][t8 + 1] = dk2[1];
        };
        // mask of one row block (rare: tiles that straddle the diagonal or the far edge of the
        // sliding window).  Register r belongs to row tile_first_q + rb*32 + 4h + (8*(r/4) + r%4);
        // causal: the key is visible iff its position <= the row's, i.e. iff the constant part is
        // >= lim; window: iff the row's position < the key's + window, i.e. constant part <= lim2.
        // A masked score becomes -inf, its P and dS become 0.
        auto mask_block = [&](int rb) __attribute__((always_inline)) {
          const long long d = kpos - (tile_first_q + rb * 32 + 4 * h);
          const int lim = !mine ? 65 : a.causal ? (int)(d < -1 ? -1 : (d > 64 ? 64 : d)) : -1;
          const long long d2 = d + a.window - 1;
          const int lim2 = a.window > 0 ? (int)(d2 < -1 ? -1 : (d2 > 64 ? 64 : d2)) : 64;
#pragma unroll
          for (int r = 0; r < 16; r++) {
            const int cpart = 8 * (r >> 2) + (r & 3);
            s[rb][r] = (cpart >= lim && cpart <= lim2) ? s[rb][r] : BURST_NEG_INF;
          }
        };
#pragma unroll
        for (int j = 0; j < LEAD; j++) issue_read(j);
        __builtin_amdgcn_sched_barrier(0);
        // ---- phases 1, 2: S and dP (slice i: rb = i / 16, ks = (i / 2) % 8, even S, odd dP); in
        // phase 2 the P / dS pairs of row block 0 ride along (one pair every second slice)
#pragma unroll
        for (int i = 0; i < 32; i++) {
          const int rb = i >> 4, isg = i & 1, ks = (i >> 1) & 7;
          if (i == 16 && need_mask) mask_block(0);
          if (i + LEAD < 32) issue_read(i + LEAD);
          if (i + TLEAD >= 32) issue_tread(i + TLEAD - 32);
          if (i == 2) load_init(1, lp, dp_);
          if constexpr (DKV_SLOTS == 2) {
            // two slots: the slot of tile t - 1 is free since the last barrier; tile t + 1 and the
            // statistics of tile t + 3 are requested here and awaited at the end of the step
            if (i == 0) dma_rowstat(t3, (n + 3) & 3);
            if (i < 2 * LPW) {
              if (i & 1) dma_tile(grs, lds0 + DKV_LDS_G + slot2 * DKV_TILE_BYTES, i >> 1, base2);
              else dma_tile(qrs, lds0 + DKV_LDS_Q + slot2 * DKV_TILE_BYTES, i >> 1, base2);
            }
          }
          if (isg) dp[rb] = mfma32(fq[i % RING], vf[ks], dp[rb]);
          else s[rb] = mfma32(fq[i % RING], kf[ks], s[rb]);
          if (i >= 16) { if (i & 1) pds_half1(0, (i - 16) >> 1); else pds_half0(0, (i - 16) >> 1); }
          __builtin_amdgcn_sched_barrier(0);
        }
        // ---- phases 3, 4: dV += P^T dO, dK += dS^T Q (slice i: rb = i / 16, u = (i / 8) % 2,
        // db = (i / 2) % 4, even: dV, odd: dK); in phase 3 the pairs of row block 1 ride along
#pragma unroll
        for (int i = 0; i < 32; i++) {
          const int rb = i >> 4, u = (i >> 3) & 1, db = (i >> 1) & 3, isk = i & 1;
          if (i == 0 && need_mask) mask_block(1);
          if (i + TLEAD < 32) issue_tread(i + TLEAD);
          if (i == 4) load_init(0, lp_next, dp_next);     // block 0 of tile t + 1
          // the loads of the previous step (tile t + 1, statistics of tile t + 2) are most of a
          // step old: wait for them here, before this step's loads are issued, and rewrite those
          // statistics (fetch now, store a few slices later)
          // (two slots: they were awaited at the end of the previous step)
          if (i == 12) { if constexpr (DKV_SLOTS == 3) __builtin_amdgcn_s_waitcnt(0x0F70); rowstat_fetch((n + 2) & 3); }
          if (i == 22) rowstat_store((n + 2) & 3);
          // phase 4 has no vector work: the DMA of tile t + 2 (into the slot of tile t - 1, free
          // since the last barrier) and of the statistics of tile t + 3 is issued here
          if (DKV_SLOTS == 3 && i == 16) dma_rowstat(t3, (n + 3) & 3);
          if (DKV_SLOTS == 3 && i > 16 && (i & 1)) {
            const int j = (i - 17) >> 1;                  // 0..7: Q rows, then dO rows
            if (j < 4) dma_tile(qrs, lds0 + DKV_LDS_Q + slot2 * DKV_TILE_BYTES, j, base2);
            else dma_tile(grs, lds0 + DKV_LDS_G + slot2 * DKV_TILE_BYTES, j - 4, base2);
          }
          const bf16x8 bt = cat4(tq[i % TRING][0], tq[i % TRING][1]);
          if (isk) mfma32_acc(dk[db], dsf[rb][u], bt);
          else mfma32_acc(dv[db], pf[rb][u], bt);
          if (i < 16) { if (i & 1) pds_half1(1, i >> 1); else pds_half0(1, i >> 1); }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // ---- three slots: the 9 loads of this step stay in flight across the barrier; two: the 17
      // loads, issued most of a step ago, must have landed.  The LDS stores of the rewritten
      // statistics must be done.
      slot = slot1;
      if constexpr (SPARSE) {
        ahead[0] = ahead[1]; ahead[1] = ahead[2]; ahead[2] = ahead[3];
        ahead[3] = __builtin_amdgcn_readfirstlane(entry4);
      }
      if constexpr (DKV_SLOTS == 3) __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0)
      else __builtin_amdgcn_s_waitcnt(0x0070);                                   // vmcnt(0), lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): no DMA may outlive the loop
    // wait for the last MFMAs before anything else touches the accumulators (inside the block:
    // behind the join with the path that skipped the loop the compiler may already move them)
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15"
                 : "+a"(dk[0]), "+a"(dk[1]), "+a"(dk[2]), "+a"(dk[3]),
                   "+a"(dv[0]), "+a"(dv[1]), "+a"(dv[2]), "+a"(dv[3]));
    if constexpr (!CHAIN) break;
    else {
      const int P_chunk = chunk, P_Nc = Nc, P_key0 = key0;   // the block that is done
      const size_t at = (size_t)head * Nc * 128 * (a.half ? 2 : 4);
      if (more) {
        // its last tile lay in the slot before `slot`; `slot` and the one after it hold the next block's keys
        __builtin_amdgcn_s_barrier();              // everyone's K and V rows have landed
        const int from = w < 2 ? slot : (slot == DKV_SLOTS - 1) ? 0 : slot + 1;
        const char* const kl = smem + DKV_LDS_Q + from * DKV_TILE_BYTES + (w & 1) * 32 * 256;
        const char* const vl = smem + DKV_LDS_G + from * DKV_TILE_BYTES + (w & 1) * 32 * 256;
#pragma unroll
        for (int ks = 0; ks < 8; ks++) {
          kf[ks] = lds_read_b128(kl, abase ^ (ks << 5));
          vf[ks] = lds_read_b128(vl, abase ^ (ks << 5));
        }
        chunk = c_next; head = head_next; kblk = blk_next; range = range_next;
        Nc = a.ch[chunk].Nc; key_wg = kblk * DKV_BC; key0 = key_wg + w * 32; k_off = a.ch[chunk].k_off;
        t_begin = range.lo; nwalk = range.hi - range.lo;
        of_head();
        __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();              // ... and have been read: the slots are free
        start_tiles();
      }
      store_dkv<4, false>(dk, dv, (char*)a.ch[P_chunk].dK + at, (char*)a.ch[P_chunk].dV + at, P_Nc, 128, P_key0, lr, h, a.scale, a.half, a.acc_dkv);
      if (!more) return;
#pragma unroll
      for (int db = 0; db < 4; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) { dk[db][r] = 0.f; dv[db][r] = 0.f; }
    }
    }
  }
  // epilogue: keys are owned by this wavefront alone. C layout: lane = d column, regs = keys.
  if constexpr (PARTS) {
    void *dk_at, *dv_at;
    int keys = Nc, k0 = key0;
    if (parts > 1) {
      dk_at = a.parts.at(part, false, a.ch[chunk], head, 128); dv_at = a.parts.at(part, true, a.ch[chunk], head, 128);
      keys = a.ch[chunk].span_keys; k0 -= a.ch[chunk].span_lo;
    } else {
      const size_t at = (size_t)head * Nc * 128 * (a.half ? 2 : 4);
      dk_at = (char*)a.ch[chunk].dK + at; dv_at = (char*)a.ch[chunk].dV + at;
    }
    store_dkv<4, false>(dk, dv, dk_at, dv_at, keys, 128, k0, lr, h, a.scale, parts > 1 ? 0 : a.half, parts > 1 ? 0 : a.acc_dkv);
  } else if constexpr (!CHAIN) {
    const size_t at = (size_t)head * Nc * 128 * (a.half ? 2 : 4);
    store_dkv<4, false>(dk, dv, (char*)a.ch[chunk].dK + at, (char*)a.ch[chunk].dV + at, Nc, 128, key0, lr, h, a.scale, a.half, a.acc_dkv);
  }
}

// n chunks, all with block flags or none.  key_waves: 4 (128-key workgroups) or 2 (64-key workgroups, calls
// with block flags only).
template <bool SPARSE, int NW, bool PARTS, bool CHAIN = false>
static int launch_shape(const DkvArgs& a, long long nb, hipStream_t stream) {
  constexpr unsigned lds = DkvShape<NW>::LDS_BYTES + (SPARSE ? DkvShape<NW>::LIST_BYTES : 0);
  static DeviceOnce lds_opt_in;
  const int st = lds_opt_in.run([] {
    return hipFuncSetAttribute((const void*)burst_bwd_dkv_kernel<SPARSE, NW, PARTS, CHAIN>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               lds) == hipSuccess ? BURST_OK : BURST_ERR_LAUNCH;
  });
  if (st != BURST_OK) return st;
  BURST_LAUNCH((burst_bwd_dkv_kernel<SPARSE, NW, PARTS, CHAIN>), dim3((unsigned)nb), dim3(64 * NW), lds, stream, a);
  return launch_status();
}
// Whether the launch's nb workgroups are computed by 256 (CHAIN), and in which order (a.items, a.turn).
// The chain saves what a workgroup does before its first tile (arguments, K and V from HBM, first tiles: 5 us) and the gap to
// the next one (2 us), of 13 us beside 1.8 us a tile, and lets the zeros of hidden chunks be written while others compute.
// It is not used where
//  - walks are long (average above 36 tiles): those launches are bound by socket power, and a CU that waits gives its share to
//    the others (32 heads x 4096 rows, 64 tiles: 3834 us as workgroups, 3855 chained; 32 tiles: 1031 / 1022; 24: 606 / 595; 16:
//    318 / 302; 8: 107 / 98);
//  - the 256 shares are unequal: the largest more than 1.08 of the average (causal 32 x 3000 rows, 1.48: 166 / 195 us; chunks
//    of 2048 on both sides of the diagonal, 1.12: 497 / 510; 1.07: 232 / 219).  One causal chunk is dealt in alternating
//    direction (a.turn = 0), long blocks with short ones: 32 x 2048 rows 100 / 76 us, 128 x 1024 117 / 92, 64 x 2048 171 / 146.
// Causal walk of 16 chunks of 512 keys (32 heads) 209 / 188 us; window of 4096 over 8 chunks of 4096, five of them hidden,
// 710 / 612 (656 with all workgroups beginning at the same chunk).
static bool chained(DkvArgs& a, long long nb) {
  constexpr int BC = DkvShape<4>::BC;
  if (nb <= 256 || nb > 16384 || a.group > 1) return false;
  a.items = (int)nb;
  a.turn = a.n == 1 && a.causal ? 0 : a.n > 1 && a.per > 0 && a.per % 256 == 0 ? a.n : 1;
  const int tiles = (a.Nq + DKV_BR - 1) / DKV_BR;
  auto blocks_of = [&](int c) { return (a.ch[c].Nc + BC - 1) / BC; };
  auto range_of = [&](int c, int b) { return row_range(a.Nq, a.causal, a.window, a.q_off, a.ch[c].k_off, a.ch[c].Nc, b * BC, BC, DKV_BR); };
  long long all = 0;
  for (int c = 0; c < a.n; c++) {
    if (blocks_of(c) > 256 || a.ch[c].ks_r != a.lay.qs_r) return false;
    for (int b = 0; b < blocks_of(c); b++) {
      const RowRange r = range_of(c, b);
      all += (long long)(r.hi - r.lo) * a.H;
      // (one tile is walked as two: only where the rows of the second one, past Nq, are zeros that the first one has too)
      if (r.hi - r.lo == 1 && (r.hi != tiles || a.Nq % DKV_BR == 0)) return false;
    }
  }
  if (all > 36 * nb) return false;
  int share[256] = {};                             // in fifths of a tile: 5 a tile, 15 a block, 6 a hidden block (turns change the order only)
  for (int c = 0; c < a.n; c++) {
    const int blocks = blocks_of(c), total = a.H * blocks, per = (total + 7) / 8;
    int cost[256];                                 // of a block
    for (int b = 0; b < blocks; b++) {
      const RowRange r = range_of(c, b);
      cost[b] = r.hi > r.lo ? 5 * (r.hi - r.lo) + 15 : 6;
    }
    for (int x = 0; x < 8; x++)
      for (int at = 0, b = x * per % blocks; at < per && x * per + at < total; at++, b = b + 1 == blocks ? 0 : b + 1) {
        const int id = a.ch[c].first_block + 8 * at + x, round = id >> 8;
        share[a.turn == 0 && (round & 1) ? (id & 255) ^ 248 : id & 255] += cost[b];
      }
  }
  long long sum = 0;
  int most = 0;
  for (int i = 0; i < 256; i++) { sum += share[i]; most = std::max(most, share[i]); }
  return 100LL * 256 * most <= 108 * sum;
}
// Fills all but the pointers of a call; returns the number of its workgroups.
static long long lay_out(DkvArgs& a, const KParams& p, const Chunk* ch, int n, int key_waves, int splits) {
  a.Nq = p.Nq; a.H = p.B * p.H / p.group; a.group = p.group;     // workgroups are laid out over key/value heads
  a.c = p.scale * kLog2e; a.scale = p.scale; a.causal = p.causal; a.q_off = p.q_off; a.window = p.window; a.bsize = p.bsize;
  a.n = n; a.lay = p.lay;
  for (int i = 0; i < n; i++) a.ch[i] = ch[i];
  for (int i = 0; i < n && splits == 1; i++) a.ch[i].order = keys_order(p, ch[i], n, a.H, 32 * key_waves, DKV_BR, key_waves == 4 ? 1 : 2);
  return chunk_grid(a.ch, n, a.H, 32 * key_waves, a.per, key_waves == 4 ? splits : 1);
}
bool dkv_chained(const KParams& p, const Chunk* ch, int n) {
  DkvArgs a;
  const long long nb = lay_out(a, p, ch, n, 4, 1);
  return ch[0].bmask == nullptr && chained(a, nb);
}
int launch_bwd_dkv_mfma(const KParams& p, const BwdIo& io, const Chunk* ch, int n, hipStream_t stream, int key_waves) {
  DkvArgs a;
  a.Q = (const bf16*)io.Q; a.dO = (const bf16*)io.dO; a.lse = io.lse; a.D = io.D;
  a.acc_dkv = io.acc_dkv; a.half = io.half;
  const bool listed = ch[0].bmask != nullptr || p.group > 1;
  if (key_waves != 4 && !(key_waves == 2 && listed)) return BURST_ERR_SHAPE;
  const long long nb = lay_out(a, p, ch, n, key_waves, io.parts != nullptr ? io.parts->parts.splits : 1);
  set_row_parts(a, io);
  if (a.parts.splits > 1 && (key_waves != 4 || ch[0].bmask != nullptr)) return BURST_ERR_SHAPE;
  if (nb > 0x7fffffffLL) return BURST_ERR_SHAPE;
  if (nb == 0) return BURST_OK;
  if (listed) {
    const int max_list = key_waves == 4 ? DkvShape<4>::MAX_LIST : DkvShape<2>::MAX_LIST;
    if ((long long)a.group * ((p.Nq + DKV_BR - 1) / DKV_BR) > max_list) return BURST_ERR_SHAPE;
  }
  if (a.parts.splits > 1) {
    const int st = listed ? launch_shape<true, 4, true>(a, nb, stream) : launch_shape<false, 4, true>(a, nb, stream);
    return st != BURST_OK ? st : launch_merge_dkv<128, DkvShape<4>::BC, DKV_BR, false>(a, stream);
  }
  if (!listed) {                                   // (the validating pass sees to the attributes of both forms; the rule is asked once)
    if (t_validate_only || chained(a, nb))
      if (const int st = launch_shape<false, 4, false, true>(a, 256, stream); st != BURST_OK || !t_validate_only) return st;
    return launch_shape<false, 4, false>(a, nb, stream);
  }
  return key_waves == 4 ? launch_shape<true, 4, false>(a, nb, stream) : launch_shape<true, 2, false>(a, nb, stream);
}

}  // namespace burst
