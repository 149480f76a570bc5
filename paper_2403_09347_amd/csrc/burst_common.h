// Shared device-side helpers for the gfx950 local-attention kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <mutex>
#include "../../include/burst.h"

namespace burst {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
#define BURST_NEG_INF (-__builtin_inff())

// Where the storage-type tensors lie in memory: element strides between batch entries, heads
// and rows of Q, dO, O (query side) and of K, V (key side); the last dimension is contiguous.
// fp32 tensors (state, lse, D, gradients) are always contiguous [B, H, rows, d] / [B, H, rows].
struct Layout {
  long long qs_b, qs_h, qs_r;
  long long ks_b, ks_h, ks_r;
  int heads, kv_heads;             // heads per batch entry on either side
  // element offset of row 0 of a head; `head` counts batch x heads
  __host__ __device__ size_t q_base(int head) const {
    const int b = head / heads;
    return (size_t)b * qs_b + (size_t)(head - b * heads) * qs_h;
  }
  __host__ __device__ size_t kv_base(int kvhead) const {
    const int b = kvhead / kv_heads;
    return (size_t)b * ks_b + (size_t)(kvhead - b * kv_heads) * ks_h;
  }
};

// Row r of the query-side tensors, r counting the rows of all (batch, head)s: element offset.
struct QRows {
  Layout lay;
  int Nq, d, dense;                // dense: contiguous [B, H, Nq, d], the offset is r * d
  __host__ __device__ size_t off(long long r) const {
    if (dense) return (size_t)r * d;
    const long long head = r / Nq;
    return lay.q_base((int)head) + (size_t)(r - head * Nq) * lay.qs_r;
  }
};

// Kernel-side copy of the call's parameters (plain data, passed by value).
struct KParams {
  Layout lay;
  int B, H, Nq, Nc, d;
  int causal;
  float scale;
  long long q_off, k_off;
  long long window;      // 0 = none
  const uint8_t* bmask;  // block mask [ceil(Nq/bsize)][bpitch] (nullptr = none), bpitch = ceil(Nc/bsize)
  int bsize, bpitch;
  long long bhstride;    // bytes between the flag matrices of consecutive (batch, query head)s; 0 = shared
  int group;             // query heads per key/value head (1 = every head has its own K, V)
  QRows q_rows() const {
    QRows q;
    q.lay = lay; q.Nq = Nq; q.d = d;
    q.dense = lay.qs_r == d && lay.qs_h == (long long)Nq * d && lay.qs_b == (long long)Nq * d * H;
    return q;
  }
};

// One key/value chunk of a call, as the kernels see it.  An entry point that is handed several chunks
// passes them to one launch (at most kMaxChunks: they travel in the kernel arguments, which hold 4 KB).
struct Chunk {
  const void* K; const void* V;
  void* dK; void* dV;                // backward only
  const uint8_t* bmask;              // block flags of this chunk (nullptr = none), [ceil(Nq/bsize)][bpitch]
  union {
    long long bhstride;              // bytes between the flag matrices of consecutive query heads (0 = shared)
    struct { int span_lo, span_keys; };   // split dK/dV walks (which have no flags): see RowSpan
  };
  long long k_off;                   // global position of key 0
  long long ks_b, ks_h, ks_r;        // element strides of K and V: batch, head, row
  int Nc, bpitch;
  int first_block;                   // dK/dV kernels: workgroups of the chunks before this one
  // (one word for both, so that a chunk is one and a half cache lines of arguments: with 104 bytes its scalar loads met one more.  dK/dV
  // of 32 heads x 512 causal rows, 16 chunks of 512 keys, where a workgroup goes from block to block, 164 us so, 160 with 96.)
  union {
    int first_row;                   // split dK/dV walks: rows of partial gradients of the chunks before this one
    int order;                       // dK/dV kernels, walks not cut: see grid_order
  };
  // element offset of row 0 of key/value head `kvhead`, which counts batch x heads
  __host__ __device__ size_t kv_base(int kvhead, int kv_heads) const {
    const int b = kvhead / kv_heads;
    return (size_t)b * ks_b + (size_t)(kvhead - b * kv_heads) * ks_h;
  }
};
static_assert(sizeof(Chunk) == 96, "see first_row");
constexpr int kMaxChunks = 32;
// fp32 rows that the generic kernels can bring to LDS: whole 16-byte granules, and 32 rows within a descriptor's 2 GiB.
inline bool fp32_tiles(int d, const Layout& lay, const Chunk* ch, int n) {
  bool ok = d % 4 == 0 && lay.qs_r < (1 << 24);
  for (int i = 0; i < n; i++) ok = ok && ch[i].ks_r < (1 << 24);
  return ok;
}
inline Chunk chunk_of(const KParams& p, const void* K, const void* V, void* dK, void* dV) {
  Chunk c = {};
  c.K = K; c.V = V; c.dK = dK; c.dV = dV;
  c.bmask = p.bmask; c.bhstride = p.bhstride; c.bpitch = p.bpitch;
  c.k_off = p.k_off; c.Nc = p.Nc;
  c.ks_b = p.lay.ks_b; c.ks_h = p.lay.ks_h; c.ks_r = p.lay.ks_r;
  return c;
}
// What a forward (backward) launch reads and writes beside its chunks.
struct FwdIo {
  const void* Q;
  float* O_acc; float* m; float* l;  // running state (nullptr: not kept; `fresh` and O_out only)
  void* O_out; float* lse;           // O_out != nullptr: the state is final after this launch, write these too
  int fresh;                         // the state before the launch is the initial one, whatever the buffers hold
  float* part; int splits;           // splits > 1: partial states of that many key ranges go to `part` instead
  int groups;                        // plain kernels: key groups of a workgroup (0 and 1: one)
};
struct BwdIo {
  const void* Q; const void* dO; const float* lse; const float* D;
  void* dQ;
  int acc_dq, acc_dkv;               // add to what the gradient buffers hold
  int half;                          // dQ, dK, dV are bf16 tensors (the inputs' type) instead of fp32; nothing accumulates then
  float* part; int splits;           // splits > 1: dQ of that many key ranges goes to `part` instead
  const struct RowPlan* parts;       // dK/dV: how the walks are cut (nullptr: not at all)
  const void* O;                     // dQ, plain and generic kernels: D = rowsum(dO o O) is computed and written first (nullptr: it is there)
  int groups;                        // dQ, plain kernels: as in FwdIo
};

// How a dK/dV launch deals out its work.  A workgroup's walk are the query tiles its keys are visible to, of all heads of
// the group: very unequal under a causal mask, and few workgroups where there are few keys.  splits > 1: the
// walk of a block of keys is cut into parts of at most about `tiles` tiles, each a workgroup of its own that leaves fp32
// partial dK, dV in `part` ([part][dK, dV][rows][d]); another launch adds them in a fixed order.  Blocks with one part write
// their gradients themselves: of each chunk the keys from the first to the last block with several have rows there, head
// after head (RowSpan; the kernels have it in the Chunk, whose cache line is there when they need it).
struct RowSpan { int first, lo, keys; };   // a chunk's first row; its keys that have some, of each head
struct RowParts {
  float* part;
  int splits;                        // workgroups per block of keys
  int most, tiles;                   // most parts of a block (<= splits); tiles of a part
  int rows;                          // keys that have rows, of all chunks and heads
  __host__ __device__ int of(int walk) const {
    const int n = (walk + tiles - 1) / tiles;
    return n < 1 ? 1 : n < most ? n : most;
  }
  // where part `i` of key/value head `head` has the keys of a chunk's span
  __device__ float* at(int i, bool dv, const Chunk& C, int head, int d) const {
    return part + ((size_t)(2 * i + dv) * rows + C.first_row + (size_t)head * C.span_keys) * d;
  }
};
struct RowPlan { RowParts parts; RowSpan span[kMaxChunks]; int groups; };   // groups: row groups of a workgroup of the plain kernels, whole walks
// The query tiles (BR rows) of one head that see a key of the block [key0, key0 + BC) of a chunk: [lo, hi).
struct RowRange { int lo, hi; };
__host__ __device__ inline RowRange row_range(int Nq, int causal, long long window, long long q_off, long long k_off, int Nc,
                                              int key0, int BC, int BR) {
  RowRange r = {0, (Nq + BR - 1) / BR};
  if (causal) {                      // rows before the first key see nothing
    const long long first = k_off + key0 - q_off;
    if (first > 0) r.lo = first / BR < r.hi ? (int)(first / BR) : r.hi;
  }
  if (window > 0) {                  // rows too far behind the last key neither
    const long long last = k_off + (key0 + BC < Nc ? key0 + BC : Nc) - 1 + window - 1 - q_off;
    if (last < 0) r.hi = 0;
    else if (last / BR + 1 < r.hi) r.hi = (int)(last / BR) + 1;
  }
  if (r.hi < r.lo) r.hi = r.lo;
  return r;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// The reference maximum of a row in the forward kernels.  Every chunk chooses it anew: the row's maximum in the first
// tile of the chunk in which it sees a key, so that the largest probability there is 1, exact in bf16 (a row that
// sees one key has O = V and lse = its score), and raised to the row's maximum in a later tile that exceeds it by more than
// 2^8.  The bf16 rounding of a chunk's P then depends on that chunk alone, not on the order of the chunks or on
// where the keys are split.  The state in registers is brought to the new reference; where that is lower, only so far
// that the row sum stays below 2^24 (what a chunk that far below the state adds, its rounding cannot change).
// m_st: the reference as it is stored (natural log); log2 units are always m_st x log2 e, so a store and a load in between
// change nothing.  cm: the chunk's reference (log2 units), -inf until the row has seen a key of the chunk.  mx: the row's
// maximum in this tile; l: its sum so far.  Returns the factor of the row's O and l.
// (References on a fixed grid of 16 did as much for the order, but rounded the largest P too: lse of a causal row that
// sees one key was up to 3.8e-3 off, the lse of 4 x 16 heads of 1024 causal rows, d = 64, 3.2e-5 of its norm instead of 2.4e-5.)
__device__ __forceinline__ float raise_reference(float& m_st, float& cm, float mx, float l) {
  float m2 = m_st * kLog2e;
  float to = fmaxf(mx, m2);
  if (cm == BURST_NEG_INF)
    to = mx == BURST_NEG_INF ? m2 : fmaxf(mx, m2 - fminf(fmaxf(24.f - __builtin_amdgcn_logf(l), 0.f), 64.f));
  if (to != m2) m_st = to * kLn2;
  asm volatile("" : "+v"(m_st));                   // (each product rounded by itself, and an unchanged one gives 1)
  float now = m_st * kLog2e;
  asm volatile("" : "+v"(m2), "+v"(now));
  if (mx != BURST_NEG_INF || cm != BURST_NEG_INF) cm = now;
  return fast_exp2(m2 - (now == BURST_NEG_INF ? 0.f : now));       // exp2(-inf) = 0 for a fresh row
}

// s x scale, rounded: the opaque move keeps the compiler from contracting it with a following difference into one fma.
__device__ __forceinline__ float product(float s, float scale) {
  float x = s * scale;
  asm("" : "+v"(x));
  return x;
}
__device__ __forceinline__ float above(float s, float scale, float ref) { return product(s, scale) - ref; }

// Sums whose order the compiler must not change (D has the same bits wherever it is computed).
__device__ __forceinline__ float fma_in_order(float x, float y, float acc) {
  acc = __builtin_fmaf(x, y, acc);
  asm("" : "+v"(acc));
  return acc;
}
__device__ __forceinline__ float add_in_order(float x, float y) {
  x += y;
  asm("" : "+v"(x));
  return x;
}

// raise_reference with everything in natural units (m_st, cm and mx): no product between a score, its maximum and what is stored.
__device__ __forceinline__ float raise_reference_natural(float& m_st, float& cm, float mx, float l) {
  const float was = m_st;
  float to = fmaxf(mx, was);
  if (cm == BURST_NEG_INF)
    to = mx == BURST_NEG_INF ? was : fmaxf(mx, was - fminf(fmaxf(24.f - __builtin_amdgcn_logf(l), 0.f), 64.f) * kLn2);
  m_st = to;
  if (mx != BURST_NEG_INF || cm != BURST_NEG_INF) cm = to;
  return fast_exp2((was - (to == BURST_NEG_INF ? 0.f : to)) * kLog2e);
}

// Workgroup id -> (head, block of the head).  Ids go round-robin to the 8 XCDs; each XCD gets one
// run of consecutive blocks, so that a head's tensors stay in one L2 and all XCDs get the same number
// of workgroups whatever the number of heads.  False: nothing to do (the grid is rounded up to 8).
// order (see grid_order): kByBlock: an XCD takes block 0 of all its heads, then block 1, ... (its heads are whole ones where
// their number is a multiple of 8, else each is spread over several XCDs); kMirror: every other 32 workgroups of an XCD, one
// for each of its CUs, take theirs in reverse.
enum { kByBlock = 1, kMirror = 2 };
__device__ __forceinline__ bool locate_block(int bid, int heads, int blocks, int& head, int& blk, int order = 0) {
  const int total = heads * blocks, per = (total + 7) >> 3, id = bid >> 3;
  int lin = (bid & 7) * per + id;
  // (An order only changes `lin`: with ways of its own to head and block, and out, the compiler moved the kernel's next loads of arguments
  // behind them, one more latency a workgroup of every launch.  dK/dV, d = 128, 16 heads x 1000 rows, 8 chunks of 1000 keys, us, so / here:
  // 136.6 / 134.5, causal with four of the chunks hidden 77.8 / 77.1.)
  if (order != 0 && id < per) {
    const int from = id & ~31, at = (order & kMirror) && (id & 32) ? from + min(from + 32, per) - 1 - id : id;
    const bool own = (heads & 7) == 0;
    const int of = own ? heads >> 3 : heads, of_all = own ? at : 8 * at + (bid & 7);
    const int b = of_all / of, hd = of_all - b * of + (own ? (bid & 7) * of : 0);
    lin = b < blocks ? hd * blocks + b : total;
  }
  if (id >= per || lin >= total) return false;
  head = lin / blocks;
  blk = lin - head * blocks;
  return true;
}
// dK/dV grids hold the workgroups of all chunks, chunk after chunk.  per > 0: every chunk has that many (the
// rule; looking through up to 31 chunks costs a scalar load's latency each).
__device__ __forceinline__ int chunk_at(int bid, const Chunk* ch, int n, int per) {
  if (per > 0) return bid / per;
  int c = 0;
  while (c + 1 < n && bid >= ch[c + 1].first_block) c++;
  return c;
}
// Whether blocks of `br` query rows differ by more than a tenth in the keys they see; the same for blocks of `bc` keys of one chunk.
inline bool unequal_rows(const KParams& p, const Chunk* ch, int n, int br) {
  if (!p.causal) return false;
  auto keys = [&](long long row0, long long row1) {
    long long sum = 0;
    for (int i = 0; i < n; i++) {
      const long long hi = p.q_off + row1 - ch[i].k_off, lo = p.window > 0 ? p.q_off + row0 - p.window + 1 - ch[i].k_off : 0;
      const long long from = lo > 0 ? lo : 0, to = hi < ch[i].Nc ? hi : ch[i].Nc;
      if (to > from) sum += to - from;
    }
    return sum;
  };
  return 10 * keys(p.Nq > br ? p.Nq - br : 0, p.Nq) > 11 * keys(0, br < p.Nq ? br : p.Nq);
}
inline bool unequal_keys(const KParams& p, const Chunk& c, int bc, int br) {
  if (!p.causal || c.Nc == 0) return false;
  const RowRange a = row_range(p.Nq, 1, p.window, p.q_off, c.k_off, c.Nc, 0, bc, br);
  const RowRange b = row_range(p.Nq, 1, p.window, p.q_off, c.k_off, c.Nc, (c.Nc - 1) / bc * bc, bc, br);
  return 10 * (a.hi - a.lo) > 11 * (b.hi - b.lo);
}
// The order in which a grid of heads x blocks workgroups, `fit` to a CU, takes its blocks.  Equal ones go head by head (L2):
// without a causal mask, few rows against many keys (walks of 512 rows x 8192 keys, 0.99 of the time), windows.  Unequal ones
// are numbered longest first by the kernels, and are taken in that order over all heads of
// an XCD: head by head, the second head's longest block starts behind the first one's shortest ones, and the launch ends with
// the last head's long ones on a few CUs.  Causal calls with gradients, us a launch, head by head / by block: d = 64, 128 heads
// x 1024 rows forward 43.5 / 31.0, dQ 57.9 / 44.2, dK/dV 81.9 / 56.2; 32 x 4096 144.7 / 97.0, 176 / 124, 230 / 174; d = 128,
// hand-scheduled, 32 x 4096 forward 205 / 153, dQ 263 / 198, 31 x 3001 118 / 94, 156 / 126, dK/dV 196 / 172; 32 x 8192 (four rounds)
// 559 / 539, 746 / 719.  Head by head also where nothing has to wait (31 x 1000, d = 96, 248 workgroups 36.0 / 37.5), and where a head
// alone has two rounds of blocks for its XCD, so that its short ones end the launch (40 x 16384, 64 blocks, 2522 / 2606).
// Grids of at most `fit` workgroups a CU, all resident from the start, are mirrored besides: in order, a CU's workgroups
// would all be long or all be short.  (Two a CU, d = 64, 64 heads x 1024 rows, 512 workgroups: 108.6 us a call in order, 94.6
// mirrored; d = 96, 32 x 1300, 352: 147 / 125.)
inline int grid_order(long long heads, long long blocks, bool unequal, int fit) {
  if (!unequal || heads * blocks <= 256 || (heads % 8 == 0 && blocks >= 64 * fit)) return 0;
  return heads * blocks <= 256LL * fit ? kByBlock | kMirror : kByBlock;
}
// The order of a chunk's blocks of bc keys in a dK/dV grid of n chunks (each a run of workgroups, none of them mirrored where others follow).  In
// a causal walk of several chunks it is the one on the diagonal that is taken by block.
inline int keys_order(const KParams& p, const Chunk& c, int n, long long heads, int bc, int br, int fit) {
  return grid_order(heads, (c.Nc + bc - 1) / bc, unequal_keys(p, c, bc, br), fit) & (n == 1 ? kByBlock | kMirror : kByBlock);
}
inline long long grid_blocks(long long heads, long long blocks) { return (heads * blocks + 7) / 8 * 8; }
// Workgroup id of a split dK/dV launch -> (head, block of keys, part).  An XCD gets whole (head, part) columns, longest
// block first; which part a column holds turns with the block, so that the XCDs with the high columns are not idle where
// blocks have few parts.  False: nothing to do.
__device__ __forceinline__ bool locate_part(int bid, int heads, int blocks, int splits, int& head, int& blk, int& part) {
  const int cols = heads * splits, per = (cols + 7) >> 3, at = bid >> 3;
  blk = at / per;
  const int col = (bid & 7) * per + at - blk * per;
  if (col >= cols || blk >= blocks) return false;
  head = col / splits;
  part = (col - head * splits + blk) % splits;
  return true;
}
inline long long part_grid(long long heads, long long blocks, int splits) { return (heads * splits + 7) / 8 * 8 * blocks; }
// Lays the chunks' workgroups (`block` keys each) out; returns their number, `per` as chunk_at wants it.
inline long long chunk_grid(Chunk* ch, int n, long long heads, int block, int& per, int splits = 1) {
  auto count = [&](int i) {
    const long long blocks = (ch[i].Nc + block - 1) / block;
    return splits > 1 ? part_grid(heads, blocks, splits) : grid_blocks(heads, blocks);
  };
  long long nb = 0;
  per = n > 0 ? (int)count(0) : 0;
  for (int i = 0; i < n; i++) {
    const long long here = count(i);
    if (here != per) per = 0;
    ch[i].first_block = (int)nb;
    nb += here;
    if (nb > 0x7fffffffLL) break;                  // (the launchers refuse it)
  }
  return nb;
}

// The opt-in to more than 64 KB of dynamic LDS is a per-device function attribute: launchers
// set it once per device (index = current device, or -1 if it cannot be determined), whichever
// host thread comes first.
constexpr int kMaxDevicesForAttr = 64;
inline int current_device_slot() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevicesForAttr) return -1;
  return dev;
}
struct DeviceOnce {
  std::once_flag flag[kMaxDevicesForAttr];
  int status[kMaxDevicesForAttr];
  template <typename F>
  int run(F&& setup) {                       // setup() returns a burst_status; it runs once per device
    const int dev = current_device_slot();
    if (dev < 0) return BURST_ERR_LAUNCH;
    std::call_once(flag[dev], [&] { status[dev] = setup(); });
    return status[dev];
  }
};

// An entry point that enqueues several kernels first walks its launchers with this flag set: they
// validate, set their function attributes and return without launching, so that an error can
// still be reported with nothing enqueued.
extern thread_local bool t_validate_only;
#define BURST_LAUNCH(...)                                          \
  do {                                                             \
    if (!::burst::t_validate_only) hipLaunchKernelGGL(__VA_ARGS__); \
  } while (0)
inline int launch_status() {
  if (t_validate_only) return BURST_OK;
  return hipGetLastError() == hipSuccess ? BURST_OK : BURST_ERR_LAUNCH;
}

// Cross-half exchange.  v_permlane32_swap exchanges the upper 32 lanes of its first operand
// with the lower 32 lanes of its second; fed the same value twice, every lane ends up with
// (value of lane%32, value of lane%32 + 32).  The second operand goes through an opaque
// register copy: the optimizer otherwise treats the swap of two identical values as the
// identity and drops the combination of the two results.
struct HalfPair { float lo, hi; };
__device__ __forceinline__ HalfPair both_halves(float x) {
  int a = __builtin_bit_cast(int, x);
  int b;
  asm volatile("v_mov_b32 %0, %1\n\ts_nop 1" : "=v"(b) : "v"(a));   // nop: VALU write -> permlane read
  auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  HalfPair p;
  p.lo = __builtin_bit_cast(float, (int)r[0]);
  p.hi = __builtin_bit_cast(float, (int)r[1]);
  return p;
}
__device__ __forceinline__ float max_both_halves(float x) {
  HalfPair p = both_halves(x);
  return fmaxf(p.lo, p.hi);
}
__device__ __forceinline__ float sum_both_halves(float x) {
  HalfPair p = both_halves(x);
  return p.lo + p.hi;
}

// LDS tile layout for a [rows][128] bf16 tile: row pitch 256 B, the sixteen 16-byte
// granules of a row are permuted by XOR with a 4-bit code of the row.  The code is a linear
// map over GF(2) of the low four row bits (images 0x7, 0xb, 0x4, 0x9 of bits 0..3), picked by
// an exhaustive search over all 20160 invertible maps, timed on the GPU, for the two access
// patterns of the MFMA operand loads on gfx950: 128-bit reads of one granule column over 32
// consecutive rows (246 B/clk/CU, the LDS peak) and transposing 64-bit reads of 4
// consecutive rows x 2 granules (185 B/clk/CU; a plain bit rotation reaches only 116).
__device__ __forceinline__ int row_code(int row) {
  return ((row & 1) ? 0x7 : 0) ^ ((row & 2) ? 0xb : 0) ^ ((row & 4) ? 0x4 : 0) ^ ((row & 8) ? 0x9 : 0);
}
__device__ __forceinline__ int tile_off(int row, int granule) {
  return row * 256 + ((granule ^ row_code(row)) << 4);
}

__device__ __forceinline__ bf16x8 lds_read_b128(const char* lds, int byte_off) {
  return *reinterpret_cast<const bf16x8*>(lds + byte_off);
}
// Transposing LDS read: within each group of 16 lanes, lane j supplies the address of 4
// consecutive bf16 of matrix row (j/4), columns 4*(j%4)..+3; lane i receives column i of
// rows 0..3.
__device__ __forceinline__ bf16x4 lds_read_tr(const char* lds, int byte_off) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (lds_s16x4*)(__attribute__((address_space(3))) char*)(lds + byte_off));
  return __builtin_bit_cast(bf16x4, v);
}

// Raw buffer access: loads beyond `bytes` return 0 without touching memory, so ragged tile
// tails and prefetches past the end need no branch.  The whole offset goes into the VGPR
// operand (the range check covers it).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ i32x4 buffer_load_b128(__amdgpu_buffer_rsrc_t rsrc, int byte_off) {
  return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, byte_off, 0, 0));
}

// HBM -> LDS DMA: one wave-wide 128-bit buffer load with the LDS modifier.  Lane i's 16
// bytes land at lds_base + 16*i (lds_base wave-uniform, passed through M0); offsets beyond
// the buffer's size write zeros.  Issued as inline assembly on purpose: the compiler then
// does not treat it as an LDS store that every later LDS read must wait for (it would drain
// the whole memory queue before each read).  Ordering against the readers is the caller's
// job: s_waitcnt vmcnt(n) followed by a workgroup barrier.
__device__ __forceinline__ void dma_b128_to_lds(__amdgpu_buffer_rsrc_t rsrc, unsigned lds_base, int voffset) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds_base), "v"(voffset), "s"(rsrc) : "memory", "m0");
}
// Same with 32 bits per lane: lane i's dword lands at lds_base + 4*i.
__device__ __forceinline__ void dma_b32_to_lds(__amdgpu_buffer_rsrc_t rsrc, unsigned lds_base, int voffset) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :: "s"(lds_base), "v"(voffset), "s"(rsrc) : "memory", "m0");
}
// LDS byte address of a pointer into the workgroup's dynamic shared memory.
__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return (unsigned)(size_t)(__attribute__((address_space(3))) const char*)(const char*)p;
}

// MFMA with the accumulator pinned to accumulation registers (AGPRs).  Used for the long-lived
// output accumulators so that the register allocator can never move them through VGPRs.
// As inline assembly the instruction is invisible to the compiler's hazard recognizer:
//  - a VGPR written by a vector instruction must not be read by an MFMA in the next two
//    cycles: the leading s_nop covers the operand copies the compiler may place right before;
//  - the accumulator must not be touched by other instructions until the MFMA has drained:
//    callers go through mfma_acc_fence() before reading or rewriting it.
__device__ __forceinline__ void mfma32_acc(f32x16& acc, bf16x8 a, bf16x8 b) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// Waits until every MFMA issued so far has written its accumulator (an MFMA takes at most
// 16 passes of 4 cycles; 3 x 16 idle cycles cover it with margin) and orders the listed
// accumulators after it.
__device__ __forceinline__ void mfma_acc_fence(f32x16 (&acc)[2][4]) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15"
               : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[0][2]), "+a"(acc[0][3]),
                 "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][2]), "+a"(acc[1][3]));
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

}  // namespace burst
