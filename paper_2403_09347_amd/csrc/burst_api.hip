// C ABI (see include/burst.h): argument validation and dispatch to the kernels.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <exception>
#include <mutex>
#include <vector>
#include "burst_common.h"

namespace burst {
int launch_state_init(const KParams&, float*, float*, float*, hipStream_t);
int launch_finalize(const KParams&, int, const float*, const float*, const float*, void*, float*, hipStream_t);
int launch_merge_state(const KParams&, float*, float*, float*, const float*, const float*, const float*, hipStream_t);
int launch_bwd_prepare(const KParams&, int, const void*, const void*, float*, hipStream_t);
int launch_zero_fill(float*, long long, bool half, hipStream_t);
int launch_fwd_mfma(const KParams&, const FwdIo&, const Chunk*, int, hipStream_t);
int launch_fwd_generic(const KParams&, int, const FwdIo&, const Chunk*, int, hipStream_t);
int launch_bwd_dq_mfma(const KParams&, const BwdIo&, const Chunk*, int, hipStream_t);
int launch_bwd_dkv_mfma(const KParams&, const BwdIo&, const Chunk*, int, hipStream_t, int key_waves);
bool dkv_chained(const KParams&, const Chunk*, int);
int launch_bwd_dq_generic(const KParams&, int, const BwdIo&, const Chunk*, int, hipStream_t);
int launch_bwd_dkv_generic(const KParams&, int, const BwdIo&, const Chunk*, int, hipStream_t);
// the plainly written kernels of burst_plain_mfma.h, one namespace per build
#define BURST_DECLARE_PLAIN(ns)                                                            \
  namespace ns {                                                                           \
  int launch_fwd(const KParams&, const FwdIo&, const Chunk*, int, hipStream_t);            \
  int launch_bwd_dq(const KParams&, const BwdIo&, const Chunk*, int, hipStream_t);         \
  int launch_bwd_dkv(const KParams&, const BwdIo&, const Chunk*, int, hipStream_t);        \
  int dkv_keys();                                                                          \
  int dkv_rows();                                                                          \
  }
int launch_merge_splits(const KParams&, const FwdIo&, hipStream_t);
int launch_fill_unseen(const KParams&, int, void*, float*, hipStream_t);
int launch_sum_splits(const KParams&, const BwdIo&, hipStream_t);
BURST_DECLARE_PLAIN(d64)
BURST_DECLARE_PLAIN(d128p)
BURST_DECLARE_PLAIN(d32x)
BURST_DECLARE_PLAIN(d64x)
BURST_DECLARE_PLAIN(d96x)
BURST_DECLARE_PLAIN(d128x)
#undef BURST_DECLARE_PLAIN
size_t materialized_workspace_bytes(const KParams&, int);
size_t materialized_bwd_workspace_bytes(const KParams&, int);
int launch_bwd_materialized(const KParams&, int, bool, const void*, const void*, const void*, const void*, const float*,
                            const float*, float*, float*, float*, int, int, void*, hipStream_t);
int launch_fwd_materialized(const KParams&, int, bool, const void*, const void*, const void*, float*, float*, float*,
                            void*, hipStream_t);
}  // namespace burst

namespace burst {
thread_local bool t_validate_only = false;
}

namespace {

using burst::KParams;
using burst::Chunk;
using burst::FwdIo;
using burst::BwdIo;

constexpr int kMaxDevices = 64;
int g_arch_ok[kMaxDevices];                 // 0 = unknown, 1 = gfx950, -1 = other
std::mutex g_mutex;

// Library-owned D buffers for burst_local_bwd(D = NULL): one per (device, stream), so that calls on
// different streams never share one.  A buffer that has become too small is replaced by one of at
// least twice its size and is NOT freed: kernels already enqueued may still read it, and hipFree
// would synchronise the device.  The retired blocks stay allocated until the process ends (less
// than the final size in total).  Calls with D = NULL hold g_bwd_mutex from the lookup to the last
// enqueue, so two host threads that share a stream cannot interleave their kernels around the
// shared buffer.
struct DScratch { int dev; hipStream_t stream; float* ptr; size_t elems; };
std::vector<DScratch> g_d_scratch;
std::mutex g_bwd_mutex;

// Static device scratch for burst_local_bwd_static (the entry point for callers that cannot
// allocate): D of one call, BURST_STATIC_MAX_ROWS floats = 8 MiB, held by every GPU the library runs
// on until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; the device address is looked up once per device (each GPU has its own
// copy) and kept here, and that pointer, never the name, is what kernels are given.
static __device__ __align__(256) float scratch[BURST_STATIC_MAX_ROWS];
float* g_static_d[kMaxDevices];
burst::DeviceOnce g_static_d_once;

int static_d_buffer(float** out) {
  const int st = g_static_d_once.run([] {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return (int)BURST_ERR_LAUNCH;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return (int)BURST_ERR_LAUNCH;
    g_static_d[dev] = static_cast<float*>(ptr);
    return (int)BURST_OK;
  });
  if (st != BURST_OK) return st;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BURST_ERR_LAUNCH;
  *out = g_static_d[dev];
  return BURST_OK;
}

int check_arch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BURST_ERR_ARCH;
  std::lock_guard<std::mutex> lock(g_mutex);
  if (g_arch_ok[dev] == 0) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return BURST_ERR_ARCH;
    g_arch_ok[dev] = (std::strncmp(prop.gcnArchName, "gfx950", 6) == 0) ? 1 : -1;
  }
  return g_arch_ok[dev] == 1 ? BURST_OK : BURST_ERR_ARCH;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Validates the parameter block; fills the kernel-side copy.
int check_params(const burst_params* p, KParams* k) {
  if (p == nullptr) return BURST_ERR_NULL;
  if (p->dtype != BURST_BF16 && p->dtype != BURST_F32) return BURST_ERR_DTYPE;
  if (p->B < 1 || p->H < 1 || p->Nq < 0 || p->Nc < 0 || p->d < 1 || p->d > 128) return BURST_ERR_SHAPE;
  if (!(p->scale > 0.f) || !std::isfinite(p->scale)) return BURST_ERR_SHAPE;
  if ((long long)p->B * p->H > 0x7fffffffLL) return BURST_ERR_SHAPE;
  // rows must be addressable with 16-byte aligned row starts for the vector kernels
  k->B = p->B; k->H = p->H; k->Nq = p->Nq; k->Nc = p->Nc; k->d = p->d;
  k->causal = p->causal != 0; k->scale = p->scale; k->q_off = p->q_off; k->k_off = p->k_off;
  if (p->window < 0) return BURST_ERR_SHAPE;
  k->window = p->window;
  k->group = 1;
  if (p->kv_heads != 0) {
    if (p->kv_heads < 0 || p->H % p->kv_heads != 0) return BURST_ERR_SHAPE;
    k->group = p->H / p->kv_heads;
  }
  // strides: all zero = contiguous [B, heads, rows, d]
  {
    const long long hk = p->H / k->group, d = p->d;
    burst::Layout& L = k->lay;
    L.heads = p->H; L.kv_heads = (int)hk;
    const int64_t* q = p->q_strides; const int64_t* kv = p->kv_strides;
    const long long unit = p->dtype == BURST_BF16 ? 8 : 4;     // 16-byte granules
    if (q[0] == 0 && q[1] == 0 && q[2] == 0) {
      L.qs_r = d; L.qs_h = (long long)p->Nq * d; L.qs_b = L.qs_h * p->H;
    } else {
      if (q[0] < 0 || q[1] < 0 || q[2] < d || q[0] % unit || q[1] % unit || q[2] % unit) return BURST_ERR_SHAPE;
      L.qs_b = q[0]; L.qs_h = q[1]; L.qs_r = q[2];
    }
    if (kv[0] == 0 && kv[1] == 0 && kv[2] == 0) {
      L.ks_r = d; L.ks_h = (long long)p->Nc * d; L.ks_b = L.ks_h * hk;
    } else {
      if (kv[0] < 0 || kv[1] < 0 || kv[2] < d || kv[0] % unit || kv[1] % unit || kv[2] % unit) return BURST_ERR_SHAPE;
      L.ks_b = kv[0]; L.ks_h = kv[1]; L.ks_r = kv[2];
    }
  }
  k->bmask = nullptr; k->bsize = 64; k->bpitch = 0; k->bhstride = 0;
  if (p->block_mask != nullptr) {
    if (p->block <= 0 || p->block % 64 != 0) return BURST_ERR_SHAPE;
    k->bmask = p->block_mask; k->bsize = p->block; k->bpitch = (p->Nc + p->block - 1) / p->block;
    k->bhstride = p->block_mask_stride;
    // one matrix per (batch, head): they must not overlap
    const long long matrix = (long long)((p->Nq + p->block - 1) / p->block) * k->bpitch;
    if (k->bhstride != 0 && k->bhstride < matrix) return BURST_ERR_SHAPE;
  }
  return BURST_OK;
}

#define REQUIRE_PTR(ptr)                                 \
  do {                                                   \
    if ((ptr) == nullptr) return BURST_ERR_NULL;         \
    if (!aligned16(ptr)) return BURST_ERR_ALIGN;         \
  } while (0)

// The MFMA kernels address a head's rows through 32-bit byte offsets (plus a few tiles of
// prefetch past the end); longer or wider-strided slices or chunks take the generic kernels.  So do
// groups whose heads together span more than 4 GiB: no kernel needs that limit since dK/dV has a
// descriptor per head, but these calls have the 24-bit probabilities of the generic kernels and keep them.
constexpr int kMaxMfmaRows = 4 * 1024 * 1024;
bool spans_fit(const burst_params* p, const KParams& k) {
  const long long q = ((long long)p->Nq + 1024) * k.lay.qs_r * 2 + (long long)(k.group - 1) * k.lay.qs_h * 2;
  const long long kv = ((long long)p->Nc + 1024) * k.lay.ks_r * 2;
  return q <= 0xffffffffLL && kv <= 0xffffffffLL;
}
// With block flags the MFMA kernels keep a list of visible tiles in LDS (8192 tiles of 64 keys or
// rows, or 16384 of 32 keys): longer masked slices or chunks take the generic kernels.
constexpr int kMaxMaskedRows = 8192 * 64;
bool use_mfma(const burst_params* p, const KParams& k) {
  return p->dtype == BURST_BF16 && p->d == 128 && p->Nq <= kMaxMfmaRows && p->Nc <= kMaxMfmaRows && spans_fit(p, k);
}
// bf16 with another head dimension than 128: the plainly written kernels, built for d = 64 and, for
// every other multiple of 8, at the next of the padded widths 32, 64, 96, 128 (their DMA descriptors
// must span less than 2 GiB, see s_dma_off).  Null where the generic kernels have to do it: rows that
// do not start on 16 bytes, sizes beyond the 32-bit addressing.  (d = 96, 32 heads of 777 causal rows,
// differentiable call with its gradients: 1375 us on the generic kernels, 121 us padded, with the same fp32
// probabilities, see s_terms.)
struct PlainFamily {
  decltype(&burst::d64::launch_fwd) fwd;
  decltype(&burst::d64::launch_bwd_dq) bwd_dq;
  decltype(&burst::d64::launch_bwd_dkv) bwd_dkv;
  decltype(&burst::d64::dkv_keys) dkv_keys, dkv_rows;
};
#define BURST_PLAIN(ns) {burst::ns::launch_fwd, burst::ns::launch_bwd_dq, burst::ns::launch_bwd_dkv, burst::ns::dkv_keys, burst::ns::dkv_rows}
const PlainFamily kD64 = BURST_PLAIN(d64), kD128p = BURST_PLAIN(d128p), kD32x = BURST_PLAIN(d32x), kD64x = BURST_PLAIN(d64x), kD96x = BURST_PLAIN(d96x),
                  kD128x = BURST_PLAIN(d128x);
#undef BURST_PLAIN
const PlainFamily* plain_family(const burst_params* p, const KParams& k) {
  if (p->dtype != BURST_BF16 || p->d == 128 || p->d % 8 != 0 || p->Nq > kMaxMfmaRows || p->Nc > kMaxMfmaRows ||
      !spans_fit(p, k)) return nullptr;
  if (p->block_mask != nullptr) {
    // with block flags: lists of at most 4096 tiles (32 keys or rows each; rows of all heads of a group)
    const long long group = (p->kv_heads > 0) ? p->H / p->kv_heads : 1;
    if (p->Nc > 4096 * 32 || group * ((p->Nq + 31) / 32) > 4096) return nullptr;
  }
  if (p->d == 64) return &kD64;
  if (((long long)p->Nq + 1024) * k.lay.qs_r * 2 > 0x7fffffffLL || ((long long)p->Nc + 1024) * k.lay.ks_r * 2 > 0x7fffffffLL)
    return nullptr;
  return p->d <= 32 ? &kD32x : p->d <= 64 ? &kD64x : p->d <= 96 ? &kD96x : &kD128x;
}
// The forward and dQ kernels for d = 128 run one 256-row workgroup per CU, so a call takes
// ceil(workgroups / 256) rounds on the chip's 256 CUs.  When the last round is at most half full
// (short query slices, or a workgroup count just above a multiple of 256) the plainly written
// kernels with 128 rows per workgroup and two workgroups per CU do better: 1.3-1.5x (forward)
// and 1.1-1.25x (backward) at up to 128 workgroups, 15 % at 320, 3-6 % (forward) at 384 .. 1152;
// they lose 3-6 % where the rounds are full, and the gain fades as the rounds grow in number.
std::atomic<int> g_kernel_family{0};            // burst_set_kernel_family
// A causal walk of one chunk (`whole`) has long and short workgroups besides, and the small ones are dealt out more evenly: us,
// hand-scheduled / plain, forward and dQ, 64 x 777 rows (256 workgroups) 36 / 24 and 43 / 31, 64 x 1024 44 / 31, 52 / 40, 16 x 4096
// 113 / 89, 146 / 117, 8 x 8192 206 / 165, 273 / 220; up to 512 workgroups 128 x 1024 71 / 55, 82 / 70, 64 x 2048 95 / 85, 116 / 115,
// but 40 x 3001 117 / 110, 148 / 152, 32 x 4096 148 / 150, 194 / 207.
bool use_plain128(const burst_params* p, const KParams& k, bool whole = false) {
  if (!use_mfma(p, k)) return false;
  const bool flags = p->block_mask != nullptr;
  if (flags && p->Nc > 4096 * 32) return false;    // their tile lists hold 4096 entries (32-key tiles in dQ)
  const int family = g_kernel_family.load(std::memory_order_relaxed);
  if (family != 0) return family == 2;
  // Block flags finer than the 256-row workgroups of the list-driven kernels: the plain kernels
  // skip per wavefront (32 rows x 64 or 32 keys), which is what such patterns need.
  if (flags) return p->block < 256;
  const long long wgs = (long long)p->B * p->H * ((p->Nq + 255) / 256);
  if (whole && wgs <= (p->Nq <= 2048 ? 512 : 256)) {
    const Chunk c = burst::chunk_of(k, nullptr, nullptr, nullptr, nullptr);
    if (burst::unequal_rows(k, &c, 1, 128)) return true;
  }
  const long long last = wgs % 256;                // workgroups of the last round (0 = full)
  return last != 0 && last <= 128 && wgs <= 1536;
}
// The hand-scheduled dK/dV kernel walks the query tiles of all heads of a group as one list of at most 8192
// tiles; longer groups take the generic kernel.  Groups whose slice is no multiple of its 64-row tiles go to the
// plain kernel padded to 128 columns, whose P and dS have 24 bits as in the generic kernel that had these calls (see
// s_terms).  (Call with gradients, 32 heads over 8, 3001 causal rows: 518 us, 1054 with
// two wavefronts a workgroup, 10.3 ms with the generic kernel; with 8-bit P and dS a walk's dV is 1.7e-3 off 64 bits instead of 7.6e-5.)
bool dkv_mfma_ok(const burst_params* p, const KParams& k) {
  if (k.group > 1) return p->Nq % 64 == 0 && (long long)k.group * (p->Nq / 64) <= 8192 && k.group <= 256;
  return p->block_mask == nullptr || p->Nq <= kMaxMaskedRows;
}
bool use_padded128_dkv(const burst_params* p, const KParams& k) {
  if (!use_mfma(p, k) || k.group == 1 || p->Nq % 64 == 0) return false;
  return p->block_mask == nullptr || (long long)k.group * ((p->Nq + 31) / 32) <= 4096;   // (its tile list)
}

// Entry points that enqueue several kernels: one pass over the launchers in validate-only mode
// (shape limits, function attributes), so that an error is reported with nothing enqueued, then
// the real pass.
template <typename F>
int validated(F&& enqueue) {
  burst::t_validate_only = true;
  const int e = enqueue();
  burst::t_validate_only = false;
  return e != BURST_OK ? e : enqueue();
}

// Block flags narrower than the 128 keys of a dK/dV workgroup: the hand-scheduled kernel runs in
// its shape with 64-key workgroups, whose tile lists hold what 64 keys need (its time then
// follows the density; a 128-key workgroup cannot skip what only half of its keys need).  Those
// lists hold 2048 entries of 64 query rows (all heads of a group).
int dkv_key_waves(const burst_params* p, const KParams& k) {
  if (p->block_mask == nullptr || p->block >= 128) return 4;
  if ((long long)k.group * ((p->Nq + 63) / 64) > 2048) return 4;
  return g_kernel_family.load(std::memory_order_relaxed) == 0 ? 2 : 4;
}
// The plainly written dK/dV kernel with 64-key workgroups runs when the plain family is forced.
// Its tile lists hold 4096 entries of 32 query rows (all heads of a group).
bool use_plain128_dkv(const burst_params* p, const KParams& k) {
  if (!use_mfma(p, k)) return false;
  const bool flags = p->block_mask != nullptr;
  if (flags && (long long)k.group * ((p->Nq + 31) / 32) > 4096) return false;
  return g_kernel_family.load(std::memory_order_relaxed) == 2;
}

// The kernels that serve one chunk's forward, dQ or dK/dV: one of the plainly written families
// (which take several chunks in one launch), the hand-scheduled d = 128 kernels, or the generic ones.
struct Kernels {
  const PlainFamily* plain;
  bool hand;
  int key_waves;                                   // hand-scheduled dK/dV
  int takes;                                       // most chunks of one launch (hand-scheduled: of one row pitch)
  bool operator==(const Kernels& o) const { return plain == o.plain && hand == o.hand && key_waves == o.key_waves && takes == o.takes; }
};
Kernels fwd_kernels(const burst_params* p, const KParams& k, bool whole = false) {      // dQ: the same choice
  if (const PlainFamily* f = plain_family(p, k)) return {f, false, 0, burst::kMaxChunks};
  if (use_plain128(p, k, whole)) return {&kD128p, false, 0, burst::kMaxChunks};
  const bool hand = use_mfma(p, k) && (p->block_mask == nullptr || p->Nc <= kMaxMaskedRows);
  return {nullptr, hand, 0, hand && p->block_mask != nullptr ? 1 : burst::kMaxChunks};
}
Kernels dkv_kernels(const burst_params* p, const KParams& k) {
  if (const PlainFamily* f = plain_family(p, k)) return {f, false, 0, burst::kMaxChunks};
  if (use_plain128_dkv(p, k)) return {&kD128p, false, 0, burst::kMaxChunks};
  if (use_padded128_dkv(p, k)) return {&kD128x, false, 0, burst::kMaxChunks};
  const bool hand = use_mfma(p, k) && dkv_mfma_ok(p, k);
  return {nullptr, hand, hand ? dkv_key_waves(p, k) : 0, burst::kMaxChunks};
}
int fwd_launch(const Kernels& f, const KParams& k, int dtype, const FwdIo& io, const Chunk* c, int n, hipStream_t s) {
  if (f.plain != nullptr) return f.plain->fwd(k, io, c, n, s);
  if (f.hand) return burst::launch_fwd_mfma(k, io, c, n, s);
  return burst::launch_fwd_generic(k, dtype, io, c, n, s);
}
int dq_launch(const Kernels& f, const KParams& k, int dtype, const BwdIo& io, const Chunk* c, int n, hipStream_t s) {
  if (f.plain != nullptr) return f.plain->bwd_dq(k, io, c, n, s);
  if (f.hand) return burst::launch_bwd_dq_mfma(k, io, c, n, s);
  return burst::launch_bwd_dq_generic(k, dtype, io, c, n, s);
}
int dkv_launch(const Kernels& f, const KParams& k, int dtype, const BwdIo& io, const Chunk* c, int n, hipStream_t s) {
  if (f.plain != nullptr) return f.plain->bwd_dkv(k, io, c, n, s);
  if (f.hand) return burst::launch_bwd_dkv_mfma(k, io, c, n, s, f.key_waves);
  return burst::launch_bwd_dkv_generic(k, dtype, io, c, n, s);
}

// A walk over several chunks: the chunks (without the empty ones), each with its own parameter block.
struct WalkChunk { burst_params p; KParams k; Chunk c; };
int walk_chunks(const burst_chunk* chunks, int n, const burst_params* p, bool backward, std::vector<WalkChunk>& out) {
  if (n < 0) return BURST_ERR_SHAPE;
  if (n > 0 && chunks == nullptr) return BURST_ERR_NULL;
  if (p == nullptr) return BURST_ERR_NULL;
  try { out.reserve((size_t)n); } catch (const std::exception&) { return BURST_ERR_ALLOC; }   // (nothing is thrown through the C ABI)
  for (int i = 0; i < n; i++) {
    const burst_chunk& in = chunks[i];
    WalkChunk w;
    w.p = *p;
    w.p.Nc = in.Nc; w.p.k_off = in.k_off; w.p.block_mask = in.block_mask; w.p.block_mask_stride = in.block_mask_stride;
    std::memcpy(w.p.kv_strides, in.kv_strides, sizeof w.p.kv_strides);
    const int st = check_params(&w.p, &w.k);
    if (st != BURST_OK) return st;
    if (in.Nc == 0) continue;
    REQUIRE_PTR(in.K); REQUIRE_PTR(in.V);
    if (backward) { REQUIRE_PTR(in.dK); REQUIRE_PTR(in.dV); }
    w.c = burst::chunk_of(w.k, in.K, in.V, in.dK, in.dV);
    out.push_back(w);
  }
  return BURST_OK;
}
// Calls launch(kernels, first chunk, chunks, is first, is last) for every run of chunks that one launch can take.
template <typename Choose, typename Launch>
int for_each_run(const std::vector<WalkChunk>& w, Choose choose, Launch launch) {
  const size_t n = w.size();
  for (size_t i = 0; i < n;) {
    const Kernels f = choose(&w[i].p, w[i].k);
    Chunk run[burst::kMaxChunks];
    size_t m = 0;
    do { run[m] = w[i + m].c; m++; }
    while (m < (size_t)f.takes && i + m < n && (w[i + m].c.bmask == nullptr) == (run[0].bmask == nullptr) &&
           (!f.hand || w[i + m].c.ks_r == run[0].ks_r) && choose(&w[i + m].p, w[i + m].k) == f);
    const int st = launch(f, w[i].k, run, (int)m, i == 0, i + m == n);
    if (st != BURST_OK) return st;
    i += m;
  }
  return BURST_OK;
}

// Caller holds g_bwd_mutex.
int get_d_scratch(hipStream_t stream, size_t elems, float** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return BURST_ERR_ALLOC;
  DScratch* slot = nullptr;
  for (DScratch& e : g_d_scratch)
    if (e.dev == dev && e.stream == stream) slot = &e;
  if (slot == nullptr) {
    g_d_scratch.push_back(DScratch{dev, stream, nullptr, 0});
    slot = &g_d_scratch.back();
  }
  if (slot->elems < elems) {
    const size_t want = elems > 2 * slot->elems ? elems : 2 * slot->elems;
    float* ptr = nullptr;
    if (hipMalloc(&ptr, want * sizeof(float)) != hipSuccess) return BURST_ERR_ALLOC;
    slot->ptr = ptr;                               // the old block, if any, is retired, not freed
    slot->elems = want;
  }
  *out = slot->ptr;
  return BURST_OK;
}

// The choice for a walk's forward and dQ launches.  `whole`: one chunk, and neither a state nor fp32 gradients that a caller could
// go on with chunk by chunk.  Other walks have the bits that they have chunk by chunk where they are not split.
auto walk_choice(bool whole) {
  return [whole](const burst_params* p, const KParams& k) { return fwd_kernels(p, k, whole); };
}

// Walks of the generic kernels that can be split: fp32 through LDS, no flags.
bool generic_splittable(const std::vector<WalkChunk>& w) {
  if (w[0].p.dtype != BURST_F32) return false;
  for (const WalkChunk& x : w) if (x.p.block_mask != nullptr || !burst::fp32_tiles(x.k.d, x.k.lay, &x.c, 1)) return false;
  return true;
}
// Into how many workgroups the tiles of a block of 32 rows are dealt.  Up to 128 blocks as many as there are CUs for (they run at the fp32
// matrix rate with one wavefront per SIMD, so that more gain nothing), with a tile for each of their four wavefronts.
// us a launch with its merge, whole / by the rule, forward and dQ: 256 rows x 1024 keys, one head, d = 64, 32 / 15 and 40 / 16
// in 8; 4 x 1000 x 3000, d = 64, 82 / 53 and 111 / 63 in 2 (3: 66, 85; 4: 56, 72); 4 x 700 x 1400, d = 128, 70 / 48 and 102 / 68
// in 2 (3: 57, 79); 8 x 300 x 600 causal, d = 80, 30 / 21 and 38 / 26 in 3 (4: 31, 32); not split: 8 x 700 x 1400 causal 71 and
// 103 (2: 69, 97; 3: 73, 101), 8 x 1000 x 4000, d = 32, 67 and 82 (2: 72, 84).
// The merging launch takes 4 us of the GPU and 4 of the host, twice in a pass with gradients, whose host needs about 36 us and 6 a chunk
// however short the walk is.  At up to 64 columns short walks are therefore whole (a workgroup then has eight wavefronts).  A pass
// with gradients, whole / split, us: d = 32, one head, 450 x 450 (15 tiles) 46 / 57, 192 rows x 1130 keys (36) 54 / 53, 256 x 1300 (41)
// 61 / 53; four chunks of 256 (32) 62 / 76, of 320 (40) 63 / 76, of 410 (52) 74 / 76, eight heads 83 / 79; d = 64, 300 x 300 (10) 60 / 61, three
// chunks of 128 (12) 55 / 69, 416 x 416 (13) 67 / 58.
int generic_splits(const std::vector<WalkChunk>& w) {
  const KParams& k = w[0].k;
  const long long heads = (long long)k.B * k.H, blocks = (k.Nq + 31) / 32;
  const bool many = heads * blocks > 128;
  if (heads * blocks > (k.d <= 64 ? 128 : 1024) || !generic_splittable(w)) return 1;
  long long most = 0, least = 0x7fffffff, sum = 0; // key tiles that a block sees
  for (long long row0 = 0; row0 < k.Nq; row0 += 32) {
    long long walk = 0;
    for (const WalkChunk& x : w) {
      long long lo = 0, hi = x.c.Nc;
      if (k.causal) hi = std::min(hi, k.q_off + std::min<long long>(row0 + 32, k.Nq) - x.c.k_off);
      if (k.window > 0) lo = std::max(lo, k.q_off + row0 - k.window + 1 - x.c.k_off);
      if (hi > lo) walk += (hi + 31) / 32 - lo / 32;
    }
    most = std::max(most, walk);
    least = std::min(least, walk);
    sum += walk;
  }
  // More than 128 blocks, above 64 columns (a workgroup a CU): in two where that ends sooner, counted in tiles of a wavefront, with 3
  // a workgroup beside its tiles and 2 for the merge.  Unequal blocks fill the CUs but for half of a long one at the end, equal ones
  // come in rounds.  us, forward and dQ with merging, whole / in 2, d = 128: 4 x 1400 x 2800 causal, 176 blocks, 283 / 244;
  // 8 x 1500, third of three causal chunks, 376 blocks, 700 / 627; equal blocks: 8 x 1100 x 2200, 280 of them, 460 / 395, 8 x 1500 x
  // 6000, 376, 1115 / 903.  Not split: 8 x 700 x 1400 causal 162 / 161, 8 x 1000 x 2000 causal 212 / 212, 8 x 1400 causal 153 / 196,
  // 8 x 600 x 1200 141 / 174.
  if (many) {
    const double B = (double)(heads * blocks), all = (double)(sum * heads);
    auto cost = [&](int s) {
      const double longest = most / (4.0 * s);
      if (10 * most <= 11 * least) return std::ceil(B * s / 256) * (longest + 3) + (s > 1 ? 2 : 0);
      return std::max(longest + 3, all / 1024 + 3 * B * s / 256 + longest / 2) + (s > 1 ? 2 : 0);
    };
    return cost(2) < 0.97 * cost(1) ? 2 : 1;
  }
  const long long s = std::min({256 / (heads * blocks), most / 4, 64LL});
  const long long others = (long long)w.size() - 1;
  return s < 2 || most < (k.d <= 32 ? 36 + 4 * others : k.d <= 64 ? 13 + 2 * others : 0) ? 1 : (int)s;
}
// Into how many key ranges a walk of the plain kernels is split (1: not at all).  Their workgroups hold
// 128 rows and two share a CU: 512 fill every place on the chip, and with 256 or fewer two ranges or more have places
// of their own.  Ranges shorter than 8 tiles would spend their time on the partial states.  Walks of fewer than
// 20 tiles are not split, so that short ones keep the bits they have chunk by chunk: that gives up a quarter of the time just
// below the line (8 x 384 rows, forward, without / with a split: 512 keys 19.5 / 20.1 us in 2; 1024 keys 28 / 21; 1536 keys,
// 24 tiles, split by the rule, 36 / 22 in 3).  Forward, us, without / with the split this rule picks, in brackets one half or
// twice as many: 32 heads x 40 rows x 32K keys 597 / 116 in 16 (8: 120, 24: 134); 32 x 512 x 8K causal 168 / 95 in 4
// (2: 106, 8: 108); 8 x 100 x 4K, d = 64, 63 / 24 in 8 (4: 28, 16: 22); 8 x 1024 x 4K 85 / 38 in 8
// (4: 39, 16: 52); backward (dQ) 32 x 512 x 8K 664 / 585, 8 x 1024 x 4K 257 / 191.
//
// Key groups: a workgroup's four wavefronts own 128 rows, or 64 rows and a half of every tile's keys each (`groups` = 2, see
// burst_plain_mfma.h): twice the workgroups, half as long, for twice the traffic into LDS.  A `whole` walk (see walk_choice) that is not
// split has two where its workgroups of 128 rows are few, or unequal and not too many (LDS rows of 128 bytes: four
// of 64 rows share a CU, of 256 bytes: two).  Forward + dQ, us, one / two groups, causal: d = 64, 8 x 512 rows (32 workgroups of
// 128) 31 / 23, 32 x 1000 (256) 49 / 37, 64 x 1024 (512) 56 / 46, 40 x 2048 (640) 96 / 92, 96 x 1024 (768) 64 / 67, 16 x 8192 (1024)
// 407 / 396, 64 x 4096 (2048) 382 / 409; d = 40, 24 x 4096 (768) 293 / 251, 128 x 1024 (1024) 112 / 111; d = 96, 32 x 777 (224) 68 /
// 51, 48 x 1024 (384) 84 / 76, 80 x 700 (480) 64 / 69, 16 x 4000 (512) 293 / 274, 128 x 1024 (1024) 157 / 169; d = 128, 32 x 1000
// (256) 65 / 49, 24 x 2048 (384) 110 / 93, 64 x 1024 (512) 71 / 79, 16 x 4096 (512) 213 / 206; without a mask: d = 64, 20 x 2048
// (320) 100 / 84, 48 x 1024 (384) 60 / 53, 64 x 1024 (512) 65 / 67; d = 96, 24 x 1024 (192) 79 / 69, 40 x 777 (280) 94 / 94; d =
// 128, 32 x 1000 (256) 66 / 61.
// Such a walk is split only where that is worth the merging launches: from 32 tiles on (24 on the padded kernels), as many
// ranges as its workgroups have places for (forward + dQ with merging and D, us, whole / split: d = 64, 8 x 1500 42 / 40,
// 8 x 2048 53 / 46, 16 x 2048 56 / 58, 8 x 4000 92 / 79; d = 96, 16 x 1000 54 / 54, 8 x 2048 89 / 71, 12 x 2048 91 / 89; d = 128,
// 8 x 1500 58 / 58, 8 x 2048 74 / 65, 12 x 2048 75 / 82).
// Split walks have two groups too where their workgroups of 128 rows are at most one a CU, or where 64 rows less a head are a good part
// of it (passes of 4 x 1698 keys, us, one / two: d = 64, 80 x 162 rows 238 / 223, 48 x 290 213 / 199, 40 x 418 223 / 226, 16 x 1058 214 / 216;
// d = 48, 80 x 162 331 / 294, 40 x 418 329 / 334, 16 x 1058 331 / 336).
// (forward, us: d = 64, 32 over 8 x 16 rows x 16K keys 40 / 31, 80 over 20 x 150 x 8K 76 / 64, 8 x 100 x 8K 26 / 22, 32 x 200 x 64K
// 188 / 221 (one); d = 128, 32 over 2 x 5 x 64K 145 / 99, 80 over 20 x 150 x 8K 107 / 114 (one), 32 x 200 x 64K 309 / 413 (one)).
struct RowsPlan { int splits, groups; };
RowsPlan walk_rows(const std::vector<WalkChunk>& w, bool backward, bool whole) {
  if (w.empty() || w[0].k.Nq == 0 || w.size() > (size_t)burst::kMaxChunks) return {1, 1};
  const Kernels f = fwd_kernels(&w[0].p, w[0].k, whole);
  if (f.plain == nullptr) return {generic_splits(w), 1};
  const KParams& k = w[0].k;
  const bool wide = f.plain == &kD96x || f.plain == &kD128x || f.plain == &kD128p;
  const bool padded = f.plain != &kD64 && f.plain != &kD128p;
  const long long blocks = (long long)k.B * k.H * ((k.Nq + 127) / 128);
  long long tiles = 0;                             // of 64 keys, that the last rows see
  for (const WalkChunk& x : w) {
    if (x.p.block_mask != nullptr || !(fwd_kernels(&x.p, x.k, whole) == f)) return {1, 1};
    long long lo = 0, hi = x.c.Nc;
    if (k.causal) hi = std::min(hi, k.q_off + k.Nq - x.c.k_off);
    if (k.window > 0) lo = std::max(lo, k.q_off + k.Nq - 128 - k.window + 1 - x.c.k_off);
    if (hi > lo) tiles += (hi - lo + 63) / 64;
  }
  const bool unequal = whole && burst::unequal_rows(k, &w[0].c, 1, 128);
  auto unsplit = [&]() -> RowsPlan {
    bool two;
    if (!wide) two = blocks <= (!unequal ? 448 : padded ? 896 : k.Nq >= 4096 ? 1024 : 640);
    else two = unequal ? blocks <= 352 || (blocks <= 448 && padded && k.Nq >= 1000) || (blocks <= 512 && k.Nq >= 2048) : blocks <= 224;
    return {1, whole && two ? 2 : 1};
  };
  if (whole && blocks > 32 && (backward || !padded)) {
    const long long s = std::min((wide ? 256 : 512) / blocks, tiles / 8);
    if (s >= 2 && tiles >= (padded ? 24 : 32)) return {(int)s, unequal || blocks * s <= 256 ? 2 : 1};
    return unsplit();
  }
  // The padded kernels' tiles take twice the time: up to 160 blocks 6 of them are a range, and walks of 12 are split (d = 96, causal,
  // whole / split, forward and backward pass, us: 16 x 900, 128 blocks, in 2 32.8 / 29.3, 99 / 95; 16 x 1216, 160, in 3 39.9 / 36.8,
  // 124 / 120; 15 x 1130, 135, in 3 38.4 / 35.6, 120 / 113).  A few workgroups more than CUs cost as much as another round of them
  // (forward, d = 96, in 2 / 3: 100 x 100 rows x 1200 keys, 300, 31.7 / 33.6; 12 x 1200 x 1200, 360, 35.8 / 39.0; 3840 causal rows
  // in 8 / 10 (300) 30.0 / 33.9; whole / in 2: 17 x 1024, 272, 35.0 / 36.4; 20 x 1000, 320, 35.2 / 37.3): then as many ranges as
  // there are CUs for.  Halfway to two a CU it pays again under a causal mask (8 x 1500, in 2 / 4, 384, 37.2 / 32.1) and where the
  // alternative is one range (130 x 100 rows x 1200 keys, in 1 / 3, 42.0 / 34.6); walks of equal length later (d = 32, 8 x 958 x 2268, in 4 / 6,
  // 24.5 / 27.6; d = 96, 8 x 1500 in 2 / 4 37.7 / 38.9).  From 161 blocks on as elsewhere
  // (24 x 1000, 192, in 2: 35.3 / 40.4, not split).
  const bool pad = padded && blocks <= 160;
  long long s = std::min(512 / blocks, tiles / (pad ? 6 : 8));
  if (pad && s * blocks > 256 && s * blocks <= (k.causal || blocks > 128 ? 360 : 400)) s = 256 / blocks;
  if (s < 2 || tiles < (pad ? 12 : 20)) return unsplit();
  return {(int)s, s * blocks <= 256 || k.Nq <= 64 || (!wide && k.Nq <= 320 && (k.Nq - 1) % 128 < 64) ? 2 : 1};
}
int dq_launches(const std::vector<WalkChunk>& w, bool whole) {
  int n = 0;
  for_each_run(w, walk_choice(whole), [&](const Kernels&, const KParams&, const Chunk*, int, bool, bool) { n++; return (int)BURST_OK; });
  return n;
}
// How the dK/dV launch of a walk is cut (RowParts; splits = 1: not at all).  Few or unequal walks leave most of the chip idle:
// under a causal mask the longest is twice the average, and with grouped heads there are few blocks of keys.  A block's walk
// is therefore cut into about as many parts as the longest walk exceeds the work of one place on the chip (two workgroups
// of the plain kernels share a CU), of at least 256 (hand-scheduled: 1024) rows, below which the partial results cost what
// the balance gains.  Equal parts for short and long blocks (down to 8 tiles) do better than parts of equal length, because
// the launch then ends with small ones.  Below a ratio of 1.9 a launch that fills the chip loses.  Walks of fewer than 24
// tiles (hand-scheduled: 32) keep the bits they have chunk by chunk.  Causal calls with gradients, us, whole / by the rule, in
// brackets one part less and more: 32 heads over 8 x 3001 rows 1055 / 633 in 3 (690, 636), x 3008 564 / 440 in 3 (448, 445);
// 32 over 8 x 2048, d = 64, 354 / 156 in 8 (153 in 6, 167 in 12); 8 over 2 x 1000 332 / 98 in 16 (101 in 12); 8 x 3000, d = 64,
// 174 / 124 in 5 (123, 124); 32 x 777, d = 96, 123 / 107 in 3 (111, 117); 8 x 8000, d = 64, 511 / 443 in 2 (447 in 3); not
// cut: 64 x 1024, d = 64, 98 (in 2: 112), 16 x 3000 279 (301), 16 x 4096 403 (440).
// Partial gradients have room for the keys of a chunk from its first block with several parts to its last: hidden chunks and
// the short ends of masked ones take none.
// Row groups: a whole walk (see walk_choice) on the plain kernels of four wavefronts may have workgroups of 64 keys instead, two halves of every
// tile's rows each (see burst_plain_mfma.h).  They take the place of the parts, whose launch and traffic they save, where
// there are blocks enough: us, whole or parts with their merge / row groups, causal: d = 64, 8 x 1000 (64 blocks of 128 keys) 20.5 / 19.5,
// 8 x 2048 (128) 37 / 35, 8 x 4000 (256) 61 / 65 (parts), 32 x 1000 (256) 35 / 22, 64 x 1024 (512) 39 / 34, 24 x 4096 (768) 136 / 131,
// 32 x 4096 (1024) 171 / 177; d = 96, 8 x 1000 (64) 31 / 36 (parts), 16 x 777 (112) 33 / 32, 8 x 2048 (128) 62 / 68 (parts), 32 x 777
// (224) 43 / 35, 20 x 2048 (320) 103 / 82, 16 x 4000 (512) 257 / 219, 64 x 2048 (1024) 226 / 216; without a mask: d = 64, 8 x 4096
// (256) 121 / 87, 48 x 1024 (384) 43 / 41, 64 x 1024 (512) 46 / 49; d = 96, 24 x 1024 (192) 72 / 53, 64 x 1024 (512) 106 / 111.
constexpr burst::RowPlan kWhole = {{nullptr, 1, 1, 1, 0}, {}, 1};
// Workgroups per block for at most `most` parts: whole (head, part) columns go to the 8 XCDs, so their number should be a
// multiple of 8 (workgroups without a part end at once).
int part_columns(long long heads, long long most) {
  for (long long s = most; s < most + 8; s++) if (heads * s % 8 == 0) return (int)s;
  return (int)most;
}
burst::RowPlan cut_walks(const std::vector<WalkChunk>& w) {
  if (w.empty() || w[0].k.Nq == 0 || w.size() > (size_t)burst::kMaxChunks) return kWhole;
  const Kernels f = dkv_kernels(&w[0].p, w[0].k);
  if (f.plain == &kD128p) return kWhole;           // (it runs only when its family is forced)
  const KParams& k = w[0].k;
  const bool generic = f.plain == nullptr && !f.hand;
  if (generic && !generic_splittable(w)) return kWhole;
  const int bc = generic ? 32 : f.plain != nullptr ? f.plain->dkv_keys() : 128, br = f.hand ? 64 : generic ? 32 : f.plain->dkv_rows();
  const int unit = f.plain != nullptr ? br / 32 : 1;   // (the plain kernels' thresholds count tiles of 32 rows)
  const long long heads = (long long)k.B * k.H / k.group, slots = f.plain != nullptr && br == 32 ? 512 : 256;   // (generic: the CUs)
  if ((long long)k.group * ((k.Nq + br - 1) / br) * unit < (generic ? 8 : f.hand ? 32 : 24)) return kWhole;   // (no walk is long enough, see below)
  auto walk_of = [&](const WalkChunk& x, int key0) {   // tiles of a block of keys, of all heads of the group
    const burst::RowRange r = burst::row_range(k.Nq, k.causal, k.window, k.q_off, x.c.k_off, x.c.Nc, key0, bc, br);
    return (long long)(r.hi - r.lo) * k.group;
  };
  long long total = 0, most = 0, blocks = 0;
  for (const WalkChunk& x : w) {
    if (x.p.block_mask != nullptr || !(dkv_kernels(&x.p, x.k) == f) || (f.hand && x.c.ks_r != w[0].c.ks_r)) return kWhole;
    blocks += heads * ((x.c.Nc + bc - 1) / bc);
    if (blocks > 2 * slots) return kWhole;         // (no walk is 1.9 times the average place's then)
    for (int key0 = 0; key0 < x.c.Nc; key0 += bc) {
      const long long walk = walk_of(x, key0);
      total += walk * heads;
      most = std::max(most, walk);
    }
  }
  auto cut = [&](long long parts, int tiles) {
    burst::RowPlan plan = {{nullptr, part_columns(heads, parts), (int)parts, tiles, 0}, {}, 1};
    burst::RowParts& p = plan.parts;
    for (size_t i = 0; i < w.size(); i++) {
      int lo = -1, hi = 0;
      for (int key0 = 0; key0 < w[i].c.Nc; key0 += bc)
        if (p.of((int)walk_of(w[i], key0)) > 1) { lo = lo < 0 ? key0 : lo; hi = std::min(key0 + bc, w[i].c.Nc); }
      plan.span[i] = {p.rows, std::max(lo, 0), hi - std::max(lo, 0)};
      p.rows += (int)(heads * plan.span[i].keys);
    }
    return plan;
  };
  if (most > 0x7fffffffLL) return kWhole;
  if (generic) {
    // as many as there are CUs for, four tiles each at least; two also where a causal launch fits the CUs once.
    // us a launch, whole / by the rule: 1024 keys x 256 rows, one head, d = 64, 28 / 19 in 2; 500 x 500, d = 128, 64 / 30 in 4 (2: 41);
    // 8 x 700 causal, d = 64, 56 / 44 in 2; not cut: 8 x 600 keys x 300 rows, causal, d = 80, 37 (2: 52).  Short walks of at most 64 columns
    // are whole, as in generic_splits: a pass, whole / cut, us: d = 32, 600 rows x 256 keys
    // (19 tiles) 42 / 48, 1400 x 128 (44) 51 / 48; d = 64, 300 x 300 (10) 60 / 60, without waiting 85 / 88, 384 x 384 (12) 60 / 57.
    long long parts = std::min({256 / blocks, most / 4, 16LL});
    if (parts < 2 && blocks <= 256 && most >= 16 && 10 * most * slots >= 18 * total) parts = 2;
    return parts < 2 || (k.d <= 32 ? most - most / parts < 16 : k.d <= 64 && most < 12) ? kWhole : cut(parts, (int)((most + parts - 1) / parts));
  }
  if (most * unit < 24 || 10 * most * slots < 19 * total) return kWhole;
  const long long ratio = (4 * most * slots + 3 * total - 1) / (4 * total);   // the ratio rounded up from a quarter on
  const long long splits = std::min({16LL, ratio, most * unit / (f.plain != nullptr ? 8 : 16)});
  if (splits < 2) return kWhole;
  // What the longest walk has above a CU's share has to be worth the merging launch: 16 tiles at d = 64, 6 on the padded kernels, whose
  // tiles take three times as long.  Backward pass, whole / cut, us: d = 64, 32 x 1226 causal, 13 tiles above, 73.2 / 78.3, 2 x 3840 x
  // 15360, 8, 177 / 202, 16 x 1984 x 1280, 15.5, 96.1 / 94.5, 16 x 919 causal, 21, 54.7 / 50.7; d = 96, 32 x 1024, 0, 113 / 119; d = 40, 16 x 851
  // x 2099, window 71, 2, 91 / 100; d = 120, 8 x 2209, window 674, 11, 245 / 204.  Hand-scheduled (one workgroup a CU): the share and a
  // part behind it have to be shorter than the longest walk (1 x 4736 x 18944, 148 equal blocks, in 2: 192 / 223; 4 x 3547, 112, in 3 143 / 139).
  const long long share = total / 256;
  if (f.hand ? share + (most + splits - 1) / splits >= most : (most - share) * unit < (f.plain == &kD64 ? 16 : 6)) return kWhole;
  return cut(splits, 8 / unit);
}
burst::RowPlan dkv_parts(const std::vector<WalkChunk>& w, bool half) {
  burst::RowPlan plan = cut_walks(w);
  if (!half || w.size() != 1 || w[0].p.block_mask != nullptr || w[0].k.Nq == 0) return plan;
  const Kernels f = dkv_kernels(&w[0].p, w[0].k);
  if (f.plain == nullptr || f.plain->dkv_keys() != 128 || f.plain->dkv_rows() != 32) return plan;
  const KParams& k = w[0].k;
  const long long blocks = (long long)k.B * k.H / k.group * ((w[0].c.Nc + 127) / 128), walk = (long long)k.group * ((k.Nq + 31) / 32);
  const bool narrow = f.plain == &kD64;
  if (plan.parts.splits > 1 && (blocks <= (narrow ? 48 : 64) || (blocks <= 128 && !narrow && walk >= 32) || (blocks <= 256 && walk >= 96))) return plan;
  if (blocks > (!burst::unequal_keys(k, w[0].c, 128, 32) ? 448 : narrow ? 768 : 1024)) return plan;
  plan = kWhole;
  plan.groups = 2;
  return plan;
}
size_t dkv_bytes(const KParams& k, const burst::RowPlan& plan) {
  const burst::RowParts& p = plan.parts;
  return p.splits > 1 ? (size_t)p.most * 2 * p.rows * k.d * sizeof(float) : 0;
}
// Whether the first dQ launch of a walk computes D (the same bits as a launch of its own).  The d = 64 and padded kernels do
// where they are not split by keys (each range would compute it, dQ of 32 over 8 heads x 3001 rows, d = 128: 116 / 125 us):
// the launch saved is worth more than the two rows read before the first tile at every size, backward pass, us, own launch /
// by dQ: d = 64, 32 heads x 512 causal rows 36.9 / 35.9, 64 x 1024 69.5 / 67.2, 32 x 4096 396 / 394, 32 x 8192 1086 / 1081, 32 x
// 65536 rows x 64 keys 475 / 476; d = 96, 64 x 1024 128 / 125, 32 x 32768 x 96 492 / 487.  The d = 128 kernels lose as much (dQ
// 153 / 163, the launch 9).  fp32: every row block starts with reads
// that nothing covers (32 x 8192 rows x 32 keys, d = 64, 220 / 249, 16 x 2000 x 32, d = 128, 112 / 119, 16 x 3000 x 1000, 758 / 767),
// so only walks of at most two blocks of 32 rows a CU, where the two forms take the GPU about the same time (8 x 1000 causal, d = 64,
// 85.3 / 85.8; 4 x 500 32.4 / 31.5; d = 128, 8 x 1423 causal, 360 blocks, 290.3 / 287.9, 16 x 1000 x 64, 512, 112.8 / 114.0; d = 96, 16 x 800 x 1600
// causal 386.0 / 385.6) and the launch saved is the host's (256 rows x 1024 keys, 82 / 77 a pass; 8 x 700 x 1400, 247.8 / 246.0);
// rows of at most 48 columns up to four a CU (d = 24, 32 x 805 x 41 29.5 / 28.3; d = 48, 16 x 1000 causal 135.0 / 133.8, 32 x 8192 x 32 205 / 216).
bool d_by_dq(const std::vector<WalkChunk>& w, int splits, bool whole) {
  if (w.empty()) return false;
  const Kernels f = fwd_kernels(&w[0].p, w[0].k, whole);
  if (f.plain != nullptr) return f.plain != &kD128p && splits == 1;
  const long long blocks = (long long)w[0].k.B * w[0].k.H * (((long long)w[0].k.Nq + 31) / 32);
  if (f.hand || w[0].p.dtype != BURST_F32 || blocks > (w[0].k.d <= 48 ? 1024 : 512)) return false;
  for (const WalkChunk& x : w) if (!burst::fp32_tiles(x.k.d, x.k.lay, &x.c, 1)) return false;
  return true;
}
size_t split_bytes(const KParams& k, int splits) {
  return splits > 1 ? (size_t)splits * k.B * k.H * k.Nq * ((size_t)k.d + 2) * sizeof(float) : 0;
}

}  // namespace

extern "C" {

int burst_state_init(float* O_acc, float* m, float* l, const burst_params* p, void* stream) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  if ((long long)k.B * k.H * k.Nq == 0) return BURST_OK;
  REQUIRE_PTR(O_acc); REQUIRE_PTR(m); REQUIRE_PTR(l);
  if ((st = check_arch()) != BURST_OK) return st;
  return burst::launch_state_init(k, O_acc, m, l, (hipStream_t)stream);
}

int burst_local_fwd(const void* Q, const void* K_chunk, const void* V_chunk,
                    float* O_acc, float* m, float* l, const burst_params* p, void* stream) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  if ((long long)k.B * k.H * k.Nq == 0 || k.Nc == 0) return BURST_OK;   // an empty chunk is the identity
  REQUIRE_PTR(Q); REQUIRE_PTR(K_chunk); REQUIRE_PTR(V_chunk);
  REQUIRE_PTR(O_acc); REQUIRE_PTR(m); REQUIRE_PTR(l);
  if ((st = check_arch()) != BURST_OK) return st;
  const FwdIo io = {Q, O_acc, m, l, nullptr, nullptr, 0, nullptr, 1, 1};
  const Chunk c = burst::chunk_of(k, K_chunk, V_chunk, nullptr, nullptr);
  return fwd_launch(fwd_kernels(p, k), k, p->dtype, io, &c, 1, (hipStream_t)stream);
}

int burst_set_kernel_family(int family) {
  if (family < 0 || family > 2) return BURST_ERR_SHAPE;
  g_kernel_family.store(family, std::memory_order_relaxed);
  return BURST_OK;
}

int burst_kernel_family_for(const burst_params* p) {
  KParams k;
  const int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  if (use_plain128(p, k)) return 2;
  return use_mfma(p, k) && (p->block_mask == nullptr || p->Nc <= kMaxMaskedRows) ? 1 : 0;
}

size_t burst_workspace_bytes(const burst_params* p) {
  KParams k;
  if (check_params(p, &k) != BURST_OK) return 0;
  return (size_t)k.B * k.H * k.Nq * sizeof(float);
}

size_t burst_materialized_workspace_bytes(const burst_params* p) {
  KParams k;
  if (check_params(p, &k) != BURST_OK) return 0;
  return burst::materialized_workspace_bytes(k, p->dtype);
}

int burst_local_fwd_materialized(const void* Q, const void* K_chunk, const void* V_chunk,
                                 float* O_acc, float* m, float* l,
                                 void* workspace, size_t workspace_bytes,
                                 const burst_params* p, void* stream) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  if ((long long)k.B * k.H * k.Nq == 0 || k.Nc == 0) return BURST_OK;   // an empty chunk is the identity
  REQUIRE_PTR(Q); REQUIRE_PTR(K_chunk); REQUIRE_PTR(V_chunk);
  REQUIRE_PTR(O_acc); REQUIRE_PTR(m); REQUIRE_PTR(l);
  if (workspace == nullptr) return BURST_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return BURST_ERR_ALIGN;
  if (workspace_bytes < burst::materialized_workspace_bytes(k, p->dtype)) return BURST_ERR_SHAPE;
  if ((st = check_arch()) != BURST_OK) return st;
  return validated([&] {
    return burst::launch_fwd_materialized(k, p->dtype, use_mfma(p, k), Q, K_chunk, V_chunk, O_acc, m, l, workspace,
                                          (hipStream_t)stream);
  });
}

size_t burst_materialized_bwd_workspace_bytes(const burst_params* p) {
  KParams k;
  if (check_params(p, &k) != BURST_OK) return 0;
  return burst::materialized_bwd_workspace_bytes(k, p->dtype);
}

int burst_local_bwd_materialized(const void* Q, const void* K_chunk, const void* V_chunk,
                                 const void* dO, const float* lse, const float* D,
                                 float* dQ, float* dK_chunk, float* dV_chunk,
                                 int accumulate_dq, int accumulate_dkv,
                                 void* workspace, size_t workspace_bytes,
                                 const burst_params* p, void* stream) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  const long long bh = (long long)k.B * k.H;
  const bool have_q = bh * k.Nq > 0, have_k = bh * k.Nc > 0;
  if (!have_q && !have_k) return BURST_OK;
  if (have_q) { REQUIRE_PTR(Q); REQUIRE_PTR(dO); REQUIRE_PTR(lse); REQUIRE_PTR(D); REQUIRE_PTR(dQ); }
  if (have_k) { REQUIRE_PTR(K_chunk); REQUIRE_PTR(V_chunk); REQUIRE_PTR(dK_chunk); REQUIRE_PTR(dV_chunk); }
  if ((st = check_arch()) != BURST_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  if (!have_q || !have_k) {                        // nothing to contract over: the contribution is zero
    if (have_q && !accumulate_dq && (st = burst::launch_zero_fill(dQ, bh * k.Nq * k.d, false, s)) != BURST_OK) return st;
    if (have_k && !accumulate_dkv) {
      if ((st = burst::launch_zero_fill(dK_chunk, bh / k.group * k.Nc * k.d, false, s)) != BURST_OK) return st;
      if ((st = burst::launch_zero_fill(dV_chunk, bh / k.group * k.Nc * k.d, false, s)) != BURST_OK) return st;
    }
    return BURST_OK;
  }
  REQUIRE_PTR(workspace);
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return BURST_ERR_ALIGN;
  if (workspace_bytes < burst::materialized_bwd_workspace_bytes(k, p->dtype)) return BURST_ERR_SHAPE;
  return validated([&] {
    return burst::launch_bwd_materialized(k, p->dtype, use_mfma(p, k), Q, K_chunk, V_chunk, dO, lse, D, dQ, dK_chunk,
                                          dV_chunk, accumulate_dq != 0, accumulate_dkv != 0, workspace, s);
  });
}

int burst_finalize(const float* O_acc, const float* m, const float* l,
                   void* O_out, float* lse, const burst_params* p, void* stream) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  if ((long long)k.B * k.H * k.Nq == 0) return BURST_OK;
  REQUIRE_PTR(O_acc); REQUIRE_PTR(m); REQUIRE_PTR(l); REQUIRE_PTR(O_out); REQUIRE_PTR(lse);
  if ((st = check_arch()) != BURST_OK) return st;
  return burst::launch_finalize(k, p->dtype, O_acc, m, l, O_out, lse, (hipStream_t)stream);
}

int burst_merge_state(float* O_a, float* m_a, float* l_a,
                      const float* O_b, const float* m_b, const float* l_b,
                      const burst_params* p, void* stream) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  if ((long long)k.B * k.H * k.Nq == 0) return BURST_OK;
  REQUIRE_PTR(O_a); REQUIRE_PTR(m_a); REQUIRE_PTR(l_a);
  REQUIRE_PTR(O_b); REQUIRE_PTR(m_b); REQUIRE_PTR(l_b);
  if ((st = check_arch()) != BURST_OK) return st;
  return burst::launch_merge_state(k, O_a, m_a, l_a, O_b, m_b, l_b, (hipStream_t)stream);
}

int burst_bwd_prepare(const void* O, const void* dO, float* D, const burst_params* p, void* stream) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  if ((long long)k.B * k.H * k.Nq == 0) return BURST_OK;
  REQUIRE_PTR(O); REQUIRE_PTR(dO); REQUIRE_PTR(D);
  if ((st = check_arch()) != BURST_OK) return st;
  return burst::launch_bwd_prepare(k, p->dtype, O, dO, D, (hipStream_t)stream);
}

// Shared by the three backward entry points.  which: 1 = dQ, 2 = dK/dV, 3 = both.
// static_d: D == NULL takes the static device scratch instead of an allocated buffer.
static int local_bwd_impl(int which, const void* Q, const void* K_chunk, const void* V_chunk,
                          const void* O, const void* dO, const float* lse, const float* D,
                          float* dQ, float* dK_chunk, float* dV_chunk,
                          int accumulate_dq, int accumulate_dkv,
                          const burst_params* p, void* stream, bool static_d = false) {
  KParams k;
  int st = check_params(p, &k);
  if (st != BURST_OK) return st;
  const bool want_dq = (which & 1) != 0, want_dkv = (which & 2) != 0;
  const long long bh = (long long)k.B * k.H;
  const bool have_q = bh * k.Nq > 0, have_k = bh * k.Nc > 0;
  if (!(want_dq && have_q) && !(want_dkv && have_k)) return BURST_OK;
  if (have_q) { REQUIRE_PTR(Q); REQUIRE_PTR(dO); REQUIRE_PTR(lse); }
  if (have_k) { REQUIRE_PTR(K_chunk); REQUIRE_PTR(V_chunk); }
  if (want_dq && have_q) REQUIRE_PTR(dQ);
  if (want_dkv && have_k) { REQUIRE_PTR(dK_chunk); REQUIRE_PTR(dV_chunk); }
  if (D != nullptr && !aligned16(D)) return BURST_ERR_ALIGN;
  if (D == nullptr && have_q && have_k) REQUIRE_PTR(O);
  if (static_d && bh * k.Nq > (long long)BURST_STATIC_MAX_ROWS) return BURST_ERR_TOO_LARGE;
  if ((st = check_arch()) != BURST_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  // Degenerate sides: nothing to contract over, the contribution is zero.
  if (!have_q || !have_k) {
    if (want_dq && have_q && !accumulate_dq &&
        (st = burst::launch_zero_fill(dQ, bh * k.Nq * k.d, false, s)) != BURST_OK) return st;
    if (want_dkv && have_k && !accumulate_dkv) {
      if ((st = burst::launch_zero_fill(dK_chunk, bh / k.group * k.Nc * k.d, false, s)) != BURST_OK) return st;
      if ((st = burst::launch_zero_fill(dV_chunk, bh / k.group * k.Nc * k.d, false, s)) != BURST_OK) return st;
    }
    return BURST_OK;
  }
  // The kernels of this call: D (when it is not given), then the dQ half, then the dK/dV half.
  const Kernels fq = fwd_kernels(p, k), fk = dkv_kernels(p, k);
  const Chunk c = burst::chunk_of(k, K_chunk, V_chunk, dK_chunk, dV_chunk);
  auto enqueue = [&](const float* Duse, float* Dwrite) -> int {
    int e;
    const BwdIo io = {Q, dO, lse, Duse, dQ, accumulate_dq != 0, accumulate_dkv != 0, 0, nullptr, 1, nullptr, nullptr, 1};
    if (Dwrite != nullptr && (e = burst::launch_bwd_prepare(k, p->dtype, O, dO, Dwrite, s)) != BURST_OK) return e;
    if (want_dq && (e = dq_launch(fq, k, p->dtype, io, &c, 1, s)) != BURST_OK) return e;
    if (want_dkv && (e = dkv_launch(fk, k, p->dtype, io, &c, 1, s)) != BURST_OK) return e;
    return BURST_OK;
  };
  if (D != nullptr) return validated([&] { return enqueue(D, nullptr); });
  std::lock_guard<std::mutex> lock(g_bwd_mutex);
  float* dbuf = nullptr;
  if ((st = static_d ? static_d_buffer(&dbuf) : get_d_scratch(s, (size_t)(bh * k.Nq), &dbuf)) != BURST_OK) return st;
  return validated([&] { return enqueue(dbuf, dbuf); });
}

int burst_local_bwd(const void* Q, const void* K_chunk, const void* V_chunk,
                    const void* O, const void* dO, const float* lse, const float* D,
                    float* dQ, float* dK_chunk, float* dV_chunk,
                    int accumulate_dq, int accumulate_dkv,
                    const burst_params* p, void* stream) {
  return local_bwd_impl(3, Q, K_chunk, V_chunk, O, dO, lse, D, dQ, dK_chunk, dV_chunk,
                        accumulate_dq, accumulate_dkv, p, stream);
}

int burst_local_bwd_static(const void* Q, const void* K_chunk, const void* V_chunk,
                           const void* O, const void* dO, const float* lse,
                           float* dQ, float* dK_chunk, float* dV_chunk,
                           int accumulate_dq, int accumulate_dkv,
                           const burst_params* p, void* stream) {
  return local_bwd_impl(3, Q, K_chunk, V_chunk, O, dO, lse, nullptr, dQ, dK_chunk, dV_chunk,
                        accumulate_dq, accumulate_dkv, p, stream, /*static_d=*/true);
}

int burst_local_bwd_dq(const void* Q, const void* K_chunk, const void* V_chunk,
                       const void* dO, const float* lse, const float* D,
                       float* dQ, int accumulate_dq, const burst_params* p, void* stream) {
  if (D == nullptr) return BURST_ERR_NULL;
  return local_bwd_impl(1, Q, K_chunk, V_chunk, nullptr, dO, lse, D, dQ, nullptr, nullptr,
                        accumulate_dq, 0, p, stream);
}

int burst_local_bwd_dkv(const void* Q, const void* K_chunk, const void* V_chunk,
                        const void* dO, const float* lse, const float* D,
                        float* dK_chunk, float* dV_chunk, int accumulate_dkv,
                        const burst_params* p, void* stream) {
  if (D == nullptr) return BURST_ERR_NULL;
  return local_bwd_impl(2, Q, K_chunk, V_chunk, nullptr, dO, lse, D, nullptr, dK_chunk, dV_chunk,
                        0, accumulate_dkv, p, stream);
}

size_t burst_walk_workspace_bytes(const burst_chunk* chunks, int n_chunks, const burst_params* p, int flags) {
  std::vector<WalkChunk> w;
  if (walk_chunks(chunks, n_chunks, p, false, w) != BURST_OK || w.empty()) return 0;
  const KParams& k = w[0].k;
  const size_t rows = (size_t)k.B * k.H * k.Nq;
  // (the two calls may plan differently: what is enough for either of them, unless it is for the forward alone)
  size_t need = split_bytes(k, walk_rows(w, false, w.size() == 1 && (flags & BURST_WALK_NO_STATE)).splits);
  if (!(flags & BURST_WALK_FORWARD))
    need = std::max(need, split_bytes(k, walk_rows(w, true, w.size() == 1 && (flags & BURST_WALK_HALF_GRADS)).splits));
  if (!(flags & (BURST_WALK_NO_STATE | BURST_WALK_FORWARD))) need = std::max(need, dkv_bytes(k, dkv_parts(w, (flags & BURST_WALK_HALF_GRADS) != 0)));
  if ((flags & (BURST_WALK_NO_STATE | BURST_WALK_HALF_GRADS)) && dq_launches(w, w.size() == 1) > 1) {          // between the launches: dQ in fp32, the state
    if (flags & BURST_WALK_HALF_GRADS) need = std::max(need, rows * k.d * sizeof(float));
    if (flags & BURST_WALK_NO_STATE) need = std::max(need, rows * ((size_t)k.d + 8) * sizeof(float));
  }
  return need;
}

int burst_walk_dkv_form(const burst_chunk* chunks, int n_chunks, const burst_params* p, int with_workspace) {
  std::vector<WalkChunk> w;
  const int st = walk_chunks(chunks, n_chunks, p, false, w);
  if (st != BURST_OK || w.empty() || w[0].k.Nq == 0) return st;
  if (with_workspace && dkv_parts(w, false).parts.splits > 1) return 1;
  int form = -1;
  for_each_run(w, dkv_kernels, [&](const Kernels& f, const KParams& kc, const Chunk* c, int n, bool, bool) {
    if (form < 0) form = f.hand && f.key_waves == 4 && burst::dkv_chained(kc, c, n) ? 2 : 0;
    return (int)BURST_OK;
  });
  return form;
}

int burst_walk_fwd(const void* Q, const burst_chunk* chunks, int n_chunks, float* O_acc, float* m, float* l,
                   void* O_out, float* lse, void* workspace, size_t workspace_bytes,
                   const burst_params* p, void* stream) {
  KParams k;
  burst_params base;
  if (p == nullptr) return BURST_ERR_NULL;
  base = *p;
  base.Nc = 0; base.block_mask = nullptr;
  std::memset(base.kv_strides, 0, sizeof base.kv_strides);
  int st = check_params(&base, &k);
  if (st != BURST_OK) return st;
  std::vector<WalkChunk> w;
  if ((st = walk_chunks(chunks, n_chunks, p, false, w)) != BURST_OK) return st;
  if ((long long)k.B * k.H * k.Nq == 0) return BURST_OK;
  REQUIRE_PTR(Q); REQUIRE_PTR(O_out); REQUIRE_PTR(lse);
  const bool keep = O_acc != nullptr || m != nullptr || l != nullptr, whole = !keep && w.size() == 1;
  if (keep) { REQUIRE_PTR(O_acc); REQUIRE_PTR(m); REQUIRE_PTR(l); }
  if (workspace != nullptr && !aligned16(workspace)) return BURST_ERR_ALIGN;
  if ((st = check_arch()) != BURST_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  if (!keep && (w.empty() || dq_launches(w, whole) > 1)) {   // (as many launches as dQ takes)
    const size_t rows = (size_t)k.B * k.H * k.Nq;
    if (w.empty()) return burst::launch_fill_unseen(k, p->dtype, O_out, lse, s);
    if (workspace == nullptr || workspace_bytes < rows * ((size_t)k.d + 8) * sizeof(float)) return BURST_ERR_SHAPE;
    O_acc = (float*)workspace; m = O_acc + rows * k.d; l = m + (rows + 3) / 4 * 4;
  }
  RowsPlan rows = walk_rows(w, false, whole);
  if (rows.splits > 1 && (workspace == nullptr || workspace_bytes < split_bytes(k, rows.splits))) rows = {1, 1};
  if (rows.splits > 1) {
    const FwdIo io = {Q, O_acc, m, l, O_out, lse, 1, (float*)workspace, rows.splits, rows.groups};
    return validated([&] {
      const int e = for_each_run(w, walk_choice(whole), [&](const Kernels& f, const KParams& kc, const Chunk* c, int n, bool, bool) {
        return fwd_launch(f, kc, p->dtype, io, c, n, s);
      });
      return e != BURST_OK || fwd_kernels(&w[0].p, w[0].k, whole).plain == nullptr ? e : burst::launch_merge_splits(k, io, s);   // (the generic launcher merges by itself)
    });
  }
  return validated([&] {
    bool fresh = true, final = false;
    const int e = for_each_run(w, walk_choice(whole), [&](const Kernels& f, const KParams& kc, const Chunk* c, int n, bool, bool last) {
      FwdIo io = {Q, O_acc, m, l, nullptr, nullptr, fresh, nullptr, 1, rows.groups};
      if (last) { io.O_out = O_out; io.lse = lse; final = true; }
      fresh = false;
      return fwd_launch(f, kc, p->dtype, io, c, n, s);
    });
    if (e != BURST_OK) return e;
    if (fresh)
      if (const int i = burst::launch_state_init(k, O_acc, m, l, s); i != BURST_OK) return i;
    return final ? (int)BURST_OK : burst::launch_finalize(k, p->dtype, O_acc, m, l, O_out, lse, s);
  });
}

int burst_walk_bwd(const void* Q, const burst_chunk* chunks, int n_chunks, const void* O, const void* dO,
                   const float* lse, float* D, void* dQ, int accumulate_dq, int accumulate_dkv, int half_grads,
                   void* workspace, size_t workspace_bytes, const burst_params* p, void* stream) {
  KParams k;
  burst_params base;
  if (p == nullptr) return BURST_ERR_NULL;
  base = *p;
  base.Nc = 0; base.block_mask = nullptr;
  std::memset(base.kv_strides, 0, sizeof base.kv_strides);
  int st = check_params(&base, &k);
  if (st != BURST_OK) return st;
  std::vector<WalkChunk> w;
  if ((st = walk_chunks(chunks, n_chunks, p, true, w)) != BURST_OK) return st;
  if (half_grads && (accumulate_dq || accumulate_dkv)) return BURST_ERR_SHAPE;
  const bool half = half_grads && p->dtype == BURST_BF16;
  const long long bh = (long long)k.B * k.H;
  const bool have_q = bh * k.Nq > 0;
  if (!have_q && w.empty()) return BURST_OK;
  if (have_q) {
    REQUIRE_PTR(Q); REQUIRE_PTR(dO); REQUIRE_PTR(lse); REQUIRE_PTR(D); REQUIRE_PTR(dQ);
    if (O != nullptr && !aligned16(O)) return BURST_ERR_ALIGN;
  }
  if (workspace != nullptr && !aligned16(workspace)) return BURST_ERR_ALIGN;
  if ((st = check_arch()) != BURST_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  const bool whole = half && w.size() == 1;
  RowsPlan rows = walk_rows(w, true, whole);
  if (rows.splits > 1 && (workspace == nullptr || workspace_bytes < split_bytes(k, rows.splits))) rows = {1, 1};
  const int splits = rows.splits;
  burst::RowPlan parts = dkv_parts(w, half);
  if (parts.parts.splits > 1 && (workspace == nullptr || workspace_bytes < dkv_bytes(k, parts))) parts = kWhole;
  parts.parts.part = (float*)workspace;
  auto zero = [&](void* ptr, long long n) { return burst::launch_zero_fill((float*)ptr, n, half, s); };
  // dQ as bf16 by several launches: fp32 in the workspace between them
  const bool staged = half && have_q && splits == 1 && !w.empty() && dq_launches(w, whole) > 1;
  if (staged && (workspace == nullptr || workspace_bytes < (size_t)bh * k.Nq * k.d * sizeof(float))) return BURST_ERR_SHAPE;
  return validated([&]() -> int {
    int e = BURST_OK;
    if (!have_q) {                                 // no rows: dK and dV are zero
      for (const WalkChunk& x : w) {
        if (accumulate_dkv) break;
        if ((e = zero(x.c.dK, bh / k.group * x.c.Nc * k.d)) != BURST_OK) return e;
        if ((e = zero(x.c.dV, bh / k.group * x.c.Nc * k.d)) != BURST_OK) return e;
      }
      return BURST_OK;
    }
    const bool fused = O != nullptr && d_by_dq(w, splits, whole);
    if (O != nullptr && !fused && (e = burst::launch_bwd_prepare(k, p->dtype, O, dO, D, s)) != BURST_OK) return e;
    if (w.empty()) return accumulate_dq ? (int)BURST_OK : zero(dQ, bh * k.Nq * k.d);
    BwdIo io = {Q, dO, lse, D, dQ, accumulate_dq != 0, accumulate_dkv != 0, half, (float*)workspace, splits,
                parts.parts.splits > 1 || parts.groups > 1 ? &parts : nullptr, nullptr, rows.groups};
    e = for_each_run(w, walk_choice(whole), [&](const Kernels& f, const KParams& kc, const Chunk* c, int n, bool first, bool) {
      BwdIo one = io;
      one.acc_dq = accumulate_dq != 0 || !first;
      one.O = fused && first ? O : nullptr;
      if (staged) { one.dQ = workspace; one.half = 0; }
      return dq_launch(f, kc, p->dtype, one, c, n, s);
    });
    if (e != BURST_OK) return e;
    if (((splits > 1 && fwd_kernels(&w[0].p, w[0].k, whole).plain != nullptr) || staged) && (e = burst::launch_sum_splits(k, io, s)) != BURST_OK) return e;
    return for_each_run(w, dkv_kernels, [&](const Kernels& f, const KParams& kc, const Chunk* c, int n, bool, bool) {
      return dkv_launch(f, kc, p->dtype, io, c, n, s);
    });
  });
}

void* burst_event_create(void) {
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return (void*)e;
}
int burst_event_record(void* event, void* stream) {
  if (event == nullptr) return BURST_ERR_NULL;
  return hipEventRecord((hipEvent_t)event, (hipStream_t)stream) == hipSuccess ? BURST_OK : BURST_ERR_LAUNCH;
}
int burst_event_elapsed_ms(void* start, void* stop, float* ms) {
  if (start == nullptr || stop == nullptr || ms == nullptr) return BURST_ERR_NULL;
  if (hipEventSynchronize((hipEvent_t)stop) != hipSuccess) return BURST_ERR_LAUNCH;
  return hipEventElapsedTime(ms, (hipEvent_t)start, (hipEvent_t)stop) == hipSuccess ? BURST_OK : BURST_ERR_LAUNCH;
}
void burst_event_destroy(void* event) {
  if (event != nullptr) (void)hipEventDestroy((hipEvent_t)event);
}

const char* burst_strerror(int status) {
  switch (status) {
    case BURST_OK: return "ok";
    case BURST_ERR_NULL: return "a required pointer is NULL";
    case BURST_ERR_ALIGN: return "a pointer is not 16-byte aligned";
    case BURST_ERR_SHAPE: return "unsupported or inconsistent sizes or scale";
    case BURST_ERR_DTYPE: return "unknown dtype";
    case BURST_ERR_ARCH: return "current device is not gfx950";
    case BURST_ERR_LAUNCH: return "HIP runtime reported a launch error";
    case BURST_ERR_ALLOC: return "internal scratch allocation failed";
    case BURST_ERR_TOO_LARGE: return "B*H*Nq exceeds the static scratch of burst_local_bwd_static (BURST_STATIC_MAX_ROWS rows)";
    default: return "unknown status";
  }
}

int burst_version(void) { return 113; }

}  // extern "C"
