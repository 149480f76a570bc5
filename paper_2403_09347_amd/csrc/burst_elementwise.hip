// HBM-bound steps of the path: state init, finalize, standalone merge (paper Alg. 1) and
// D = rowsum(dO o O) (paper Alg. 2 pre-step).  One thread handles 4 consecutive elements of
// a row (128-bit accesses); the d/4 threads of a row are consecutive lanes, so every
// wavefront touches whole rows and per-row scalars are read once per row.
#include "burst_common.h"

namespace burst {

__global__ void __launch_bounds__(256)
state_init_kernel(float* __restrict__ O_acc, float* __restrict__ m, float* __restrict__ l,
                  long long n_o4, long long n_rows) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  long long stride = (long long)gridDim.x * 256;
  f32x4 z = {0.f, 0.f, 0.f, 0.f};
  for (long long k = i; k < n_o4; k += stride) reinterpret_cast<f32x4*>(O_acc)[k] = z;
  for (long long k = i; k < n_rows; k += stride) { m[k] = BURST_NEG_INF; l[k] = 0.f; }
}

// Scalar tail-safe variant for d not a multiple of 4 is handled by VEC = 1.
template <typename OutT, int VEC>
__global__ void __launch_bounds__(256)
finalize_kernel(const float* __restrict__ O_acc, const float* __restrict__ m, const float* __restrict__ l,
                OutT* __restrict__ O_out, float* __restrict__ lse, long long n_rows, int d, QRows qr) {
  const int per_row = d / VEC;
  long long total = n_rows * per_row;
  long long stride = (long long)gridDim.x * 256;
  for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < total; k += stride) {
    long long row = k / per_row;
    int c = (int)(k - row * per_row);
    float lv = l[row];
    float inv = lv > 0.f ? 1.0f / lv : 0.f;
    if (c == 0) lse[row] = lv > 0.f ? m[row] + __logf(lv) : BURST_NEG_INF;
    const float* src = O_acc + row * d + c * VEC;
    OutT* dst = O_out + qr.off(row) + c * VEC;
    if (VEC == 4) {
      f32x4 v = *reinterpret_cast<const f32x4*>(src);
      if (sizeof(OutT) == 4) {
        f32x4 r;
        for (int t = 0; t < 4; t++) r[t] = lv > 0.f ? v[t] * inv : 0.f;
        *reinterpret_cast<f32x4*>(dst) = r;
      } else {
        bf16x4 r;
        for (int t = 0; t < 4; t++) r[t] = (bf16)(lv > 0.f ? v[t] * inv : 0.f);
        *reinterpret_cast<bf16x4*>(dst) = r;
      }
    } else {
      dst[0] = (OutT)(lv > 0.f ? src[0] * inv : 0.f);
    }
  }
}

// Standalone merge.  The state is updated in place, so every thread of a row must read the
// row's old (m, l) before the new ones are written.  Both kernels keep a row inside ONE
// wavefront: its loads of (m, l) precede the store in program order.
//   packed: d/4 lanes per row (d/4 divides 64), 128-bit accesses
__global__ void __launch_bounds__(256)
merge_state_packed_kernel(float* __restrict__ O_a, float* __restrict__ m_a, float* __restrict__ l_a,
                          const float* __restrict__ O_b, const float* __restrict__ m_b,
                          const float* __restrict__ l_b, long long n_rows, int d) {
  const int per_row = d >> 2;
  long long total = n_rows * per_row;
  long long stride = (long long)gridDim.x * 256;
  for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < total; k += stride) {
    long long row = k / per_row;
    int c = (int)(k - row * per_row);
    float ma = m_a[row], mb = m_b[row], la = l_a[row], lb = l_b[row];
    float mn = fmaxf(ma, mb);
    float ref = (mn == BURST_NEG_INF) ? 0.f : mn;
    float fa = __expf(ma - ref), fb = __expf(mb - ref);   // exp(-inf) = 0
    float* pa = O_a + row * d + c * 4;
    f32x4 va = *reinterpret_cast<const f32x4*>(pa);
    f32x4 vb = *reinterpret_cast<const f32x4*>(O_b + row * d + c * 4);
    f32x4 r;
    for (int t = 0; t < 4; t++)
      r[t] = (fa == 0.f ? 0.f : fa * va[t]) + (fb == 0.f ? 0.f : fb * vb[t]);
    *reinterpret_cast<f32x4*>(pa) = r;
    if (c == 0) {
      m_a[row] = mn;
      l_a[row] = (fa == 0.f ? 0.f : fa * la) + (fb == 0.f ? 0.f : fb * lb);
    }
  }
}
//   generic: one wavefront per row, any d
__global__ void __launch_bounds__(256)
merge_state_row_kernel(float* __restrict__ O_a, float* __restrict__ m_a, float* __restrict__ l_a,
                       const float* __restrict__ O_b, const float* __restrict__ m_b,
                       const float* __restrict__ l_b, long long n_rows, int d) {
  const int lane = threadIdx.x & 63;
  long long wave = ((long long)blockIdx.x * 256 + threadIdx.x) >> 6;
  long long nwaves = ((long long)gridDim.x * 256) >> 6;
  for (long long row = wave; row < n_rows; row += nwaves) {
    float ma = m_a[row], mb = m_b[row], la = l_a[row], lb = l_b[row];
    float mn = fmaxf(ma, mb);
    float ref = (mn == BURST_NEG_INF) ? 0.f : mn;
    float fa = __expf(ma - ref), fb = __expf(mb - ref);
    for (int c = lane; c < d; c += 64) {
      float* pa = O_a + row * d + c;
      pa[0] = (fa == 0.f ? 0.f : fa * pa[0]) + (fb == 0.f ? 0.f : fb * O_b[row * d + c]);
    }
    if (lane == 0) {
      m_a[row] = mn;
      l_a[row] = (fa == 0.f ? 0.f : fa * la) + (fb == 0.f ? 0.f : fb * lb);
    }
  }
}

// D = rowsum(dO o O).  L lanes per row (a power of two), each with 16 bytes of either tensor per step;
// HBM bound.  65536 rows of d = 64: 10.1 us with one wavefront per row (of which 16 lanes had work), 4.6 us
// with 8 lanes a row.
template <typename T, int L>
__global__ void __launch_bounds__(256)
bwd_prepare_kernel(const T* __restrict__ O, const T* __restrict__ dO, float* __restrict__ D,
                   long long n_rows, int d, QRows qr) {
  constexpr int E = 16 / sizeof(T);
  typedef __attribute__((ext_vector_type(E))) T vec;
  const int part = threadIdx.x % L;
  const long long stride = (long long)gridDim.x * (256 / L);
  // (every lane stays in the loop as long as one of its wavefront has a row: the shuffles need them)
  for (long long row = (long long)blockIdx.x * (256 / L) + threadIdx.x / L; row - (threadIdx.x & 63) / L < n_rows; row += stride) {
    float acc = 0.f;
    if (row < n_rows) {
      const size_t base = qr.off(row);
      for (int c = part * E; c < d; c += L * E) {
        const vec x = *reinterpret_cast<const vec*>(O + base + c), y = *reinterpret_cast<const vec*>(dO + base + c);
#pragma unroll
        for (int t = 0; t < E; t++) acc = fma_in_order((float)x[t], (float)y[t], acc);
      }
    }
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (row < n_rows && part == 0) D[row] = acc;
  }
}
// rows that do not start on 16 bytes: one wavefront per row
template <typename T>
__global__ void __launch_bounds__(256)
bwd_prepare_row_kernel(const T* __restrict__ O, const T* __restrict__ dO, float* __restrict__ D,
                       long long n_rows, int d, QRows qr) {
  const int lane = threadIdx.x & 63;
  const long long nwaves = ((long long)gridDim.x * 256) >> 6;
  for (long long row = ((long long)blockIdx.x * 256 + threadIdx.x) >> 6; row < n_rows; row += nwaves) {
    const size_t base = qr.off(row);
    float acc = 0.f;
    for (int c = lane; c < d; c += 64) acc += (float)O[base + c] * (float)dO[base + c];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) D[row] = acc;
  }
}

__global__ void __launch_bounds__(256)
zero_fill_kernel(float* __restrict__ p, long long n) {
  long long stride = (long long)gridDim.x * 256;
  long long n4 = n >> 2;
  f32x4 z = {0.f, 0.f, 0.f, 0.f};
  for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < n4; k += stride)
    reinterpret_cast<f32x4*>(p)[k] = z;
  for (long long k = (n4 << 2) + (long long)blockIdx.x * 256 + threadIdx.x; k < n; k += stride) p[k] = 0.f;
}

// Partial states of `splits` key ranges (O [splits][rows][d], then m, in log2 units or natural, and l, each
// [splits][rows]) -> one, merged with the stored state unless that is the initial one; with O_out also
// finalized (Alg. 1 merge step and last two steps).  HBM bound: every partial is read once.  d a
// multiple of 8; d / 4 threads per row, whole rows per workgroup, so that a barrier separates the
// reads of a row's old m and l from the write of the new ones.
__global__ void __launch_bounds__(256)
merge_splits_kernel(const float* __restrict__ part, int splits, float* __restrict__ O_acc, float* __restrict__ m,
                    float* __restrict__ l, bf16* __restrict__ O_out, float* __restrict__ lse, int fresh,
                    int natural, long long n_rows, int d, QRows qr) {
  const float to_log2 = natural ? kLog2e : 1.f, to_units = natural ? 1.f : kLog2e, to_stored = natural ? 1.f : kLn2;
  const int per_row = d >> 2;
  const float* const pm = part + (size_t)splits * n_rows * d;
  const float* const pl = pm + (size_t)splits * n_rows;
  const int rows_here = 256 / per_row, r_in = threadIdx.x / per_row, c = threadIdx.x - r_in * per_row;
  const bool live = r_in < rows_here && (long long)blockIdx.x * rows_here + r_in < n_rows;
  const long long row = live ? (long long)blockIdx.x * rows_here + r_in : 0;
  // (8 and 4 ranges at a time, their loads requested together: 32 heads x
  // 40 rows, 16 ranges, 11.6 us one after the other, 9.3 so)
  float mg = BURST_NEG_INF;
  for (int i = 0; i < splits; i += 8) {
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; j++) x[j] = pm[min(i + j, splits - 1) * n_rows + row];
#pragma unroll
    for (int j = 0; j < 8; j++) mg = fmaxf(mg, x[j]);
  }
  const float m_old = fresh ? BURST_NEG_INF : m[row], l_old = fresh ? 0.f : l[row];
  float m_st = m_old, lsum = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  f32x4* const state = reinterpret_cast<f32x4*>(O_acc + row * d + c * 4);
  if (mg != BURST_NEG_INF) {
    const float m_old_u = m_old * to_units, mn = fmaxf(mg, m_old_u);
    const float fa = fast_exp2((m_old_u - mn) * to_log2);
    if (fa != 0.f) {
      const f32x4 old = *state;
      for (int t = 0; t < 4; t++) o[t] = fa * old[t];
      lsum = fa * l_old;
    }
    for (int i = 0; i < splits; i += 4) {
      f32x4 v[4];
      float x[4], l4[4];
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int k = min(i + j, splits - 1);
        v[j] = *reinterpret_cast<const f32x4*>(part + ((size_t)k * n_rows + row) * d + c * 4);
        x[j] = pm[k * n_rows + row];
        l4[j] = pl[k * n_rows + row];
      }
#pragma unroll
      for (int j = 0; j < 4; j++) {
        if (i + j >= splits) break;
        const float f = fast_exp2((x[j] - mn) * to_log2);
        for (int t = 0; t < 4; t++) o[t] += f * v[j][t];
        lsum += f * l4[j];
      }
    }
    m_st = mn * to_stored;
  } else if (m_old != BURST_NEG_INF) {             // no range saw a key: the state stays
    o = *state;
    lsum = l_old;
  }
  __syncthreads();
  if (!live) return;
  if (O_acc != nullptr && (fresh || mg != BURST_NEG_INF)) {
    *state = o;
    if (c == 0) { m[row] = m_st; l[row] = lsum; }
  }
  if (O_out != nullptr) {
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    bf16x4 r;
    for (int t = 0; t < 4; t++) r[t] = (bf16)(lsum > 0.f ? o[t] * inv : 0.f);
    *reinterpret_cast<bf16x4*>(O_out + qr.off(row) + c * 4) = r;
    if (c == 0) lse[row] = lsum > 0.f ? m_st + __logf(lsum) : BURST_NEG_INF;
  }
}

// dQ = (acc ? dQ : 0) + the sum of `splits` partial dQ [splits][n], in that order; half: dQ is bf16.  More than one part
// only with n a multiple of 4; else (odd head dimensions) one thread takes the last elements.
__global__ void __launch_bounds__(256)
sum_splits_kernel(const float* __restrict__ part, int splits, void* __restrict__ dQ, int acc, int half, long long n) {
  const long long k = (long long)blockIdx.x * 256 + threadIdx.x, n4 = n >> 2;
  if (k > n4) return;
  if (k == n4) {
    for (long long e = n4 << 2; e < n; e++) {
      if (half) reinterpret_cast<bf16*>(dQ)[e] = (bf16)part[e];
      else reinterpret_cast<float*>(dQ)[e] = (acc ? reinterpret_cast<const float*>(dQ)[e] : 0.f) + part[e];
    }
    return;
  }
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (acc) v = reinterpret_cast<const f32x4*>(dQ)[k];
  for (int i = 0; i < splits; i += 4) {            // (four parts' loads together)
    f32x4 x[4];
#pragma unroll
    for (int j = 0; j < 4; j++) x[j] = reinterpret_cast<const f32x4*>(part)[(size_t)min(i + j, splits - 1) * n4 + k];
#pragma unroll
    for (int j = 0; j < 4; j++)
      if (i + j < splits)
        for (int t = 0; t < 4; t++) v[t] += x[j][t];
  }
  if (half) {
    bf16x4 r;
    for (int t = 0; t < 4; t++) r[t] = (bf16)v[t];
    reinterpret_cast<bf16x4*>(dQ)[k] = r;
  } else {
    reinterpret_cast<f32x4*>(dQ)[k] = v;
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
fill_unseen_kernel(T* __restrict__ O_out, float* __restrict__ lse, long long n_rows, int d, QRows qr) {
  const long long stride = (long long)gridDim.x * 256;
  for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < n_rows * d; k += stride) {
    const long long row = k / d;
    const int c = (int)(k - row * d);
    O_out[qr.off(row) + c] = (T)0.f;
    if (c == 0) lse[row] = BURST_NEG_INF;
  }
}

__global__ void zero_tail_kernel(unsigned short* p) { *p = 0; }

static inline unsigned grid_for(long long work_items, int per_block = 256, unsigned cap = 256 * 16) {
  long long b = (work_items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}


int launch_state_init(const KParams& p, float* O_acc, float* m, float* l, hipStream_t s) {
  long long rows = (long long)p.B * p.H * p.Nq;
  long long n_o = rows * p.d;
  if (rows == 0) return BURST_OK;
  if (n_o % 4 != 0) {  // odd sizes: scalar fill through the generic zero kernel + row init
    BURST_LAUNCH(zero_fill_kernel, dim3(grid_for(n_o)), dim3(256), 0, s, O_acc, n_o);
    BURST_LAUNCH(state_init_kernel, dim3(grid_for(rows)), dim3(256), 0, s, O_acc, m, l, 0LL, rows);
  } else {
    BURST_LAUNCH(state_init_kernel, dim3(grid_for(n_o / 4)), dim3(256), 0, s, O_acc, m, l, n_o / 4, rows);
  }
  return launch_status();
}

int launch_finalize(const KParams& p, int dtype, const float* O_acc, const float* m, const float* l,
                    void* O_out, float* lse, hipStream_t s) {
  long long rows = (long long)p.B * p.H * p.Nq;
  if (rows == 0) return BURST_OK;
  bool vec = (p.d % 4) == 0;
  unsigned g = grid_for(rows * (vec ? p.d / 4 : p.d));
  if (dtype == BURST_BF16) {
    if (vec) BURST_LAUNCH((finalize_kernel<bf16, 4>), dim3(g), dim3(256), 0, s, O_acc, m, l, (bf16*)O_out, lse, rows, p.d, p.q_rows());
    else BURST_LAUNCH((finalize_kernel<bf16, 1>), dim3(g), dim3(256), 0, s, O_acc, m, l, (bf16*)O_out, lse, rows, p.d, p.q_rows());
  } else {
    if (vec) BURST_LAUNCH((finalize_kernel<float, 4>), dim3(g), dim3(256), 0, s, O_acc, m, l, (float*)O_out, lse, rows, p.d, p.q_rows());
    else BURST_LAUNCH((finalize_kernel<float, 1>), dim3(g), dim3(256), 0, s, O_acc, m, l, (float*)O_out, lse, rows, p.d, p.q_rows());
  }
  return launch_status();
}

// O = 0, lse = -inf: the output of a walk without any key
int launch_fill_unseen(const KParams& p, int dtype, void* O_out, float* lse, hipStream_t s) {
  const long long rows = (long long)p.B * p.H * p.Nq;
  if (rows == 0) return BURST_OK;
  const unsigned g = grid_for(rows * p.d);
  if (dtype == BURST_BF16) BURST_LAUNCH(fill_unseen_kernel<bf16>, dim3(g), dim3(256), 0, s, (bf16*)O_out, lse, rows, p.d, p.q_rows());
  else BURST_LAUNCH(fill_unseen_kernel<float>, dim3(g), dim3(256), 0, s, (float*)O_out, lse, rows, p.d, p.q_rows());
  return launch_status();
}

int launch_merge_splits(const KParams& p, const FwdIo& io, hipStream_t s) {
  const long long rows = (long long)p.B * p.H * p.Nq;
  const int here = 256 / (p.d / 4);
  const long long blocks = (rows + here - 1) / here;
  if (rows == 0) return BURST_OK;
  if (blocks > 0x7fffffffLL) return BURST_ERR_SHAPE;
  BURST_LAUNCH(merge_splits_kernel, dim3((unsigned)blocks), dim3(256), 0, s, io.part, io.splits, io.O_acc, io.m, io.l,
               (bf16*)io.O_out, io.lse, io.fresh, p.d != 64 && p.d != 128, rows, p.d, p.q_rows());   // (natural: the padded builds)
  return launch_status();
}

int launch_sum_splits(const KParams& p, const BwdIo& io, hipStream_t s) {
  const long long n = (long long)p.B * p.H * p.Nq * p.d, blocks = (n / 4 + 256) / 256;
  if (n == 0) return BURST_OK;
  if (blocks > 0x7fffffffLL) return BURST_ERR_SHAPE;
  BURST_LAUNCH(sum_splits_kernel, dim3((unsigned)blocks), dim3(256), 0, s, io.part, io.splits, io.dQ, io.acc_dq,
               io.half, n);
  return launch_status();
}

int launch_merge_state(const KParams& p, float* O_a, float* m_a, float* l_a,
                       const float* O_b, const float* m_b, const float* l_b, hipStream_t s) {
  long long rows = (long long)p.B * p.H * p.Nq;
  if (rows == 0) return BURST_OK;
  if (p.d % 4 == 0 && 64 % (p.d / 4) == 0) {
    BURST_LAUNCH(merge_state_packed_kernel, dim3(grid_for(rows * (p.d / 4))), dim3(256), 0, s,
                       O_a, m_a, l_a, O_b, m_b, l_b, rows, p.d);
  } else {
    BURST_LAUNCH(merge_state_row_kernel, dim3(grid_for(rows * 64)), dim3(256), 0, s,
                       O_a, m_a, l_a, O_b, m_b, l_b, rows, p.d);
  }
  return launch_status();
}

template <typename T>
static int prepare_for(const KParams& p, const T* O, const T* dO, float* D, long long rows, hipStream_t s) {
  constexpr int E = 16 / sizeof(T);
  if (p.d % E != 0) {
    BURST_LAUNCH((bwd_prepare_row_kernel<T>), dim3(grid_for(rows * 64)), dim3(256), 0, s, O, dO, D, rows, p.d, p.q_rows());
    return launch_status();
  }
  const int pieces = p.d / E;                      // 16-byte pieces of a row
  if (pieces > 8) BURST_LAUNCH((bwd_prepare_kernel<T, 16>), dim3(grid_for(rows * 16)), dim3(256), 0, s, O, dO, D, rows, p.d, p.q_rows());
  else if (pieces > 4) BURST_LAUNCH((bwd_prepare_kernel<T, 8>), dim3(grid_for(rows * 8)), dim3(256), 0, s, O, dO, D, rows, p.d, p.q_rows());
  else BURST_LAUNCH((bwd_prepare_kernel<T, 4>), dim3(grid_for(rows * 4)), dim3(256), 0, s, O, dO, D, rows, p.d, p.q_rows());
  return launch_status();
}

int launch_bwd_prepare(const KParams& p, int dtype, const void* O, const void* dO, float* D, hipStream_t s) {
  const long long rows = (long long)p.B * p.H * p.Nq;
  if (rows == 0) return BURST_OK;
  return dtype == BURST_BF16 ? prepare_for(p, (const bf16*)O, (const bf16*)dO, D, rows, s)
                             : prepare_for(p, (const float*)O, (const float*)dO, D, rows, s);
}

// n elements, fp32 or (half) bf16
int launch_zero_fill(float* ptr, long long n, bool half, hipStream_t s) {
  if (half) {
    if (n % 2 != 0) {                              // an odd tail of two bytes
      BURST_LAUNCH(zero_tail_kernel, dim3(1), dim3(1), 0, s, (unsigned short*)ptr + n - 1);
    }
    n /= 2;
  }
  if (n <= 0) return launch_status();
  BURST_LAUNCH(zero_fill_kernel, dim3(grid_for(n / 4 + 1)), dim3(256), 0, s, ptr, n);
  return launch_status();
}

}  // namespace burst
