// Anchor selection (Sec. 3, Algorithms 1-2): the sketch Y and the column-pivoted QR of Y^T.
//
// Layout: the sketch is kept transposed, Yt = Y^T (l rows x N columns, row stride ldy = padded N),
// so that the QR's per-step pass r = q^T Yt reads each row coalesced.
//
// Pivoted QR (left-looking, classical Gram-Schmidt applied twice): with Q_j = [q_0 .. q_{j-1}]
// orthonormal (l x j, FP64) and nrm2[c] the squared residual norm of column c,
//   p      = argmax_c nrm2[c] over unselected columns (lowest index on ties)
//   w      = Yt[:, p];  w -= Q_j (Q_j^T w) twice;  q_j = w / ||w||
//   r[c]   = q_j^T Yt[:, c];  nrm2[c] -= r[c]^2 (clamped at 0)
// This selects the same pivots as Householder QR with column pivoting in exact arithmetic
// (the residual norms are those of the trailing columns), without forming R or T (Sec. 2.3:
// only the permutation is needed).
#include <hip/hip_runtime.h>

#include <cstdlib>

#include "gemm.h"
#include "kmv_kernels.h"
#include "radix_sort.h"
#include "scan.h"
#include "sketch_qrcp.h"

namespace krr {

// ------------------------------------------------------------------ sparse sketch (Algorithm 2)
// Yt[i, a] = sum_s sign[i, s] k(x_a, x_{idx[i, s]}).  Block: 256 targets a (one per thread) x kSkCols
// sketch columns; the r source points of a column are wave-uniform (scalar loads).  DM is the
// compile-time bound on d (coordinates held in registers).
constexpr int kSkCols = 8;

template <int DM, bool F64>
__global__ __launch_bounds__(256) void k_sketch_sparse(const double* __restrict__ X, int64_t n, int d,
                                                       const int64_t* __restrict__ idx,
                                                       const double* __restrict__ sign, int l, int r,
                                                       double inv_eps, float scale, void* __restrict__ Ytv,
                                                       int64_t ldy) {
  const int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool live = a < n;
  const int64_t ar = live ? a : 0;
  double xa[DM];
#pragma unroll
  for (int k = 0; k < DM; ++k) xa[k] = k < d ? X[ar * d + k] : 0.0;
  for (int ci = 0; ci < kSkCols; ++ci) {
    const int i = blockIdx.y * kSkCols + ci;
    if (i >= l) return;
    double acc = 0.0;
    float accf = 0.0f;
    for (int s = 0; s < r; ++s) {
      int64_t j = idx[(int64_t)i * r + s];
      j = j < 0 ? 0 : (j >= n ? n - 1 : j);
      const double w = sign[(int64_t)i * r + s];
      if (F64) {
        double d2 = 0.0;
#pragma unroll
        for (int k = 0; k < DM; ++k) {
          if (k < d) {
            const double df = xa[k] - X[j * d + k];
            d2 = __builtin_fma(df, df, d2);
          }
        }
        acc = __builtin_fma(w, exp_neg_f64(d2 * inv_eps), acc);
      } else {
        float d2 = 0.0f;
#pragma unroll
        for (int k = 0; k < DM; ++k) {
          if (k < d) {
            const float df = (float)(xa[k] - X[j * d + k]) * scale;   // difference taken in FP64
            d2 = __builtin_fmaf(df, df, d2);
          }
        }
        accf = __builtin_fmaf((float)w, __builtin_amdgcn_exp2f(-d2), accf);
      }
    }
    if (live) {
      if (F64) ((double*)Ytv)[(int64_t)i * ldy + a] = acc;
      else ((float*)Ytv)[(int64_t)i * ldy + a] = accf;
    }
  }
}

template <bool F64>
static void sketch_go(int dm, dim3 grid, hipStream_t s, const double* X, int64_t n, int d, const int64_t* idx,
                      const double* sign, int l, int r, double inv_eps, float scale, void* Yt, int64_t ldy) {
#define KRR_SK(DM) \
  hipLaunchKernelGGL((k_sketch_sparse<DM, F64>), grid, dim3(256), 0, s, X, n, d, idx, sign, l, r, inv_eps, scale, Yt, ldy)
  if (dm <= 4) KRR_SK(4);
  else if (dm <= 8) KRR_SK(8);
  else if (dm <= 16) KRR_SK(16);
  else if (dm <= 32) KRR_SK(32);
  else if (dm <= 64) KRR_SK(64);
  else KRR_SK(128);
#undef KRR_SK
}

void sketch_sparse_t(const double* X, int64_t n, int d, double eps, const int64_t* idx, const double* sign, int l,
                     int r, int prec, void* Yt, int64_t ldy, hipStream_t s) {
  dim3 grid((unsigned)ceil_div(n, 256), (unsigned)ceil_div(l, kSkCols));
  const float scale = (float)std::sqrt(kLog2e / eps);
  if (prec == KRR_FP64) sketch_go<true>(d, grid, s, X, n, d, idx, sign, l, r, 1.0 / eps, scale, Yt, ldy);
  else sketch_go<false>(d, grid, s, X, n, d, idx, sign, l, r, 1.0 / eps, scale, Yt, ldy);
  KRR_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ transposes
template <typename T>
__global__ void k_transpose_to(const double* __restrict__ Y, int64_t n, int l, T* __restrict__ Yt, int64_t ldy) {
  // Y n x l row-major -> Yt l x n (row stride ldy)
  __shared__ double tile[32][33];
  const int64_t a0 = (int64_t)blockIdx.x * 32;
  const int i0 = blockIdx.y * 32;
  for (int t = threadIdx.y; t < 32; t += 8) {
    const int64_t a = a0 + t;
    const int i = i0 + threadIdx.x;
    tile[t][threadIdx.x] = (a < n && i < l) ? Y[a * l + i] : 0.0;
  }
  __syncthreads();
  for (int t = threadIdx.y; t < 32; t += 8) {
    const int i = i0 + t;
    const int64_t a = a0 + threadIdx.x;
    if (i < l && a < n) Yt[(int64_t)i * ldy + a] = (T)tile[threadIdx.x][t];
  }
}

template <typename T>
__global__ void k_transpose_from(const T* __restrict__ Yt, int64_t ldy, int64_t n, int l, double* __restrict__ Y) {
  __shared__ double tile[32][33];
  const int64_t a0 = (int64_t)blockIdx.x * 32;
  const int i0 = blockIdx.y * 32;
  for (int t = threadIdx.y; t < 32; t += 8) {
    const int i = i0 + t;
    const int64_t a = a0 + threadIdx.x;
    tile[t][threadIdx.x] = (i < l && a < n) ? (double)Yt[(int64_t)i * ldy + a] : 0.0;
  }
  __syncthreads();
  for (int t = threadIdx.y; t < 32; t += 8) {
    const int64_t a = a0 + t;
    const int i = i0 + threadIdx.x;
    if (a < n && i < l) Y[a * l + i] = tile[threadIdx.x][t];
  }
}

void transpose_to_t(const double* Y, int64_t n, int l, int prec, void* Yt, int64_t ldy, hipStream_t s) {
  dim3 grid((unsigned)ceil_div(n, 32), (unsigned)ceil_div(l, 32));
  if (prec == KRR_FP64)
    hipLaunchKernelGGL(k_transpose_to<double>, grid, dim3(32, 8), 0, s, Y, n, l, (double*)Yt, ldy);
  else
    hipLaunchKernelGGL(k_transpose_to<float>, grid, dim3(32, 8), 0, s, Y, n, l, (float*)Yt, ldy);
  KRR_LAUNCH_CHECK();
}

void transpose_from_t(const void* Yt, int64_t ldy, int64_t n, int l, int prec, double* Y, hipStream_t s) {
  dim3 grid((unsigned)ceil_div(n, 32), (unsigned)ceil_div(l, 32));
  if (prec == KRR_FP64)
    hipLaunchKernelGGL(k_transpose_from<double>, grid, dim3(32, 8), 0, s, (const double*)Yt, ldy, n, l, Y);
  else
    hipLaunchKernelGGL(k_transpose_from<float>, grid, dim3(32, 8), 0, s, (const float*)Yt, ldy, n, l, Y);
  KRR_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ pivoted QR kernels
// (value, index) argmax with ties to the lower index; -1 marks selected columns.
struct ArgMax {
  double v;
  int64_t i;
};
__device__ __forceinline__ ArgMax amax(ArgMax a, ArgMax b) {
  if (b.v > a.v || (b.v == a.v && b.i < a.i)) return b;
  return a;
}

constexpr int kQrBlock = 256;

// Partial column sums over one slab of rows [i0, i0 + slab): part[slab, c] = sum_i q_i Yt[i, c] (MODE 0)
// or sum_i Yt[i, c]^2 (MODE 1).  2-D grid (column blocks x row slabs) so that a pass over Yt fills the
// chip even when n / 256 is small; one column per thread, rows unrolled by 4 for memory-level parallelism.
template <typename T, int MODE>
__global__ __launch_bounds__(kQrBlock) void k_qr_slab(const T* __restrict__ Yt, int64_t ldy, int64_t N, int l,
                                                      int slab, const double* __restrict__ q,
                                                      double* __restrict__ part) {
  const int64_t c = (int64_t)blockIdx.x * kQrBlock + threadIdx.x;
  const int i0 = blockIdx.y * slab;
  const int i1 = i0 + slab < l ? i0 + slab : l;
  if (c >= N) return;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  int i = i0;
  for (; i + 4 <= i1; i += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double y = (double)Yt[(int64_t)(i + u) * ldy + c];
      acc[u] = MODE == 1 ? __builtin_fma(y, y, acc[u]) : __builtin_fma(q[i + u], y, acc[u]);
    }
  }
  for (; i < i1; ++i) {
    const double y = (double)Yt[(int64_t)i * ldy + c];
    acc[0] = MODE == 1 ? __builtin_fma(y, y, acc[0]) : __builtin_fma(q[i], y, acc[0]);
  }
  part[(int64_t)blockIdx.y * N + c] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Column update after a pass, summing the slab partials in slab order: mode 1 sets nrm2[c] to the sum
// (initial squared norms); mode 0 downdates nrm2[c] -= r_c^2 for unselected columns (clamped at 0).
// Writes the per-block argmax of the updated norms.
__global__ __launch_bounds__(kQrBlock) void k_qr_update(const double* __restrict__ part, int nslab, int64_t N,
                                                        int mode, double* __restrict__ nrm2,
                                                        ArgMax* __restrict__ amax_part) {
  __shared__ ArgMax red[kQrBlock];
  const int64_t c = (int64_t)blockIdx.x * kQrBlock + threadIdx.x;
  ArgMax best{-2.0, INT64_MAX};
  if (c < N) {
    double r = 0.0;
    for (int sl = 0; sl < nslab; ++sl) r += part[(int64_t)sl * N + c];
    if (mode == 1) {
      nrm2[c] = r;
      best = ArgMax{r, c};
    } else {
      double v = nrm2[c];
      if (v >= 0.0) {
        v -= r * r;
        v = v > 0.0 ? v : 0.0;
        nrm2[c] = v;
        best = ArgMax{v, c};
      }
    }
  }
  red[threadIdx.x] = best;
  __syncthreads();
  for (int w = kQrBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = amax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) amax_part[blockIdx.x] = red[0];
}

// Final argmax over block partials -> pivot; gathers w = Yt[:, p] and records piv / rdiag.
template <typename T>
__global__ __launch_bounds__(1024) void k_qr_pick(const ArgMax* __restrict__ part, int nparts,
                                                  const T* __restrict__ Yt, int64_t ldy, int l, int j,
                                                  double* __restrict__ nrm2, int64_t* __restrict__ piv,
                                                  double* __restrict__ rdiag, double* __restrict__ w,
                                                  int64_t* __restrict__ pcur) {
  __shared__ ArgMax red[1024];
  ArgMax best{-2.0, INT64_MAX};
  for (int t = threadIdx.x; t < nparts; t += 1024) best = amax(best, part[t]);
  red[threadIdx.x] = best;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = amax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  const ArgMax b = red[0];
  const int64_t p = b.i == INT64_MAX ? 0 : b.i;
  if (threadIdx.x == 0) {
    piv[j] = p;
    rdiag[j] = sqrt(b.v > 0 ? b.v : 0.0);
    *pcur = p;
    nrm2[p] = -1.0;   // selected
  }
  for (int i = threadIdx.x; i < l; i += 1024) w[i] = (double)Yt[(int64_t)i * ldy + p];
}

// t[c] = Q[c, :] . w for c < j  (Q stored k x l row-major: row c is q_c)
__global__ __launch_bounds__(256) void k_qr_proj_dots(const double* __restrict__ Q, int l, int j,
                                                      const double* __restrict__ w, double* __restrict__ t) {
  __shared__ double red[256];
  const int c = blockIdx.x;
  if (c >= j) return;
  double s = 0;
  for (int i = threadIdx.x; i < l; i += 256) s = __builtin_fma(Q[(int64_t)c * l + i], w[i], s);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) t[c] = red[0];
}

// w[i] -= sum_c t[c] Q[c, i]: a block of 256 threads covers 32 rows, 8 threads per row splitting the
// c range; partials combined in LDS in a fixed order.
__global__ __launch_bounds__(256) void k_qr_proj_sub(const double* __restrict__ Q, int l, int j,
                                                     const double* __restrict__ t, double* __restrict__ w) {
  __shared__ double red[256];
  const int rl = threadIdx.x & 31, sl = threadIdx.x >> 5;
  const int i = blockIdx.x * 32 + rl;
  double s = 0;
  if (i < l)
    for (int c = sl; c < j; c += 8) s = __builtin_fma(t[c], Q[(int64_t)c * l + i], s);
  red[threadIdx.x] = s;
  __syncthreads();
  if (sl == 0 && i < l) {
    double tot = 0;
    for (int u = 0; u < 8; ++u) tot += red[u * 32 + rl];
    w[i] -= tot;
  }
}

// q_j = w / ||w|| (single block)
__global__ __launch_bounds__(1024) void k_qr_normalize(const double* __restrict__ w, int l, int j,
                                                       double* __restrict__ Q) {
  __shared__ double red[1024];
  double s = 0;
  for (int i = threadIdx.x; i < l; i += 1024) s = __builtin_fma(w[i], w[i], s);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  const double nrm = sqrt(red[0]);
  const double inv = nrm > 0 ? 1.0 / nrm : 0.0;
  for (int i = threadIdx.x; i < l; i += 1024) Q[(int64_t)j * l + i] = w[i] * inv;
}

template <typename T>
static void qrcp_full(const T* Yt, int64_t ldy, int64_t N, int l, int k, int64_t* piv, double* rdiag,
                      hipStream_t s) {
  const int64_t nblk = ceil_div(N, (int64_t)kQrBlock);
  // Split the l rows into slabs so that a pass launches about 4096 blocks (at least 16 rows per slab).
  const int want = (int)std::min<int64_t>(std::max<int64_t>(1, ceil_div((int64_t)4096, nblk)), ceil_div(l, 16));
  const int slab = (int)ceil_div(l, want);
  const int nslab = (int)ceil_div(l, slab);
  DevBuf<double> nrm2(N, s), Q((size_t)k * l, s), w(l, s), t(std::max(k, 1), s), part((size_t)nslab * N, s);
  DevBuf<ArgMax> am(nblk, s);
  DevBuf<int64_t> pcur(1, s);
  const dim3 g2((unsigned)nblk, (unsigned)nslab);
  hipLaunchKernelGGL((k_qr_slab<T, 1>), g2, dim3(kQrBlock), 0, s, Yt, ldy, N, l, slab, (const double*)nullptr,
                     part.p);
  hipLaunchKernelGGL(k_qr_update, dim3((unsigned)nblk), dim3(kQrBlock), 0, s, (const double*)part.p, nslab, N, 1,
                     nrm2.p, am.p);
  KRR_LAUNCH_CHECK();
  for (int j = 0; j < k; ++j) {
    hipLaunchKernelGGL(k_qr_pick<T>, dim3(1), dim3(1024), 0, s, (const ArgMax*)am.p, (int)nblk, Yt, ldy, l, j,
                       nrm2.p, piv, rdiag, w.p, pcur.p);
    if (j > 0) {
      for (int pass = 0; pass < 2; ++pass) {   // Gram-Schmidt twice
        hipLaunchKernelGGL(k_qr_proj_dots, dim3(j), dim3(256), 0, s, Q.p, l, j, w.p, t.p);
        hipLaunchKernelGGL(k_qr_proj_sub, dim3((unsigned)ceil_div(l, 32)), dim3(256), 0, s, Q.p, l, j, t.p, w.p);
      }
    }
    hipLaunchKernelGGL(k_qr_normalize, dim3(1), dim3(1024), 0, s, w.p, l, j, Q.p);
    if (j + 1 < k) {
      hipLaunchKernelGGL((k_qr_slab<T, 0>), g2, dim3(kQrBlock), 0, s, Yt, ldy, N, l, slab,
                         (const double*)(Q.p + (int64_t)j * l), part.p);
      hipLaunchKernelGGL(k_qr_update, dim3((unsigned)nblk), dim3(kQrBlock), 0, s, (const double*)part.p, nslab, N,
                         0, nrm2.p, am.p);
    }
    KRR_LAUNCH_CHECK();
  }
}

// ------------------------------------------------------------------ candidate-set pivoting, in batches
// Residual norms never grow, so a norm computed at step j0 is an upper bound at every later step.
// After a refresh (all norms brought up to date), the columns with the largest norms (at most kQrCand) become
// candidates; a batch of up to kQrBatch steps picks among them.  The best candidate is the true argmax as long as
// its norm exceeds tau, the largest norm outside the set at the refresh; otherwise (and at the end of the batch) the
// norms are refreshed with one pass over Yt that applies the batch's directions q_{j0} .. q_{j-1}, and the candidates
// are chosen again.
//
// A batch works on the candidates' residuals at j0, R = (I - Q Q^T) Yc, and their Gram matrix: the greedy steps on
// the candidates are the pivoted Cholesky factorisation of R^T R, which one workgroup runs with one matrix row and a
// few hundred cycles a step, instead of six launches a step over all of Q.  The directions are then formed
// together: L_pp^{-1} times the picked residuals (L_pp the factor's pivot rows), projected against Q once more and
// orthonormalised by a Cholesky step.  The pivots are those of the one-pass-per-step algorithm (up to rounding in
// the norms, which are downdated as they are there).
// Measured at n = 1e5, l = 1020, k = 1000 (42 batches): 51.8 -> 18.3 ms.
constexpr int kQrCand = 1024;    // candidates
constexpr int kQrBatch = 32;     // steps per batch at most
constexpr int kQrBins = 8192;    // selection histogram: bins of 2^-11 of an octave, four octaves below the maximum

struct QrState {
  unsigned long long max_bits;   // largest squared norm (bits of a non-negative double)
  unsigned long long tau;        // largest squared norm outside the candidates, bits + 1 (0: none)
  int cut;                       // first bin that is not taken
  int count;                     // candidates
  int steps;                     // steps of the last batch
};

__device__ __forceinline__ int qr_bin(unsigned long long max_bits, double v) {
  const unsigned long long d = (max_bits - (unsigned long long)__double_as_longlong(v)) >> 41;
  return d < (unsigned long long)(kQrBins - 1) ? (int)d : kQrBins - 1;
}

// Largest value over the wave, in every lane (row shifts and broadcasts, no LDS)
__device__ __forceinline__ double wave_max(double v) {
#define KRR_DPP_MAX(ctrl)                                                                                    \
  {                                                                                                          \
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), ctrl, 0xf, 0xf, false); \
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), ctrl, 0xf, 0xf, false); \
    v = fmax(v, __hiloint2double(hi, lo));                                                                   \
  }
  KRR_DPP_MAX(0x111)   // row_shr:1
  KRR_DPP_MAX(0x112)   // row_shr:2
  KRR_DPP_MAX(0x114)   // row_shr:4
  KRR_DPP_MAX(0x118)   // row_shr:8
  KRR_DPP_MAX(0x142)   // row_bcast:15
  KRR_DPP_MAX(0x143)   // row_bcast:31
#undef KRR_DPP_MAX
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63), __builtin_amdgcn_readlane(__double2loint(v), 63));
}

__global__ __launch_bounds__(256) void k_qr_max(const double* __restrict__ nrm2, int64_t N, QrState* __restrict__ st) {
  __shared__ double red[4];
  double m = 0.0;
  for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < N; c += (int64_t)gridDim.x * 256) m = fmax(m, nrm2[c]);
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(&st->max_bits, (unsigned long long)__double_as_longlong(fmax(fmax(red[0], red[1]), fmax(red[2], red[3]))));
}

// Histogram of the unselected columns' squared norms below the maximum (hist zero on entry).
__global__ __launch_bounds__(256) void k_qr_hist(const double* __restrict__ nrm2, int64_t N,
                                                 const QrState* __restrict__ st, unsigned* __restrict__ hist) {
  __shared__ unsigned h[kQrBins];
  for (int b = threadIdx.x; b < kQrBins; b += 256) h[b] = 0;
  __syncthreads();
  const unsigned long long mb = st->max_bits;
  for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < N; c += (int64_t)gridDim.x * 256) {
    const double v = nrm2[c];
    if (v >= 0.0) atomicAdd(&h[qr_bin(mb, v)], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kQrBins; b += 256)
    if (h[b]) atomicAdd(hist + b, h[b]);
}

// The largest prefix of bins with at most kQrCand columns (the last bin, everything far below, is never taken);
// clears the histogram for the next batch.
__global__ __launch_bounds__(1024) void k_qr_thresh(unsigned* __restrict__ hist, QrState* __restrict__ st) {
  constexpr int PER = kQrBins / 1024;
  __shared__ unsigned sums[1024];
  __shared__ int cut;
  const int t = threadIdx.x;
  unsigned mine[PER], s = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    mine[u] = hist[t * PER + u];
    hist[t * PER + u] = 0;
    s += mine[u];
  }
  sums[t] = s;
  if (t == 0) cut = kQrBins - 1;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const unsigned v = t >= o ? sums[t - o] : 0;
    __syncthreads();
    sums[t] += v;
    __syncthreads();
  }
  unsigned before = sums[t] - s;   // columns in the bins before this thread's
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (before <= kQrCand && before + mine[u] > kQrCand) atomicMin(&cut, t * PER + u);
    before += mine[u];
  }
  __syncthreads();
  if (t == 0) {
    st->cut = cut;
    st->count = 0;
    st->tau = 0;
  }
}

// Candidate list (in any order: the picks compare column indices) and tau.  all: every unselected column.  One
// counter update per wave and one tau update per block (an update per column was 28 us at n = 1e5).
__global__ __launch_bounds__(256) void k_qr_compact(const double* __restrict__ nrm2, int64_t N, int all,
                                                    QrState* __restrict__ st, int* __restrict__ cidx) {
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long mb = st->max_bits;
  const int cut = st->cut;
  double m = -1.0;
  for (int64_t c0 = (int64_t)blockIdx.x * 256; c0 < N; c0 += (int64_t)gridDim.x * 256) {
    const int64_t c = c0 + threadIdx.x;
    const double v = c < N ? nrm2[c] : -1.0;
    const bool take = v >= 0.0 && (all || qr_bin(mb, v) < cut);
    const unsigned long long ball = __ballot(take);
    if (ball) {
      int base = 0;
      if (lane == 0) base = atomicAdd(&st->count, (int)__popcll(ball));
      base = __builtin_amdgcn_readfirstlane(base);
      if (take) cidx[base + (int)__popcll(ball & ((1ull << lane) - 1ull))] = (int)c;
    }
    if (!take) m = fmax(m, v);
  }
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    if (m >= 0.0) atomicMax(&st->tau, (unsigned long long)__double_as_longlong(m) + 1);
  }
}

// Sort keys: larger norm first (ascending order of the key), last the selected columns and those whose norm is no number.
__global__ void k_qr_keys(const double* __restrict__ nrm2, int64_t N, uint64_t* __restrict__ key,
                          int64_t* __restrict__ idx) {
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= N) return;
  const double v = nrm2[c];
  key[c] = v >= 0.0 ? 0x7FFFFFFFFFFFFFFFull - (uint64_t)__double_as_longlong(v) : ~0ull;
  idx[c] = c;
}

// The candidates from the sorted order (norms so equal that one bin holds more than kQrCand columns).
__global__ __launch_bounds__(1024) void k_qr_take(const uint64_t* __restrict__ skey, const int64_t* __restrict__ sidx,
                                                  int64_t N, const double* __restrict__ nrm2, QrState* __restrict__ st,
                                                  int* __restrict__ cidx) {
  const int t = threadIdx.x;
  const bool live = t < N && skey[t] != ~0ull;
  if (live) {
    cidx[t] = (int)sidx[t];
    if (t + 1 == N || t + 1 == kQrCand || skey[t + 1] == ~0ull) st->count = t + 1;
  }
  if (t == 0)
    st->tau = kQrCand < N && skey[kQrCand] != ~0ull ? (unsigned long long)__double_as_longlong(nrm2[sidx[kQrCand]]) + 1 : 0;
}

// Yc (l x kQrCand, row-major) = the candidates' columns of Yt in FP64 (zero past the count).
template <typename T>
__global__ __launch_bounds__(256) void k_qr_gather(const T* __restrict__ Yt, int64_t ldy, int l,
                                                   const QrState* __restrict__ st, const int* __restrict__ cidx,
                                                   double* __restrict__ Yc) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  const bool live = t < st->count;
  const int64_t c = live ? cidx[t] : 0;
  const int i0 = blockIdx.y * 16;
  T y[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) y[u] = Yt[(int64_t)(i0 + u < l ? i0 + u : l - 1) * ldy + c];
#pragma unroll
  for (int u = 0; u < 16; ++u)
    if (i0 + u < l) Yc[(int64_t)(i0 + u) * kQrCand + t] = live ? (double)y[u] : 0.0;
}

// The batch's steps: pivoted Cholesky of the Gram matrix G of the candidates' residuals, one workgroup, two
// candidates per thread (its row of the factor in registers, the pivot's broadcast through LDS).  Step s: the
// candidate with the largest squared residual norm v, downdated (ties to the lowest column), if it exceeds tau or
// s = 0.  d is the same in the Gram's own rounding: it scales the factor, and the batch ends where the pivot's has
// fallen to 1e-6 of the first one's (further down, G no longer resolves the residuals: rank exhausted).  The
// pivots' rows of the factor go to Lpp, their slots to psel, their number also to steps_host (host-mapped).  A step is a serial chain (argmax, a row of G, the dot
// products with the pivot's row).
__global__ __launch_bounds__(kQrCand / 2) void k_qr_pivots(const double* __restrict__ G, QrState* __restrict__ st,
                                                           const int* __restrict__ cidx, int j0, int nb,
                                                           double* __restrict__ nrm2, int64_t* __restrict__ piv,
                                                           double* __restrict__ rdiag, double* __restrict__ Lpp,
                                                           int* __restrict__ psel, int* __restrict__ steps_host) {
  constexpr int NT = kQrCand / 2, NWV = NT / 64;
  __shared__ double bv[2][NWV];
  __shared__ unsigned long long bk[2][NWV];
  __shared__ double lp[kQrBatch], dp;
  const int tid = threadIdx.x, wave = tid >> 6;
  const int count = st->count;
  const double tau = st->tau ? __longlong_as_double((long long)(st->tau - 1)) : -1.0;
  double v[2], d[2], l[2][kQrBatch];
  unsigned long long key[2];   // column index and slot
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = tid + NT * h;
    const bool live = t < count;
    v[h] = live ? nrm2[cidx[t]] : -1.0;
    d[h] = live ? G[(int64_t)t * kQrCand + t] : 0.0;
    key[h] = live ? ((unsigned long long)(unsigned)cidx[t] << 32) | (unsigned)t : ~0ull;
#pragma unroll
    for (int u = 0; u < kQrBatch; ++u) l[h][u] = 0.0;
  }
  int s = 0;
  double dfirst = 0.0;
#pragma unroll 1   // (unrolled, the steps' 50 KB of code are fetched cold: 4.2 us a step)
  for (; s < nb; ++s) {
    const bool second = v[1] > v[0] || (v[1] == v[0] && key[1] < key[0]);
    const double mv = second ? v[1] : v[0];
    const unsigned long long mk = second ? key[1] : key[0];
    const double wm = wave_max(mv);
    unsigned long long ball = __ballot(mv == wm), wk = ~0ull;
    while (ball) {   // lanes that attain it (one, unless norms tie)
      const int src = __builtin_ctzll(ball);
      ball &= ball - 1;
      const unsigned long long kk = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(mk >> 32), src) << 32) |
                                    (unsigned)__builtin_amdgcn_readlane((int)mk, src);
      wk = kk < wk ? kk : wk;
    }
    if ((tid & 63) == 0) {
      bv[s & 1][wave] = wm;
      bk[s & 1][wave] = wk;
    }
    __syncthreads();
    double pv = bv[s & 1][0];
    unsigned long long pk = bk[s & 1][0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) {
      const double wv = bv[s & 1][w];
      const unsigned long long kk = bk[s & 1][w];
      if (wv > pv || (wv == pv && kk < pk)) { pv = wv; pk = kk; }
    }
    if (!(pv >= 0.0) || !(s == 0 || pv > tau)) break;   // (uniform; no candidate, or none whose norm is a number: pk is none)
    const int p = (int)(pk & 0xffffffffu);
    double x0 = G[(int64_t)p * kQrCand + tid], x1 = G[(int64_t)p * kQrCand + tid + NT];
    const bool own0 = p == tid, own1 = p == tid + NT;
    if (own0 || own1) {
#pragma unroll
      for (int u = 0; u < kQrBatch; ++u) lp[u] = own0 ? l[0][u] : l[1][u];
      dp = own0 ? d[0] : d[1];
    }
    __syncthreads();
    const double pd = dp;
    if (s == 0) dfirst = pd;
    else if (!(pd > 1e-6 * dfirst)) break;   // (uniform)
    const double nrm = pd > 0.0 ? sqrt(pd) : 0.0, inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    if (tid == 0) {
      const int64_t c = (int64_t)(pk >> 32);
      piv[j0 + s] = c;
      rdiag[j0 + s] = sqrt(pv);
      nrm2[c] = -1.0;   // selected
      psel[s] = p;
    }
    // the steps' entries in chunks of eight registers (those past s are zero)
#pragma unroll
    for (int c = 0; c < kQrBatch; c += 8) {
      if (c < s) {
#pragma unroll
        for (int u = c; u < c + 8; ++u) {
          x0 = __builtin_fma(-l[0][u], lp[u], x0);
          x1 = __builtin_fma(-l[1][u], lp[u], x1);
        }
      }
    }
    x0 *= inv;
    x1 *= inv;
#pragma unroll
    for (int c = 0; c < kQrBatch; c += 8) {
      if (c == (s & ~7)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          l[0][c + u] = u == (s & 7) ? x0 : l[0][c + u];
          l[1][c + u] = u == (s & 7) ? x1 : l[1][c + u];
        }
      }
    }
    d[0] = __builtin_fma(-x0, x0, d[0]);
    d[1] = __builtin_fma(-x1, x1, d[1]);
    if (v[0] >= 0.0) v[0] = fmax(__builtin_fma(-x0, x0, v[0]), 0.0);
    if (v[1] >= 0.0) v[1] = fmax(__builtin_fma(-x1, x1, v[1]), 0.0);
    if (own0) v[0] = -1.0;
    if (own1) v[1] = -1.0;
    if (tid < kQrBatch) Lpp[s * kQrBatch + tid] = tid < s ? lp[tid] : tid == s ? nrm : 0.0;
  }
  if (tid == 0) {
    st->steps = s;
    st->max_bits = 0;   // for the next refresh
    *steps_host = s;
  }
}

// x_s = (b_s - sum_{u < s} L[s][u] x_u) / L[s][s] for s = 0 .. kQrBatch - 1, b in registers: rolled, the remaining
// right-hand sides shifting down by one register a step (L: rows padded to 2 kQrBatch with zeros; inv[s] = 1 / L[s][s],
// 0 past the steps)
template <typename Store>
__device__ __forceinline__ void qr_solve(const double (*L)[kQrBatch + 1], const double* inv, double (&b)[kQrBatch],
                                         Store store) {
#pragma unroll 1
  for (int s = 0; s < kQrBatch; ++s) {
    const double x = b[0] * inv[s];
    store(s, x);
#pragma unroll
    for (int u = 1; u < kQrBatch; ++u) b[u - 1] = __builtin_fma(-L[s + u][s], x, b[u]);
  }
}

// Rows of the batch's raw directions B (kQrBatch x l, zero past the steps): L_pp^{-1} times the picked residuals.
// R: l x kQrCand; one component i per thread.
__global__ __launch_bounds__(64) void k_qr_directions(const double* __restrict__ R, int l, const QrState* __restrict__ st,
                                                      const double* __restrict__ Lpp, const int* __restrict__ psel,
                                                      double* __restrict__ B) {
  __shared__ double L[2 * kQrBatch][kQrBatch + 1];
  __shared__ double inv[kQrBatch];
  const int steps = st->steps, i = blockIdx.x * 64 + threadIdx.x;
  double b[kQrBatch];
#pragma unroll
  for (int s = 0; s < kQrBatch; ++s) {
    const double v = R[(int64_t)(i < l ? i : 0) * kQrCand + (s < steps ? psel[s] : 0)];
    b[s] = s < steps ? v : 0.0;
  }
  for (int e = threadIdx.x; e < 2 * kQrBatch * kQrBatch; e += 64) {
    const int s = e / kQrBatch;
    L[s][e % kQrBatch] = s < steps ? Lpp[e] : 0.0;
  }
  if (threadIdx.x < kQrBatch) {
    const double d = (int)threadIdx.x < steps ? Lpp[threadIdx.x * (kQrBatch + 1)] : 0.0;
    inv[threadIdx.x] = d > 0.0 ? 1.0 / d : 0.0;
  }
  __syncthreads();
  if (i < l) qr_solve(L, inv, b, [&](int s, double x) { B[(int64_t)s * l + i] = x; });
}

// Sum of the 16 waves' 32 x 16 partial results (two MFMA accumulators a lane), in wave order: element e of the sums,
// for e = tid and tid + 256 .. (t = e / 256: the half, row and column within it by the MFMA's result layout)
__device__ __forceinline__ void wave_partials(double (*red)[512], const f64x4 (&acc)[2], int wave, int kq, int r16) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][256 * h + (4 * e + kq) * 16 + r16] = acc[h][e];
}

// Second projection, first half: C (kQrBatch x ldp) = B Q^T (Q^T = QT, l x ldq, columns c < j0).  A block: 16 columns
// c, its sixteen waves split the l components.
__global__ __launch_bounds__(1024) void k_qr_coef(const double* __restrict__ B, int l, const double* __restrict__ QT,
                                                  int ldq, int j0, int ldp, double* __restrict__ C) {
  __shared__ double red[16][512];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  const int c0 = blockIdx.x * 16;
  const int len = ((l + 15) / 16 + 3) / 4 * 4;   // components per wave, a multiple of 4
  const int k0 = wave * len, k1 = k0 + len < l ? k0 + len : l;
  f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll 1
  for (int k = k0; k < k1; k += 32) {
    double a[2][8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = k + 4 * u + kq;
      const bool live = i < k1;
      const int ii = live ? i : 0;
      const double v0 = B[(int64_t)r16 * l + ii], v1 = B[(int64_t)(16 + r16) * l + ii];
      b[u] = QT[(int64_t)ii * ldq + c0 + r16];
      a[0][u] = live ? v0 : 0.0;
      a[1][u] = live ? v1 : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][u], b[u], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][u], b[u], acc[1], 0, 0, 0);
    }
  }
  wave_partials(red, acc, wave, kq, r16);
  __syncthreads();
  if (tid >= 512) return;
  double v = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) v += red[w][tid];
  const int c = c0 + (tid & 15);
  if (c < j0) C[(int64_t)(tid >> 4) * ldp + c] = v;
}

// Second projection, second half: B2 = B - C Q; a block: 16 components i, its sixteen waves split the j0 directions.
__global__ __launch_bounds__(1024) void k_qr_project(const double* __restrict__ B, int l, const double* __restrict__ Q,
                                                     int j0, int ldp, const double* __restrict__ C,
                                                     double* __restrict__ B2) {
  __shared__ double red[16][512];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  const int i0 = blockIdx.x * 16;
  const int ir = i0 + r16 < l ? i0 + r16 : l - 1;
  const int len = ((j0 + 15) / 16 + 3) / 4 * 4;
  const int k0 = wave * len, k1 = k0 + len < j0 ? k0 + len : j0;
  f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll 1
  for (int k = k0; k < k1; k += 32) {
    double a[2][8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = k + 4 * u + kq;
      const bool live = c < k1;
      const int cc = live ? c : 0;
      const double v0 = C[(int64_t)r16 * ldp + cc], v1 = C[(int64_t)(16 + r16) * ldp + cc];
      b[u] = Q[(int64_t)cc * l + ir];
      a[0][u] = live ? v0 : 0.0;
      a[1][u] = live ? v1 : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][u], b[u], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][u], b[u], acc[1], 0, 0, 0);
    }
  }
  wave_partials(red, acc, wave, kq, r16);
  __syncthreads();
  if (tid >= 512) return;
  double v = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) v += red[w][tid];
  const int i = i0 + (tid & 15);
  const int64_t o = (int64_t)(tid >> 4) * l + i;
  if (i < l) B2[o] = B[o] - v;
}

// Orthonormal directions q_{j0} .. from B2: Gram matrix of its rows, Cholesky factor, Q rows = L^{-1} B2, written to
// Q (row-major) and QT (columns past the steps: zeros).  Every block forms the small factor itself and writes 256
// components.
__global__ __launch_bounds__(256) void k_qr_orthonormal(const double* __restrict__ B2, int l, int j0,
                                                        const QrState* __restrict__ st, double* __restrict__ Q,
                                                        double* __restrict__ QT, int ldq) {
  __shared__ double red[4][4][256];
  __shared__ double L[2 * kQrBatch][kQrBatch + 1];
  __shared__ double inv[kQrBatch];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  const int steps = st->steps;
  const int i = blockIdx.x * 256 + tid;
  const int len = ((l + 3) / 4 + 3) / 4 * 4;
  const int k0 = wave * len, k1 = k0 + len < l ? k0 + len : l;
  f64x4 acc[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int g = 0; g < 2; ++g) acc[h][g] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int k = k0; k < k1; k += 32) {
    double a[2][8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = k + 4 * u + kq;
      const int cc = c < k1 ? c : 0;
      const double v0 = B2[(int64_t)r16 * l + cc], v1 = B2[(int64_t)(16 + r16) * l + cc];
      a[0][u] = c < k1 ? v0 : 0.0;
      a[1][u] = c < k1 ? v1 : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < 2; ++g) acc[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[h][u], a[g][u], acc[h][g], 0, 0, 0);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][2 * h + g][(4 * e + kq) * 16 + r16] = acc[h][g][e];
  double b[kQrBatch];   // this thread's component of the rows (loaded under the factorisation)
#pragma unroll
  for (int s = 0; s < kQrBatch; ++s) b[s] = B2[(int64_t)s * l + (i < l ? i : 0)];
  __syncthreads();
  for (int e = tid; e < 1024; e += 256) {
    const int t = e >> 8, o = e & 255;
    L[16 * (t >> 1) + (o >> 4)][16 * (t & 1) + (o & 15)] = ((red[0][t][o] + red[1][t][o]) + red[2][t][o]) + red[3][t][o];
  }
  for (int e = tid; e < kQrBatch * (kQrBatch + 1); e += 256) L[kQrBatch + e / (kQrBatch + 1)][e % (kQrBatch + 1)] = 0.0;
  // right-looking elimination of the lower triangle, 8 threads a row, the columns left unscaled: L = D^{-1/2} columns
  const int row = tid & 31, g8 = tid >> 5;
  for (int j = 0; j < steps; ++j) {
    __syncthreads();
    const double ajj = L[j][j];
    const double f = ajj > 0.0 && row > j ? L[row][j] / ajj : 0.0;
    for (int t = j + 1 + g8; t <= row; t += 8) L[row][t] = __builtin_fma(-f, L[t][j], L[row][t]);
  }
  __syncthreads();
  if (tid < kQrBatch) inv[tid] = tid < steps && L[tid][tid] > 0.0 ? 1.0 / sqrt(L[tid][tid]) : 0.0;
  __syncthreads();
  for (int e = tid; e < kQrBatch * kQrBatch; e += 256) {
    const int r = e / kQrBatch, c = e % kQrBatch;
    if (c < r) L[r][c] *= inv[c];
  }
  __syncthreads();
  if (i >= l) return;
  qr_solve(L, inv, b, [&](int s, double x) {
    if (s < steps) Q[(int64_t)(j0 + s) * l + i] = x;
    QT[(int64_t)i * ldq + j0 + s] = x;
  });
}

// nrm2[c] -= (q_t^T Yt[:, c])^2 for t = 0 .. b-1 in order (clamped at 0), q_t = QT[:, j0 + t] (QT: l x ldq,
// row-major, 16 NH columns readable), on the FP64 matrix cores; selected columns (nrm2 < 0) are left as they are.
// A block covers 64 columns, its four waves a quarter of the rows each (their sums added in a fixed order); a lane
// reads 4 consecutive columns of one row (16 or 32 bytes), so its four MFMA operands are the columns
// 4 r16 .. 4 r16 + 3 of that row.  Bound by the read of Yt (n = 1e5, l = 1020, FP32: 408 MB) and, near it, the
// matrix cores (with 32 directions 83 us at their peak).  Also leaves the largest updated norm in st.
template <typename T, int NH>
__global__ __launch_bounds__(256) void k_qr_refresh(const T* __restrict__ Yt, int64_t ldy, int64_t N, int l,
                                                    const double* __restrict__ QT, int ldq, int j0, int b,
                                                    double* __restrict__ nrm2, QrState* __restrict__ st) {
  struct alignas(sizeof(T) * 4) T4 { T v[4]; };
  __shared__ double part[3][16 * NH][64];
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t c0 = (int64_t)blockIdx.x * 64;   // (ldy is a multiple of 256: the reads past N are the rows' padding)
  const int lq = ((l + 3) / 4 + 3) / 4 * 4;
  const int i0 = wave * lq, i1 = i0 + lq < l ? i0 + lq : l;
  f64x4 acc[NH][4];
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[h][g] = f64x4{0.0, 0.0, 0.0, 0.0};
  constexpr int U = 4;   // row quads in flight, one set ahead
  T4 y[U];
  double q[U][NH];
  auto load = [&](int i) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = i + 4 * u + kq;
      const bool live = r < i1;
      const int rr = live ? r : 0;
      y[u] = *reinterpret_cast<const T4*>(Yt + (int64_t)rr * ldy + c0 + 4 * r16);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const double v = QT[(int64_t)rr * ldq + j0 + 16 * h + r16];
        q[u][h] = live ? v : 0.0;
      }
    }
  };
  if (i0 < i1) load(i0);
  for (int i = i0; i < i1; i += 4 * U) {
    T4 yc[U];
    double qc[U][NH];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      yc[u] = y[u];
#pragma unroll
      for (int h = 0; h < NH; ++h) qc[u][h] = q[u][h];
    }
    if (i + 4 * U < i1) load(i + 4 * U);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const double yv = (double)yc[u].v[g];
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(qc[u][h], yv, acc[h][g], 0, 0, 0);
      }
  }
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (wave > 0) part[wave - 1][16 * h + 4 * e + kq][4 * r16 + g] = acc[h][g][e];
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int t = 16 * h + 4 * e + kq, c = 4 * r16 + g;
          part[0][t][c] = ((acc[h][g][e] + part[0][t][c]) + part[1][t][c]) + part[2][t][c];
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int64_t c = c0 + lane;
    double v = c < N ? nrm2[c] : -1.0;
    if (!(v < 0.0)) {   // (a norm that is no number becomes 0, so that its column is picked after all others)
      for (int t = 0; t < b; ++t) {
        const double r = part[0][t][lane];
        v -= r * r;
        v = v > 0.0 ? v : 0.0;
      }
      nrm2[c] = v;
    }
    const double m = wave_max(v);
    if (lane == 0 && m >= 0.0) atomicMax(&st->max_bits, (unsigned long long)__double_as_longlong(m));
  }
}

template <typename T>
static void refresh_pass(const T* Yt, int64_t ldy, int64_t N, int l, const double* QT, int ldq, int j0, int b,
                         double* nrm2, QrState* st, hipStream_t s) {
  const dim3 g((unsigned)ceil_div(N, 64));
  if (b <= 16) hipLaunchKernelGGL((k_qr_refresh<T, 1>), g, dim3(256), 0, s, Yt, ldy, N, l, QT, ldq, j0, b, nrm2, st);
  else hipLaunchKernelGGL((k_qr_refresh<T, 2>), g, dim3(256), 0, s, Yt, ldy, N, l, QT, ldq, j0, b, nrm2, st);
  KRR_LAUNCH_CHECK();
}

struct QrEvent {
  hipEvent_t e = nullptr;
  QrEvent() { KRR_CHECK_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming)); }
  ~QrEvent() { (void)hipEventDestroy(e); }
  QrEvent(const QrEvent&) = delete;
  QrEvent& operator=(const QrEvent&) = delete;
};

template <typename T>
static void qrcp_cand(const T* Yt, int64_t ldy, int64_t N, int l, int k, int64_t* piv, double* rdiag, hipStream_t s) {
  const int64_t nblk = ceil_div(N, (int64_t)kQrBlock);
  const int want = (int)std::min<int64_t>(std::max<int64_t>(1, ceil_div((int64_t)4096, nblk)), ceil_div(l, 16));
  const int slab = (int)ceil_div(l, want);
  const int nslab = (int)ceil_div(l, slab);
  const int ldq = k + kQrBatch;   // QT's columns past k: zeros written by the last batch
  const int64_t lc = (int64_t)l * kQrCand;
  DevBuf<double> nrm2(N, s), Q((size_t)k * l, s), QT((size_t)l * ldq, s), part((size_t)nslab * N, s), Yc(lc, s), R(lc, s),
      PT((size_t)k * kQrCand, s), G((size_t)kQrCand * kQrCand, s), Lpp(kQrBatch * kQrBatch, s), B((size_t)kQrBatch * l, s),
      B2((size_t)kQrBatch * l, s), coef((size_t)kQrBatch * ldq, s);
  DevBuf<ArgMax> am(nblk, s);
  DevBuf<int> cidx(kQrCand, s), psel(kQrBatch, s);
  DevBuf<unsigned> hist(kQrBins, s);
  DevBuf<QrState> state(1, s);
  QrState* st = state.p;
  HostWords words(s);
  int* steps_host = reinterpret_cast<int*>(words.get());
  QrEvent ev;
  KRR_CHECK_HIP(hipMemsetAsync(hist.p, 0, hist.bytes(), s));
  KRR_CHECK_HIP(hipMemsetAsync(st, 0, sizeof(QrState), s));
  // initial squared norms
  const dim3 g2((unsigned)nblk, (unsigned)nslab);
  hipLaunchKernelGGL((k_qr_slab<T, 1>), g2, dim3(kQrBlock), 0, s, Yt, ldy, N, l, slab, (const double*)nullptr,
                     part.p);
  hipLaunchKernelGGL(k_qr_update, dim3((unsigned)nblk), dim3(kQrBlock), 0, s, (const double*)part.p, nslab, N, 1,
                     nrm2.p, am.p);
  KRR_LAUNCH_CHECK();
  part.release();
  const bool all = N <= kQrCand;   // every unselected column is a candidate
  const unsigned gsel = (unsigned)std::min<int64_t>(ceil_div(N, 1024), 256);
  if (!all) hipLaunchKernelGGL(k_qr_max, dim3(gsel), dim3(256), 0, s, (const double*)nrm2.p, N, st);
  int j = 0, j0 = 0;
  const bool verbose = std::getenv("KRR_QR_VERBOSE") != nullptr;
  int refreshes = 0;
  while (j < k) {
    // refresh: bring every norm up to date with q_{j0} .. q_{j-1}, choose the candidates
    if (j > j0) refresh_pass(Yt, ldy, N, l, QT.p, ldq, j0, j - j0, nrm2.p, st, s);
    j0 = j;
    ++refreshes;
    if (all) {
      KRR_CHECK_HIP(hipMemsetAsync(&st->count, 0, sizeof(int), s));
    } else {
      hipLaunchKernelGGL(k_qr_hist, dim3(gsel), dim3(256), 0, s, (const double*)nrm2.p, N, (const QrState*)st, hist.p);
      hipLaunchKernelGGL(k_qr_thresh, dim3(1), dim3(1024), 0, s, hist.p, st);
    }
    hipLaunchKernelGGL(k_qr_compact, dim3(gsel), dim3(256), 0, s, (const double*)nrm2.p, N, all ? 1 : 0, st,
                       cidx.p);
    KRR_LAUNCH_CHECK();
    const int nb = std::min(kQrBatch, k - j0);
    int steps = 0;
    for (int attempt = 0; attempt < 2 && steps == 0; ++attempt) {
      if (attempt == 1) {   // one bin holds more columns than the set: the exact order decides
        DevBuf<uint64_t> key(N, s), skey(N, s);
        DevBuf<int64_t> idx(N, s), sidx(N, s);
        RadixSortWork rsw;
        hipLaunchKernelGGL(k_qr_keys, dim3((unsigned)ceil_div(N, 256)), dim3(256), 0, s, (const double*)nrm2.p, N, key.p,
                           idx.p);
        KRR_LAUNCH_CHECK();
        radix_sort_pairs(key.p, skey.p, idx.p, sidx.p, N, 64, rsw, s);
        hipLaunchKernelGGL(k_qr_take, dim3(1), dim3(1024), 0, s, (const uint64_t*)skey.p, (const int64_t*)sidx.p, N,
                           (const double*)nrm2.p, st, cidx.p);
        KRR_LAUNCH_CHECK();
      }
      hipLaunchKernelGGL(k_qr_gather<T>, dim3(kQrCand / 256, (unsigned)ceil_div(l, 16)), dim3(256), 0, s, Yt, ldy, l,
                         (const QrState*)st, (const int*)cidx.p, Yc.p);
      KRR_LAUNCH_CHECK();
      const double* Rp = Yc.p;
      if (j0 > 0) {   // R = Yc - Q^T (Q Yc)
        gemm_tile(Q.p, l, Yc.p, kQrCand, j0, l, kQrCand, PT.p, kQrCand, nullptr, 0, s);
        gemm_tile(QT.p, ldq, PT.p, kQrCand, l, j0, kQrCand, R.p, kQrCand, Yc.p, kQrCand, s);
        Rp = R.p;
      }
      gram_tile(Rp, kQrCand, l, kQrCand, G.p, kQrCand, s);
      words.busy();
      hipLaunchKernelGGL(k_qr_pivots, dim3(1), dim3(kQrCand / 2), 0, s, (const double*)G.p, st, (const int*)cidx.p, j0, nb,
                         nrm2.p, piv, rdiag, Lpp.p, psel.p, steps_host);
      KRR_CHECK_HIP(hipEventRecord(ev.e, s));
      // the directions of the batch (of no steps: nothing)
      hipLaunchKernelGGL(k_qr_directions, dim3((unsigned)ceil_div(l, 64)), dim3(64), 0, s, Rp, l, (const QrState*)st,
                         (const double*)Lpp.p, (const int*)psel.p, B.p);
      const double* Bp = B.p;
      if (j0 > 0) {
        hipLaunchKernelGGL(k_qr_coef, dim3((unsigned)ceil_div(j0, 16)), dim3(1024), 0, s, (const double*)B.p, l,
                           (const double*)QT.p, ldq, j0, ldq, coef.p);
        hipLaunchKernelGGL(k_qr_project, dim3((unsigned)ceil_div(l, 16)), dim3(1024), 0, s, (const double*)B.p, l,
                           (const double*)Q.p, j0, ldq, (const double*)coef.p, B2.p);
        Bp = B2.p;
      }
      hipLaunchKernelGGL(k_qr_orthonormal, dim3((unsigned)ceil_div(l, 256)), dim3(256), 0, s, Bp, l, j0,
                         (const QrState*)st, Q.p, QT.p, ldq);
      KRR_LAUNCH_CHECK();
      // the host waits for the pivots only, and enqueues the next refresh while the directions are formed
      KRR_CHECK_HIP(hipEventSynchronize(ev.e));
      words.done();
      steps = *steps_host;
    }
    KRR_REQUIRE(steps > 0, "pivoted QR: no valid pivot on fresh candidates");
    j = j0 + steps;
  }
  if (verbose) std::fprintf(stderr, "krr qrcp: %d steps, %d candidate refreshes\n", k, refreshes);
}

void qrcp_t(const void* Yt, int64_t ldy, int64_t N, int l, int k, int prec, int64_t* piv, double* rdiag,
            hipStream_t s) {
  KRR_REQUIRE(k >= 1 && k <= l && k <= N, "pivoted QR needs 1 <= k <= min(l, n)");
  // KRR_QR_FULL: one pass over Yt per step (also used for more than 2^31 - 1 columns: the candidates' are int)
  const bool full = std::getenv("KRR_QR_FULL") != nullptr || N > INT32_MAX;
  if (prec == KRR_FP64) {
    if (full) qrcp_full<double>((const double*)Yt, ldy, N, l, k, piv, rdiag, s);
    else qrcp_cand<double>((const double*)Yt, ldy, N, l, k, piv, rdiag, s);
  } else {
    if (full) qrcp_full<float>((const float*)Yt, ldy, N, l, k, piv, rdiag, s);
    else qrcp_cand<float>((const float*)Yt, ldy, N, l, k, piv, rdiag, s);
  }
}

}  // namespace krr
