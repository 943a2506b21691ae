// Blocked Cholesky factorisation and triangular inverse of the preconditioner's cores (Eq. chol_factor), FP64,
// trailing and off-diagonal products on v_mfma_f64_16x16x4_f64 (operand layouts as in gemm.hip).
#include "dense.h"

namespace krr {

typedef double f64x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kCB = 64;   // panel width

// 1 / sqrt(x) to a unit or two in the last place (hardware estimate, two Newton steps; x normal): the elimination
// steps are a serial chain, and the IEEE square root and divisions were most of it
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = __builtin_fma(0.5 * y, __builtin_fma(-x * y, y, 1.0), y);
  return __builtin_fma(0.5 * y, __builtin_fma(-x * y, y, 1.0), y);
}

// One panel of the right-looking factorisation: columns [j0, j0 + 64) of L.  Block 0 writes the diagonal block's
// factor, block b > 0 the 64 rows j0 + 64 b .. of L21 = A21 L11^{-T}.  Every block factors the diagonal block
// itself, its own 64 rows riding along as rows 64 .. 127 of the same elimination, so that a panel is one launch:
// the serial chain of its 64 steps bounds it, and repeating them in every block costs no time.
// Wave w holds the columns 16 w .. 16 w + 15 of all 128 rows (lane: rows lane, lane + 64), so that what a step does
// is the same in a whole wave; the steps are rolled loops, a wave's own columns shifting down by one register a step.
// (Broadcasting by lane reads inside a wave instead of LDS and a barrier a step was slower: 36 us.)
// A bad pivot (NaN from there on) is remembered and reported at the end.  A is only read, so that the blocks may start
// in any order; rows and columns past k are those of an identity.
__global__ __launch_bounds__(256) void k_chol_panel(const double* __restrict__ A, double* __restrict__ L, int k, int j0,
                                                    int* __restrict__ info) {
  __shared__ double col[kCB][128];   // the columns as eliminated, unscaled
  __shared__ double rsv[kCB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = j0 + lane, row1 = j0 + 64 * (int)blockIdx.x + lane;   // rows of L11; of L21 (riding along)
  const bool live1 = row1 < k && blockIdx.x != 0;
  const int stopped = *info;   // an earlier panel failed: this one computes nothing of use and stores nothing
  double a0[16], a1[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const int t = j0 + 16 * wave + c, tr = t < k ? t : k - 1;
    const double v0 = A[(int64_t)tr * k + (row0 < k ? row0 : k - 1)], v1 = A[(int64_t)tr * k + (row1 < k ? row1 : k - 1)];
    a0[c] = row0 < k && t <= row0 ? v0 : (row0 == t ? 1.0 : 0.0);
    a1[c] = live1 && t < k ? v1 : 0.0;
  }
  int bad = kCB;
  // the columns of earlier waves
#pragma unroll 1
  for (int j = 0; j < 16 * wave; ++j) {
    __syncthreads();
    const double ajj = col[j][j], rs = rsqrt_nr(ajj);
    if (!(ajj > 0.0) || !isfinite(ajj)) bad = bad < j ? bad : j;
    const double f0 = col[j][lane] * rs * rs, f1 = col[j][lane + 64] * rs * rs;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const double at = col[j][16 * wave + u];
      a0[u] = __builtin_fma(-f0, at, a0[u]);
      a1[u] = __builtin_fma(-f1, at, a1[u]);
    }
  }
  // this wave's own
#pragma unroll 1
  for (int c = 0; c < 16; ++c) {
    const int j = 16 * wave + c;
    col[j][lane] = a0[0];
    col[j][lane + 64] = a1[0];
    __syncthreads();
    const double ajj = col[j][j], rs = rsqrt_nr(ajj);
    if (!(ajj > 0.0) || !isfinite(ajj)) bad = bad < j ? bad : j;
    if (lane == 0) rsv[j] = rs;
    const double f0 = a0[0] * rs * rs, f1 = a1[0] * rs * rs;
#pragma unroll
    for (int u = 1; u < 16; ++u) {
      const double at = col[j][j + u];   // (past this wave's columns: registers never used)
      a0[u - 1] = __builtin_fma(-f0, at, a0[u]);
      a1[u - 1] = __builtin_fma(-f1, at, a1[u]);
    }
  }
  // the later waves' barriers
#pragma unroll 1
  for (int j = 16 * wave + 16; j <= kCB; ++j) __syncthreads();
  // the last wave has seen every pivot
  if (wave == 3 && lane == 0 && blockIdx.x == 0 && bad < kCB && !stopped) *info = j0 + bad + 1;
  if (stopped) return;
  const int r = lane, o = blockIdx.x == 0 ? 0 : 64, row = blockIdx.x == 0 ? row0 : row1;
#pragma unroll 4
  for (int c = wave; c < kCB; c += 4)
    if (j0 + c < k && row < k && (o || r >= c)) L[(int64_t)(j0 + c) * k + row] = col[c][o + r] * rsv[c];
}

// Trailing update A22 -= L21 L21^T after the panel at j0: one 64 x 64 tile of the lower triangle per block, wave w
// its rows 16 w .., the contraction over the panel's 64 columns.  The tile is formed transposed (operand A from the
// tile's columns, B from its rows), so that the 16 lanes of a result register are consecutive rows of one column.
__global__ __launch_bounds__(256) void k_chol_trail(double* __restrict__ A, const double* __restrict__ L, int k, int j0,
                                                    const int* __restrict__ info) {
  if (*info != 0) return;   // (written by an earlier launch)
  const int id = blockIdx.x;
  int ti = (int)((sqrt(8.0 * id + 1.0) - 1.0) / 2.0);
  while (ti * (ti + 1) / 2 > id) --ti;
  while ((ti + 1) * (ti + 2) / 2 <= id) ++ti;
  const int tj = id - ti * (ti + 1) / 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, kq = lane >> 4;
  const int row = j0 + kCB + kCB * ti + 16 * wave + r16;
  const int c0 = j0 + kCB + kCB * tj;
  const int rr = row < k ? row : k - 1;
  double b[16];
#pragma unroll
  for (int kc = 0; kc < 16; ++kc) b[kc] = L[(int64_t)(j0 + 4 * kc + kq) * k + rr];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int cr = c0 + 16 * u + r16 < k ? c0 + 16 * u + r16 : k - 1;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kc = 0; kc < 16; ++kc)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(L[(int64_t)(j0 + 4 * kc + kq) * k + cr], b[kc], acc, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = c0 + 16 * u + 4 * e + kq;
      if (row < k && c <= row) A[(int64_t)c * k + row] -= acc[e];
    }
  }
}

// Dinv[b] (64 x 64 row-major) = inverse of L's b-th diagonal block (identity past k): wave w inverts the 16 x 16
// diagonal block w by substitution (lane c its column c), then X21 = -X22 L21 X11 joins pairs of blocks of 16 and
// of 32 on the matrix cores.
__global__ __launch_bounds__(256) void k_tri_inv_diag(const double* __restrict__ L, int k, double* __restrict__ Dinv) {
  __shared__ double S[kCB][kCB + 1], X[kCB][kCB + 1], Y[32][33];
  const int j0 = blockIdx.x * kCB, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  for (int e = tid; e < kCB * kCB; e += 256) {
    const int i = e % kCB, t = e / kCB;
    S[i][t] = t <= i && j0 + i < k ? L[(int64_t)(j0 + t) * k + j0 + i] : (t == i ? 1.0 : 0.0);
    X[i][t] = 0.0;
  }
  __syncthreads();
  {
    const int o = 16 * wave;
    double x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = i == r16 ? 1.0 : 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      x[i] /= S[o + i][o + i];
#pragma unroll
      for (int t = i + 1; t < 16; ++t) x[t] = __builtin_fma(-S[o + t][o + i], x[i], x[t]);
    }
    if (kq == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) X[o + i][o + r16] = x[i];
    }
  }
  __syncthreads();
  // tile (16 x 16) at (dr, dc) of -P Q or P Q over K terms: rows pr .. of P, columns qc .. of Q
  auto product = [&](const double* P, int lp, const double* Q, int lq, int K) {
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
    for (int t = 0; t < K; t += 4) d = __builtin_amdgcn_mfma_f64_16x16x4f64(P[r16 * lp + t + kq], Q[(t + kq) * lq + r16], d, 0, 0, 0);
    return d;
  };
  constexpr int ld = kCB + 1;
  // blocks of 16: pair w (w < 2) joins diagonal blocks 2 w, 2 w + 1
  f64x4 d = {0.0, 0.0, 0.0, 0.0};
  if (wave < 2) {
    const int o = 32 * wave;
    d = product(&S[o + 16][o], ld, &X[o][o], ld, 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) Y[16 * wave + 4 * e + kq][r16] = d[e];
  }
  __syncthreads();
  if (wave < 2) {
    const int o = 32 * wave;
    d = product(&X[o + 16][o + 16], ld, &Y[16 * wave][0], 33, 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) X[o + 16 + 4 * e + kq][o + r16] = -d[e];
  }
  __syncthreads();
  // blocks of 32: wave w forms the tile (w / 2, w % 2)
  const int ti = 16 * (wave >> 1), tj = 16 * (wave & 1);
  d = product(&S[32 + ti][0], ld, &X[0][tj], ld, 32);
#pragma unroll
  for (int e = 0; e < 4; ++e) Y[ti + 4 * e + kq][tj + r16] = d[e];
  __syncthreads();
  d = product(&X[32 + ti][32], ld, &Y[0][tj], 33, 32);
#pragma unroll
  for (int e = 0; e < 4; ++e) X[32 + ti + 4 * e + kq][tj + r16] = -d[e];
  __syncthreads();
  double* out = Dinv + (int64_t)blockIdx.x * kCB * kCB;
  for (int e = tid; e < kCB * kCB; e += 256) out[e] = X[e / kCB][e % kCB];
}

// X = L^{-1} (row-major), 16 columns per block: block rows i = c0 / 64 .. in turn,
// X_i = Dinv_i (E_i - sum_{t < i} L_it X_t), wave w the rows 16 w .. of a block row.  The columns are independent
// and the sequential chain is k / 64 block rows long; the finished rows are read back from global memory (the
// block's own writes).
__global__ __launch_bounds__(256) void k_tri_inv_cols(const double* __restrict__ L, const double* __restrict__ Dinv, int k,
                                                      double* X) {
  __shared__ double R[kCB][17];
  const int c0 = blockIdx.x * 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, kq = lane >> 4;
  const int cb = c0 / kCB, nb = (k + kCB - 1) / kCB;
  const bool cl = c0 + r16 < k;
  const int cx = cl ? c0 + r16 : k - 1;   // (dead columns repeat the last one and are not stored)
  for (int e = threadIdx.x; e < cb * kCB * 16; e += 256)
    if (c0 + e % 16 < k) X[(int64_t)(e / 16) * k + c0 + e % 16] = 0.0;
  for (int i = cb; i < nb; ++i) {
    const int row = i * kCB + 16 * wave + r16;
    const double* lp = L + (row < k ? row : k - 1);
    f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
    for (int t0 = cb * kCB; t0 < i * kCB; t0 += 32) {   // whole blocks: every t below is < k
      double a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = t0 + 4 * u + kq;
        a[u] = lp[(int64_t)t * k];
        b[u] = X[(int64_t)t * k + cx];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[u & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc[u & 1], 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int rl = 16 * wave + 4 * e + kq;
      R[rl][r16] = (i * kCB + rl == c0 + r16 ? 1.0 : 0.0) - (acc[0][e] + acc[1][e]);
    }
    __syncthreads();
    const double* D = Dinv + (int64_t)i * kCB * kCB + (16 * wave + r16) * kCB;
    f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kc = 0; kc < 16; ++kc)
      x = __builtin_amdgcn_mfma_f64_16x16x4f64(D[4 * kc + kq], R[4 * kc + kq][r16], x, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = i * kCB + 16 * wave + 4 * e + kq;
      if (r < k && cl) X[(int64_t)r * k + c0 + r16] = x[e];
    }
    __syncthreads();
  }
}

}  // namespace

int cholesky_lower(double* A, double* L, int k, hipStream_t s) {
  DevBuf<int> info(1, s);
  KRR_CHECK_HIP(hipMemsetAsync(info.p, 0, sizeof(int), s));
  KRR_CHECK_HIP(hipMemsetAsync(L, 0, sizeof(double) * (size_t)k * k, s));
  for (int j0 = 0; j0 < k; j0 += kCB) {
    const int nb = (int)ceil_div(k - j0, kCB);
    hipLaunchKernelGGL(k_chol_panel, dim3((unsigned)nb), dim3(256), 0, s, A, L, k, j0, info.p);
    if (nb > 1)
      hipLaunchKernelGGL(k_chol_trail, dim3((unsigned)(nb * (nb - 1) / 2)), dim3(256), 0, s, A, L, k, j0, info.p);
    KRR_LAUNCH_CHECK();
  }
  int h = 0;
  KRR_CHECK_HIP(hipMemcpyAsync(&h, info.p, sizeof(int), hipMemcpyDeviceToHost, s));
  KRR_CHECK_HIP(hipStreamSynchronize(s));
  return h;
}

void lower_inverse(const double* L, double* X, int k, hipStream_t s) {
  const int nb = (int)ceil_div(k, kCB);
  DevBuf<double> Dinv((size_t)nb * kCB * kCB, s);
  hipLaunchKernelGGL(k_tri_inv_diag, dim3((unsigned)nb), dim3(256), 0, s, L, k, Dinv.p);
  hipLaunchKernelGGL(k_tri_inv_cols, dim3((unsigned)ceil_div(k, 16)), dim3(256), 0, s, L, Dinv.p, k, X);
  KRR_LAUNCH_CHECK();
}

}  // namespace krr
