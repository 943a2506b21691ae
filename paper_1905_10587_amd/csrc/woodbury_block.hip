// The preconditioner's apply to 2 .. 16 columns at once: out = (X - W Z) diag(1 / beta), Z_r = G_{beta_r} (W^T X)_r.
//
// Both passes over W are bound by reading it (29 MB at 12000 x 600 in FP32), and by latency where it is smaller: so a wave
// loads four neighbouring values of W a lane and feeds them to FP64 matrix instructions of 16 columns as they lie, without
// LDS, and the rows (W^T X, G T) or the columns (W Z) are split until every compute unit has blocks.  General tiles of 128
// x 16 through LDS left most of the chip idle here: 3500 rows, 350 columns, four right-hand sides: W^T X 70 us, now 5,
// W Z 57 us, now 5; 12000 rows, 600 columns, sixteen: 86 and 105 us, now 11 and 11.
#include "precond.h"

namespace krr {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kC = kBlockColumns;   // columns of X, T and Z (padded): one tile

// The values of row p at columns c .. c + 3 (rows are aligned to their element only).  Past the row's end: with FAST
// whatever follows it, at most three values and only where rows follow, so that the loop's loads have no branch and go
// out together; zeros otherwise.  Either is finite, and meets a row of T that is not used or a zero row of Z.
template <bool FAST, typename TW>
__device__ __forceinline__ void load4(const TW* p, int c, int kept, double (&v)[4]) {
  TW t[4] = {TW(0), TW(0), TW(0), TW(0)};
  if (FAST) {
    __builtin_memcpy(t, p + (c < kept ? c : 0), sizeof(t));
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (c + s < kept) t[s] = p[c + s];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) v[s] = (double)t[s];
}

// part[y, c, r] = sum over rows [y rows, (y + 1) rows) of W[i, c] X[i, r] for the block's 64 columns c (kp: columns padded
// to 64).  Lane l of wave w: rows 4 w + l / 16 of every 16, columns 4 (l % 16) .. + 3; instruction s takes column 4 m + s as
// its row m.  rows is a multiple of 16.
template <typename TW>
__global__ __launch_bounds__(256) void k_wb_tn(const TW* __restrict__ W, int64_t n, int kept, int kp,
                                               const double* __restrict__ X, int ldx, int R, int64_t rows,
                                               double* __restrict__ part) {
  __shared__ double red[4][16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, m = lane & 15, k = lane >> 4;
  const int c0 = blockIdx.x * 64, c = c0 + 4 * m;
  const int64_t r0 = (int64_t)blockIdx.y * rows, r1 = r0 + rows < n ? r0 + rows : n;
  f64x4 acc[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = f64x4{0.0, 0.0, 0.0, 0.0};
  // whole sixteens with three more rows behind them, then the rest
  const int64_t whole = r1 + 3 <= n ? r1 : r0 + (r1 - r0 > 3 ? (r1 - r0 - 3) / 16 * 16 : 0);
  const int xm = m < R ? m : 0;
#pragma unroll 4
  for (int64_t j = r0; j < whole; j += 16) {
    const int64_t i = j + 4 * w + k;
    double a[4];
    load4<true>(W + i * kept, c, kept, a);
    const double x = X[i * ldx + xm];   // (columns past R are not used)
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], x, acc[s], 0, 0, 0);
  }
  for (int64_t j = whole; j < r1; j += 16) {
    const int64_t i = j + 4 * w + k;
    const bool in = i < r1;
    double a[4];
    load4<false>(W + (in ? i : r0) * kept, c, kept, a);
    const double x = in ? X[i * ldx + xm] : 0.0;
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], x, acc[s], 0, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[w][4 * s + e][lane] = acc[s][e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int u = 4 * w + e;   // s = w: column 4 (4 e + k) + w
    const double v = ((red[0][u][lane] + red[1][u][lane]) + red[2][u][lane]) + red[3][u][lane];
    part[((int64_t)blockIdx.y * kp + c0 + 4 * (4 * e + k) + w) * kC + m] = v;
  }
}

// out[c, r] = sum over the S splits; zeros in rows from kept on.  With bidx: only the columns r whose beta is b (and those
// past R, which hold no use).
__global__ __launch_bounds__(256) void k_wb_sum(const double* __restrict__ part, int S, int kept, int kp,
                                                const int* __restrict__ bidx, int R, int b, double* __restrict__ out) {
  __shared__ double sum[3][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t idx = (int64_t)blockIdx.x * 64 + lane;   // kp * kC of them: whole blocks
  double v = 0.0;
#pragma unroll 8
  for (int s = w; s < S; s += 4) v += part[(int64_t)s * kp * kC + idx];
  if (w) sum[w - 1][lane] = v;
  __syncthreads();
  if (w) return;
  const int c = (int)(idx / kC), r = (int)(idx % kC);
  if (bidx && r < R && bidx[r] != b) return;
  out[idx] = c < kept ? ((v + sum[0][lane]) + sum[1][lane]) + sum[2][lane] : 0.0;
}

// out[i, r] = (X[i, r] - sum_c W[i, c] Z[c, r]) invb[r], 16 rows to a block, every fourth 16 columns to a wave.  Lane l:
// row l % 16, columns 4 (l / 16) .. + 3 of the 16; instruction s takes column 4 k + s as its k-th.  (X may be out.)
template <typename TW>
__global__ __launch_bounds__(256) void k_wb_nz(const TW* __restrict__ W, int64_t n, int kept,
                                               const double* __restrict__ Z, const double* X, int R,
                                               const double* __restrict__ invb, double* out) {
  __shared__ double red[4][4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, m = lane & 15, k = lane >> 4;
  const int64_t i0 = (int64_t)blockIdx.x * 16;
  const TW* row = W + (i0 + m < n ? i0 + m : n - 1) * kept;
  f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
  auto run = [&](auto fast) {
#pragma unroll 4
    for (int c0 = 16 * w; c0 < kept; c0 += 64) {
      const int c = c0 + 4 * k;
      double a[4];
      load4<decltype(fast)::value>(row, c, kept, a);
#pragma unroll
      for (int s = 0; s < 4; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], Z[(int64_t)(c + s) * kC + m], acc, 0, 0, 0);
    }
  };
  if (i0 + 16 + 3 <= n) run(std::true_type{});
  else run(std::false_type{});
#pragma unroll
  for (int e = 0; e < 4; ++e) red[w][e][lane] = acc[e];
  __syncthreads();
  const double v = ((red[0][w][lane] + red[1][w][lane]) + red[2][w][lane]) + red[3][w][lane];
  const int64_t i = i0 + 4 * w + k;   // element e = w
  if (i < n && m < R) out[i * R + m] = (X[i * R + m] - v) * invb[m];
}

int padded_columns(int kept) { return (int)round_up(kept, 64); }

// Row splits for about 512 blocks, of 16 rows at least (64 a block keep the partial sums below a fourth of W).
int64_t split_rows(int64_t n, int kept) {
  const int64_t S = std::max<int64_t>(1, ceil_div(512, padded_columns(kept) / 64));
  return std::max<int64_t>(64, round_up(ceil_div(n, S), 16));
}

}  // namespace

void woodbury_block_prepare(const krr_precond& P, WoodburyWork& w, hipStream_t s) {
  const int kp = padded_columns(P.kept);
  const int64_t S = std::max(ceil_div(P.n, split_rows(P.n, P.kept)), ceil_div(P.kept, split_rows(P.kept, P.kept)));
  w.partial.alloc((size_t)(S * kp * kC), s);
  w.T.alloc((size_t)kp * kC, s);
  w.Z.alloc((size_t)kp * kC, s);
}

void woodbury_block_apply(const krr_precond& P, const double* X, WoodburyWork& w, bool use32, double* out, hipStream_t s) {
  const int kept = P.kept, kp = padded_columns(kept), R = w.R;
  const int64_t n = P.n;
  auto product_t = [&](auto* W, int64_t rows_of_w, const double* V, int ldv, int cols, const int* bidx, int b, double* o) {
    using TW = std::remove_cv_t<std::remove_pointer_t<decltype(W)>>;
    const int64_t rows = split_rows(rows_of_w, kept);
    const int S = (int)ceil_div(rows_of_w, rows);
    hipLaunchKernelGGL(k_wb_tn<TW>, dim3((unsigned)(kp / 64), (unsigned)S), dim3(256), 0, s, (const TW*)W, rows_of_w, kept,
                       kp, V, ldv, cols, rows, w.partial.p);
    hipLaunchKernelGGL(k_wb_sum, dim3((unsigned)(kp * kC / 64)), dim3(256), 0, s, (const double*)w.partial.p, S, kept, kp,
                       bidx, R, b, o);
  };
  if (use32) product_t(P.W32.p, n, X, R, R, nullptr, 0, w.T.p);
  else product_t(P.W64.p, n, X, R, R, nullptr, 0, w.T.p);
  // G is symmetric, so G T is a product of the same kind; each beta in use writes its columns
  for (size_t b = 0; b < P.betas.size(); ++b) {
    if (std::find(w.bidx_host.begin(), w.bidx_host.end(), (int)b) == w.bidx_host.end()) continue;
    product_t((use32 ? P.G32[b].p : P.G64[b].p), kept, (const double*)w.T.p, kC, kC, (const int*)w.bidx.p, (int)b, w.Z.p);
  }
  const dim3 grid((unsigned)ceil_div(n, 16));
  if (use32)
    hipLaunchKernelGGL(k_wb_nz<float>, grid, dim3(256), 0, s, (const float*)P.W32.p, n, kept, (const double*)w.Z.p, X, R,
                       (const double*)w.invb.p, out);
  else
    hipLaunchKernelGGL(k_wb_nz<double>, grid, dim3(256), 0, s, (const double*)P.W64.p, n, kept, (const double*)w.Z.p, X, R,
                       (const double*)w.invb.p, out);
  KRR_LAUNCH_CHECK();
}

}  // namespace krr
