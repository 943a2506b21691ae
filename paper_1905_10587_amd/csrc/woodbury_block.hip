// The preconditioner's apply to 2 .. 256 columns at once: out = (X - W Z) diag(1 / beta), Z_r = G_{beta_r} (W^T X)_r.
//
// Both passes over W are bound by reading it (29 MB at 12000 x 600 in FP32), and by latency where it is smaller: so a wave
// loads four neighbouring values of W a lane and feeds them to FP64 matrix instructions of 16 columns as they lie, without
// LDS (four such tiles to a wave where there are more columns), and the rows (W^T X, G T) or the columns (W Z) are split
// until every compute unit has blocks.  General tiles of 128 x 16 through LDS left most of the chip idle here: 3500 rows,
// 350 columns, four right-hand sides: W^T X 70 us, now 5, W Z 57 us, now 5; 12000 rows, 600 columns, sixteen: 86 and 105
// us, now 11 and 11.  At 100000 rows, 1000 columns, an apply to 16 columns takes 272 us (general tiles: 1178), to 64 769
// us (1562), to 128 1564 us (2138), to 256 2710 us (3521).
#include "precond.h"

namespace krr {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kC = 16;   // columns of a tile; T and Z have rp, a multiple of it

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
// its row m.  NT column tiles share the loads of W.  rows is a multiple of 16.
template <typename TW, int NT>
__global__ __launch_bounds__(256) void k_wb_tn(const TW* __restrict__ W, int64_t n, int kept, int kp,
                                               const double* __restrict__ X, int ldx, int R, int rp, int64_t rows,
                                               double* __restrict__ part) {
  __shared__ double red[4][16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, m = lane & 15, k = lane >> 4;
  const int c0 = blockIdx.x * 64, c = c0 + 4 * m;
  const int64_t r0 = (int64_t)blockIdx.y * rows, r1 = r0 + rows < n ? r0 + rows : n;
  const int x0 = blockIdx.z * NT * kC;
  int xc[NT];
  f64x4 acc[NT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    xc[t] = x0 + t * kC + m < R ? x0 + t * kC + m : 0;   // (columns past R are not used)
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[t][s] = f64x4{0.0, 0.0, 0.0, 0.0};
  }
  // whole sixteens with three more rows behind them, then the rest
  const int64_t whole = r1 + 3 <= n ? r1 : r0 + (r1 - r0 > 3 ? (r1 - r0 - 3) / 16 * 16 : 0);
#pragma unroll (NT == 1 ? 4 : 2)
  for (int64_t j = r0; j < whole; j += 16) {
    const int64_t i = j + 4 * w + k;
    double a[4];
    load4<true>(W + i * kept, c, kept, a);
    double x[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) x[t] = X[i * ldx + xc[t]];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[t][s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], x[t], acc[t][s], 0, 0, 0);
  }
  for (int64_t j = whole; j < r1; j += 16) {
    const int64_t i = j + 4 * w + k;
    const bool in = i < r1;
    double a[4];
    load4<false>(W + (in ? i : r0) * kept, c, kept, a);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const double x = in ? X[i * ldx + xc[t]] : 0.0;
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[t][s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], x, acc[t][s], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (x0 + t * kC >= rp) break;
    if (t) __syncthreads();
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[w][4 * s + e][lane] = acc[t][s][e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int u = 4 * w + e;   // s = w: column 4 (4 e + k) + w
      const double v = ((red[0][u][lane] + red[1][u][lane]) + red[2][u][lane]) + red[3][u][lane];
      part[((int64_t)blockIdx.y * kp + c0 + 4 * (4 * e + k) + w) * rp + x0 + t * kC + m] = v;
    }
  }
}

// out[c, r] = sum over the S splits; zeros in rows from kept on.  With bidx: only the columns r whose beta is b (and those
// past R, which hold no use).
__global__ __launch_bounds__(256) void k_wb_sum(const double* __restrict__ part, int S, int kept, int kp, int rp,
                                                const int* __restrict__ bidx, int R, int b, double* __restrict__ out) {
  __shared__ double sum[3][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t idx = (int64_t)blockIdx.x * 64 + lane;   // kp * rp of them: whole blocks
  double v = 0.0;
#pragma unroll 8
  for (int s = w; s < S; s += 4) v += part[(int64_t)s * kp * rp + idx];
  if (w) sum[w - 1][lane] = v;
  __syncthreads();
  if (w) return;
  const int c = (int)(idx / rp), r = (int)(idx % rp);
  if (bidx && r < R && bidx[r] != b) return;
  out[idx] = c < kept ? ((v + sum[0][lane]) + sum[1][lane]) + sum[2][lane] : 0.0;
}

// out[i, r] = (X[i, r] - sum_c W[i, c] Z[c, r]) invb[r], 16 RT rows and NT column tiles to a block, every fourth 16 columns
// of W to a wave.  Lane l: row l % 16, columns 4 (l / 16) .. + 3 of the 16; instruction s takes column 4 k + s as its k-th.
// (X may be out.)
template <typename TW, int NT, int RT>
__global__ __launch_bounds__(256) void k_wb_nz(const TW* __restrict__ W, int64_t n, int kept,
                                               const double* __restrict__ Z, int rp, const double* X, int R,
                                               const double* __restrict__ invb, double* out) {
  __shared__ double red[4][4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, m = lane & 15, k = lane >> 4;
  const int64_t i0 = ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * (16 * RT);   // (rows over x and z: flat_grid)
  if (i0 >= n) return;
  const int x0 = blockIdx.y * NT * kC;
  const TW* row[RT];
  f64x4 acc[RT][NT];
  int zc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) zc[t] = x0 + t * kC < rp ? x0 + t * kC + m : m;
#pragma unroll
  for (int q = 0; q < RT; ++q) {
    row[q] = W + (i0 + 16 * q + m < n ? i0 + 16 * q + m : n - 1) * kept;
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[q][t] = f64x4{0.0, 0.0, 0.0, 0.0};
  }
  auto run = [&](auto fast) {
#pragma unroll (NT == 1 ? 4 : 1)
    for (int c0 = 16 * w; c0 < kept; c0 += 64) {
      const int c = c0 + 4 * k;
      double a[RT][4];
#pragma unroll
      for (int q = 0; q < RT; ++q) load4<decltype(fast)::value>(row[q], c, kept, a[q]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const double z = Z[(int64_t)(c + s) * rp + zc[t]];
#pragma unroll
          for (int q = 0; q < RT; ++q)
            acc[q][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q][s], z, acc[q][t], 0, 0, 0);
        }
    }
  };
  if (i0 + 16 * RT + 3 <= n) run(std::true_type{});
  else run(std::false_type{});
#pragma unroll
  for (int q = 0; q < RT; ++q)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (q || t) __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e) red[w][e][lane] = acc[q][t][e];
      __syncthreads();
      const double v = ((red[0][w][lane] + red[1][w][lane]) + red[2][w][lane]) + red[3][w][lane];
      const int64_t i = i0 + 16 * q + 4 * w + k;   // element e = w
      const int r = x0 + t * kC + m;
      if (i < n && r < R) out[i * R + r] = (X[i * R + r] - v) * invb[r];
    }
}

int padded_columns(int kept) { return (int)round_up(kept, 64); }

// Row splits for about 512 blocks, of 16 rows at least (64 a block keep the partial sums below a fourth of W).
int64_t split_rows(int64_t n, int kept) {
  const int64_t S = std::max<int64_t>(1, ceil_div(512, padded_columns(kept) / 64));
  return std::max<int64_t>(64, round_up(ceil_div(n, S), 16));
}

}  // namespace

int column_tiles(int R) { return R <= 16 ? 1 : R <= 32 ? 2 : 4; }

void woodbury_block_prepare(const krr_precond& P, WoodburyWork& w, hipStream_t s) {
  const int kp = padded_columns(P.kept), rp = (int)round_up(w.R, kC);
  const int64_t S = std::max(ceil_div(P.n, split_rows(P.n, P.kept)), ceil_div(P.kept, split_rows(P.kept, P.kept)));
  w.partial.alloc((size_t)(S * kp * rp), s);
  w.T.alloc((size_t)kp * rp, s);
  w.Z.alloc((size_t)kp * rp, s);
}

template <typename TW, int NT>
static void product_t(const TW* W, int64_t n, int kept, const double* V, int ldv, int cols, int rp, const int* bidx, int R,
                      int b, WoodburyWork& w, double* out, hipStream_t s) {
  const int kp = padded_columns(kept);
  const int64_t rows = split_rows(n, kept);
  const int S = (int)ceil_div(n, rows);
  hipLaunchKernelGGL((k_wb_tn<TW, NT>), dim3((unsigned)(kp / 64), (unsigned)S, (unsigned)ceil_div(rp, NT * kC)), dim3(256),
                     0, s, W, n, kept, kp, V, ldv, cols, rp, rows, w.partial.p);
  hipLaunchKernelGGL(k_wb_sum, dim3((unsigned)(kp * rp / 64)), dim3(256), 0, s, (const double*)w.partial.p, S, kept, kp, rp,
                     bidx, R, b, out);
}

template <typename TW, int NT>
static void apply_tiles(const krr_precond& P, const TW* W, const std::vector<DevBuf<double>>& G, const double* X,
                        WoodburyWork& w, double* out, hipStream_t s) {
  const int kept = P.kept, R = w.R, rp = (int)round_up(R, kC);
  const int64_t n = P.n;
  product_t<TW, NT>(W, n, kept, X, R, R, rp, nullptr, R, 0, w, w.T.p, s);
  // G is symmetric, so G T is a product of the same kind; each beta in use writes its columns
  for (size_t b = 0; b < P.betas.size(); ++b)
    if (std::find(w.bidx_host.begin(), w.bidx_host.end(), (int)b) != w.bidx_host.end())
      product_t<double, NT>(G[b].p, kept, kept, w.T.p, rp, rp, rp, w.bidx.p, R, (int)b, w, w.Z.p, s);
  const unsigned gy = (unsigned)ceil_div(rp, NT * kC);
  auto nz = [&](auto rt) {
    constexpr int RT = decltype(rt)::value;
    const dim3 rows = flat_grid(ceil_div(n, 16 * RT));
    hipLaunchKernelGGL((k_wb_nz<TW, NT, RT>), dim3(rows.x, gy, rows.y), dim3(256), 0, s, W, n, kept,
                       (const double*)w.Z.p, rp, X, R, (const double*)w.invb.p, out);
  };
  // two row tiles to a block halve its reads of Z; where that still leaves two blocks to a compute unit
  if (ceil_div(n, 32) * gy >= 512) nz(std::integral_constant<int, 2>{});
  else nz(std::integral_constant<int, 1>{});
  KRR_LAUNCH_CHECK();
}

void woodbury_block_apply(const krr_precond& P, const double* X, WoodburyWork& w, bool use32, double* out, hipStream_t s) {
  auto tiles = [&](auto nt) {
    constexpr int NT = decltype(nt)::value;
    if (use32) apply_tiles<float, NT>(P, P.W32.p, P.G32, X, w, out, s);
    else apply_tiles<double, NT>(P, P.W64.p, P.G64, X, w, out, s);
  };
  switch (column_tiles(w.R)) {
    case 1: tiles(std::integral_constant<int, 1>{}); break;
    case 2: tiles(std::integral_constant<int, 2>{}); break;
    default: tiles(std::integral_constant<int, 4>{});
  }
}

template <typename TW>
static void touch(hipStream_t s) {
  constexpr int n = 8, kp = 64, rp = kC, R = 2;
  DevBuf<TW> W(n * n, s);
  DevBuf<double> X(n * R, s), Z((size_t)kp * rp, s), out(n * R, s);
  WoodburyWork w;
  w.partial.alloc((size_t)kp * rp, s);
  for (auto [p, bytes] : {std::pair<void*, size_t>{W.p, W.bytes()}, {X.p, X.bytes()}, {Z.p, Z.bytes()}})
    KRR_CHECK_HIP(hipMemsetAsync(p, 0, bytes, s));
  product_t<TW, 1>(W.p, n, n, X.p, R, R, rp, nullptr, R, 0, w, Z.p, s);
  hipLaunchKernelGGL((k_wb_nz<TW, 1, 1>), dim3(1, 1), dim3(256), 0, s, (const TW*)W.p, (int64_t)n, n, (const double*)Z.p,
                     rp, (const double*)X.p, R, (const double*)X.p, out.p);
  KRR_LAUNCH_CHECK();
}

void woodbury_block_load(hipStream_t s) {
  touch<double>(s);
  touch<float>(s);
}

}  // namespace krr
