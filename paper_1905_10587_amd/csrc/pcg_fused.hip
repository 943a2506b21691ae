// One column's iteration in five or six launches besides the product's main kernel: the product's last kernel adds p^T q,
// the update of x and r takes the pass W^T r along, its reduction the status, the pass W z the new r^T z, and the next
// direction is written staged for the product.  What bounds an iteration of up to some 30000 points is the launches (each
// about 4.5 us with its dependency) and, inside one, latency; every block adds the few partial sums it needs itself, in
// the same order.  n = 2000, 200 columns of W in FP64: 38.5 us an
// iteration in nine launches, now 28 in six; n = 20000, 500 columns in FP32: 14 launches, now 7, 34 us less.
#include "pcg_fused.h"

namespace krr {

namespace {

// The sum over a block of 256 threads, for all of them: butterflies, then the four waves in order.
__device__ __forceinline__ double block_sum(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

__device__ __forceinline__ double parts_sum(const double* __restrict__ part, int count, double* red) {
  double v = 0.0;
  for (int i = threadIdx.x; i < count; i += 256) v += part[i];
  return block_sum(v, red);
}

// Block b: rows [b rows, (b + 1) rows), at most 256.  STEP: gamma from the partials of p^T q, the rows of x and r, and
// rr_part[b].  WT: partial[b, c] = sum_i W[i, c] r[i].
template <typename TW, bool STEP, bool WT>
__global__ __launch_bounds__(256) void k_step_wt(const TW* __restrict__ W, int64_t n, int kept, int rows,
                                                 double* __restrict__ x, double* __restrict__ r,
                                                 const double* __restrict__ p, const double* __restrict__ q,
                                                 const double* __restrict__ pq_part, int npq, double* __restrict__ pq,
                                                 double* __restrict__ rr_part, DotEpilogue eg, Gate gate,
                                                 double* __restrict__ partial) {
  if (STEP && gate.closed()) return;
  __shared__ double red[4], rs[256];
  const int t = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * rows, i = i0 + t;
  const bool mine = t < rows && i < n;
  double u = mine ? r[i] : 0.0;
  if (STEP) {
    const double pi = mine ? p[i] : 0.0, qi = mine ? q[i] : 0.0, xi = mine ? x[i] : 0.0;
    const double v = parts_sum(pq_part, npq, red);
    const double g = eg.active[0] && v > 0.0 && isfinite(v) ? eg.rho[0] / v : 0.0;   // (as the epilogue's)
    if (blockIdx.x == 0 && t == 0) dot_epilogue(eg, gate, 0, 1, v, pq);
    if (mine) {
      x[i] = __builtin_fma(g, pi, xi);
      u = __builtin_fma(-g, qi, u);
      r[i] = u;
    }
    const double s = block_sum(mine ? u * u : 0.0, red);
    if (t == 0) rr_part[blockIdx.x] = s;
  }
  if (!WT) return;
  rs[t] = u;
  __syncthreads();
  const int cnt = (int)(i0 + rows < n ? rows : n - i0);
  for (int c = t; c < kept; c += 256) {
    const TW* w = W + i0 * kept + c;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int j = 0;
#pragma unroll 4
    for (; j + 4 <= cnt; j += 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] = __builtin_fma((double)w[(int64_t)(j + k) * kept], rs[j + k], acc[k]);
    }
    for (; j < cnt; ++j) acc[0] = __builtin_fma((double)w[(int64_t)j * kept], rs[j], acc[0]);
    partial[(int64_t)blockIdx.x * kept + c] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  }
}

// Block c < cols: t[c] = sum_b partial[b, c]; one block more (with a status): r^T r and the status.
__global__ __launch_bounds__(256) void k_reduce_status(const double* __restrict__ partial, int nb, int kept, int cols,
                                                       double* __restrict__ t, const double* __restrict__ rr_part,
                                                       double* __restrict__ rr, DotEpilogue es, Gate gate) {
  __shared__ double red[4];
  const int c = blockIdx.x;
  if (c < cols) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) v += partial[(int64_t)b * kept + c];
    v = block_sum(v, red);
    if (threadIdx.x == 0) t[c] = v;
    return;
  }
  if (gate.closed()) return;
  const double v = parts_sum(rr_part, nb, red);
  if (threadIdx.x == 0) dot_epilogue(es, gate, 0, 1, v, rr);
}

// Few partials: block s adds those of its 16 columns to t and writes their share of z = G t, zpart[s, i] = sum over its
// columns of G[c, i] t[c]; the next kernel adds the shares.  (Every block adding all columns for some rows of G instead
// reads 200 KB through one compute unit: 7.4 us at n = 2000, 200 columns, now 5.)  One block more as above.
constexpr int kSliceCols = 16;
__global__ __launch_bounds__(256) void k_gemv_status(const double* __restrict__ partial, int nb, int kept,
                                                     const double* __restrict__ G, double* __restrict__ zpart, int slices,
                                                     const double* __restrict__ rr_part, double* __restrict__ rr,
                                                     DotEpilogue es, Gate gate) {
  __shared__ double ts[256], red[4];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x == slices) {
    if (gate.closed()) return;
    const double v = parts_sum(rr_part, nb, red);
    if (tid == 0) dot_epilogue(es, gate, 0, 1, v, rr);
    return;
  }
  const int c0 = blockIdx.x * kSliceCols, cl = tid % kSliceCols, cols = min(kSliceCols, kept - c0);
  double v = 0.0;
  if (cl < cols) {
#pragma unroll 8
    for (int b = tid / kSliceCols; b < nb; b += 256 / kSliceCols) v += partial[(int64_t)b * kept + c0 + cl];
  }
  ts[tid] = v;
  __syncthreads();
  if (tid < kSliceCols) {
#pragma unroll
    for (int k = 1; k < 256 / kSliceCols; ++k) v += ts[k * kSliceCols + tid];
    ts[tid] = v;   // (0 past the last column)
  }
  __syncthreads();
  for (int i = tid; i < kept; i += 256) {
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < kSliceCols; ++c) s = __builtin_fma(G[(int64_t)(c < cols ? c0 + c : c0) * kept + i], ts[c], s);
    zpart[(int64_t)blockIdx.x * kept + i] = s;
  }
}

// out[i] = (r[i] - sum_c W[i, c] z[c]) / beta, z the sum of its shares, two rows to a wave, and part[b] = sum r[i] out[i] over block b's rows.
template <typename TW>
__global__ __launch_bounds__(256) void k_wz_dot(const TW* __restrict__ W, int64_t n, int kept,
                                                const double* __restrict__ z, int shares, const double* __restrict__ r,
                                                double inv_beta, double* __restrict__ out, double* __restrict__ part) {
  extern __shared__ double zs[];
  __shared__ double red[4];
  for (int c = threadIdx.x; c < kept; c += 256) {
    double v = z[c];
#pragma unroll 8
    for (int s = 1; s < shares; ++s) v += z[(int64_t)s * kept + c];
    zs[c] = v;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  double dot = 0.0;
  for (int64_t i0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 2; i0 < n; i0 += (int64_t)gridDim.x * 8) {
    const TW* w0 = W + i0 * kept;
    const TW* w1 = W + (i0 + 1 < n ? i0 + 1 : i0) * kept;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
    for (int c = lane; c < kept; c += 64) {
      const double zc = zs[c];
      s0 = __builtin_fma((double)w0[c], zc, s0);
      s1 = __builtin_fma((double)w1[c], zc, s1);
    }
    for (int o = 32; o > 0; o >>= 1) {
      s0 += __shfl_xor(s0, o);
      s1 += __shfl_xor(s1, o);
    }
    if (lane < 2 && i0 + lane < n) {
      const double ri = r[i0 + lane], v = (ri - (lane ? s1 : s0)) * inv_beta;
      out[i0 + lane] = v;
      dot = __builtin_fma(ri, v, dot);
    }
  }
  dot = block_sum(dot, red);
  if (threadIdx.x == 0) part[blockIdx.x] = dot;
}

// beta from the partials of r^T z, and staged row i of the next direction (the caller's row perm[i]).
__global__ __launch_bounds__(256) void k_next_direction(const double* __restrict__ rho_part, int np,
                                                        const double* __restrict__ z, const double* pin, double* pout,
                                                        int64_t n, const int64_t* __restrict__ perm,
                                                        double* __restrict__ v64, float* __restrict__ v32,
                                                        double* __restrict__ rho_new, DotEpilogue eb, Gate gate) {
  if (gate.closed()) return;
  __shared__ double red[4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t o = i < n ? (perm ? perm[i] : i) : 0;
  const double zi = z[o], pi = pin[o];
  const double v = parts_sum(rho_part, np, red);
  const bool act = eb.active[0] != 0;
  const double b = act && eb.rho[0] != 0.0 ? v / eb.rho[0] : 0.0;   // (as the epilogue's)
  if (blockIdx.x == 0 && threadIdx.x == 0) dot_epilogue(eb, gate, 0, 1, v, rho_new);
  if (i >= n) return;
  const double pn = act ? __builtin_fma(b, pi, zi) : pi;
  pout[o] = pn;
  if (v64) v64[i] = pn;
  if (v32) v32[i] = (float)pn;
}

// Up to so many columns and partials z is left in shares; more would make the shares a load of their own (each block of the
// pass W z reads them: kept^2 / 2 bytes).  An iteration in FP64 with shares and without: 1000 rows, 60 and 130 columns 30.3
// and 31.7, 30.9 and 32.1 us; 2000 rows, 60, 130 and 200: 31.4 and 31.8, 32.2 and 32.5, 33.3 and 32.4; past the line, 4000
// rows, 200 and 256: 47.7 and 46.2, 48.3 and 47.0; 20000 rows, 400: 385.6 and 382.9.
constexpr int kSharedCols = 256;
constexpr int64_t kFewPartials = 32768;

}  // namespace

void FusedIteration::init(const krr_precond& P, int b, bool use32, int64_t n, hipStream_t s) {
  P_ = &P;
  b_ = b;
  use32_ = use32;
  n_ = n;
  rows_ = woodbury_rows(n);
  nb_ = (int)ceil_div(n, rows_);
  wz_ = (int)std::min<int64_t>(ceil_div(n, 8), 1024);
  pq_part.alloc(ceil_div(n, kDotRows), s);
  rr_part_.alloc(nb_, s);
  rho_part_.alloc(wz_, s);
  partial_.alloc((size_t)nb_ * P.kept, s);
  t_.alloc(P.kept, s);
  few_ = P.kept <= kSharedCols && (int64_t)nb_ * P.kept <= kFewPartials;
  shares_ = few_ ? (int)ceil_div(P.kept, kSliceCols) : 1;
  z_.alloc((size_t)shares_ * P.kept, s);
}

void FusedIteration::step_wt(double* x, double* r, const double* p, const double* q, double* pq, const DotEpilogue& eg,
                             bool step, bool wt, Gate gate, hipStream_t s) {
  const int npq = (int)pq_part.n;
  auto go = [&](auto W, auto st, auto w) {
    using TW = std::remove_cv_t<std::remove_pointer_t<decltype(W)>>;
    hipLaunchKernelGGL((k_step_wt<TW, decltype(st)::value, decltype(w)::value>), dim3((unsigned)nb_), dim3(256), 0, s,
                       (const TW*)W, n_, P_->kept, rows_, x, r, p, q, (const double*)pq_part.p, npq, pq, rr_part_.p,
                       eg, gate, partial_.p);
  };
  auto typed = [&](auto st, auto w) {
    if (use32_) go(P_->W32.p, st, w);
    else go(P_->W64.p, st, w);
  };
  if (step && wt) typed(std::true_type{}, std::true_type{});
  else if (step) typed(std::true_type{}, std::false_type{});
  else typed(std::false_type{}, std::true_type{});
  KRR_LAUNCH_CHECK();
}

void FusedIteration::reduce(double* rr, const DotEpilogue& es, bool status, bool wt, Gate gate, hipStream_t s) {
  const int kept = P_->kept;
  const double* G = use32_ ? P_->G32[b_].p : P_->G64[b_].p;
  if (wt && few_) {
    hipLaunchKernelGGL(k_gemv_status, dim3((unsigned)(shares_ + status)), dim3(256), 0, s, (const double*)partial_.p,
                       nb_, kept, G, z_.p, shares_, (const double*)rr_part_.p, rr, es, gate);
  } else {
    const int cols = wt ? kept : 0;
    hipLaunchKernelGGL(k_reduce_status, dim3((unsigned)(cols + status)), dim3(256), 0, s, (const double*)partial_.p,
                       nb_, kept, cols, t_.p, (const double*)rr_part_.p, rr, es, gate);
    if (wt) woodbury_gemv(G, kept, t_.p, z_.p, s);
  }
  KRR_LAUNCH_CHECK();
}

void FusedIteration::step(double* x, double* r, const double* p, const double* q, double* pq, double* rr,
                          const DotEpilogue& eg, const DotEpilogue& es, bool next, Gate gate, hipStream_t s) {
  step_wt(x, r, p, q, pq, eg, true, next, gate, s);
  reduce(rr, es, true, next, gate, s);
}

void FusedIteration::direction(const double* r, double* z, const double* pin, double* pout, double* rho_new,
                               const DotEpilogue& eb, bool after_step, StagedVec& V, const int64_t* perm, Gate gate,
                               hipStream_t s) {
  KRR_REQUIRE(V.R == 1 && (V.v64.p || V.v32.p), "internal: a direction is staged over an earlier one");
  if (!after_step) {
    step_wt(nullptr, const_cast<double*>(r), nullptr, nullptr, nullptr, DotEpilogue(), false, true, Gate(), s);
    reduce(nullptr, DotEpilogue(), false, true, Gate(), s);
  }
  const size_t lds = (size_t)P_->kept * sizeof(double);
  const double inv_beta = 1.0 / P_->betas[b_];
  if (use32_)
    hipLaunchKernelGGL(k_wz_dot<float>, dim3((unsigned)wz_), dim3(256), lds, s, (const float*)P_->W32.p, n_, P_->kept,
                       (const double*)z_.p, shares_, r, inv_beta, z, rho_part_.p);
  else
    hipLaunchKernelGGL(k_wz_dot<double>, dim3((unsigned)wz_), dim3(256), lds, s, (const double*)P_->W64.p, n_, P_->kept,
                       (const double*)z_.p, shares_, r, inv_beta, z, rho_part_.p);
  hipLaunchKernelGGL(k_next_direction, dim3((unsigned)ceil_div(n_, 256)), dim3(256), 0, s, (const double*)rho_part_.p,
                     wz_, (const double*)z, pin, pout, n_, perm, V.v64.p, V.v32.p, rho_new, eb, gate);
  KRR_LAUNCH_CHECK();
}

}  // namespace krr
