// Kernel blocks and row gathers of the preconditioner build (see dense.h).
#include "dense.h"
#include "kmv_kernels.h"   // exp_neg_f64

namespace krr {

// ------------------------------------------------------------------ kernel blocks, gather
__global__ void k_kernel_block(const double* __restrict__ A, int64_t ma, const double* __restrict__ B, int64_t nb,
                               int d, double inv_eps, double* __restrict__ out, int64_t ldo, int rowmajor) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= ma * nb) return;
  int64_t a, b;
  if (rowmajor) { a = idx / nb; b = idx % nb; }
  else { a = idx % ma; b = idx / ma; }
  double d2 = 0;
  for (int k = 0; k < d; ++k) {
    const double df = A[a * d + k] - B[b * d + k];
    d2 = __builtin_fma(df, df, d2);
  }
  const double v = exp_neg_f64(d2 * inv_eps);
  if (rowmajor) out[a * ldo + b] = v;
  else out[a + b * ldo] = v;
}

void kernel_block_colmajor(const double* A, int64_t ma, const double* B, int64_t nb, int d, double eps,
                           double* out, int64_t ldo, hipStream_t s) {
  const int64_t tot = ma * nb;
  hipLaunchKernelGGL(k_kernel_block, dim3((unsigned)ceil_div(tot, 256)), dim3(256), 0, s, A, ma, B, nb, d,
                     1.0 / eps, out, ldo, 0);
  KRR_LAUNCH_CHECK();
}

void kernel_block_rowmajor(const double* A, int64_t ma, const double* B, int64_t nb, int d, double eps,
                           double* out, int64_t ldo, hipStream_t s) {
  const int64_t tot = ma * nb;
  hipLaunchKernelGGL(k_kernel_block, dim3((unsigned)ceil_div(tot, 256)), dim3(256), 0, s, A, ma, B, nb, d,
                     1.0 / eps, out, ldo, 1);
  KRR_LAUNCH_CHECK();
}

__global__ void k_gather_rows(const double* __restrict__ X, int64_t n, int d, const int64_t* __restrict__ idx,
                              int64_t k, double* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= k * d) return;
  const int64_t a = t / d;
  const int c = (int)(t % d);
  int64_t r = idx[a];
  r = r < 0 ? 0 : (r >= n ? n - 1 : r);   // indices are validated on the host path; clamp keeps reads in bounds
  out[t] = X[r * d + c];
}

void gather_rows(const double* X, int64_t n, int d, const int64_t* idx, int64_t k, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)ceil_div(k * d, 256)), dim3(256), 0, s, X, n, d, idx, k, out);
  KRR_LAUNCH_CHECK();
}

}  // namespace krr
