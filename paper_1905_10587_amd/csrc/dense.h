// Small dense FP64 linear algebra for the preconditioner build (k x k with k up to a few
// thousand): kernel blocks K(A, B), a one-sided Jacobi symmetric EVD, a Cholesky factorisation and
// a lower-triangular inverse.
#pragma once

#include <algorithm>

#include "krr_internal.h"

namespace krr {

// out[a + b*ldo] = exp(-||A_a - B_b||^2 / eps)  (A: ma x d, B: nb x d, row-major); column-major out.
void kernel_block_colmajor(const double* A, int64_t ma, const double* B, int64_t nb, int d, double eps,
                           double* out, int64_t ldo, hipStream_t s);
// Row-major variant: out[a*ldo + b].
void kernel_block_rowmajor(const double* A, int64_t ma, const double* B, int64_t nb, int d, double eps,
                           double* out, int64_t ldo, hipStream_t s);
// out[a, :] = X[idx[a], :]
void gather_rows(const double* X, int64_t n, int d, const int64_t* idx, int64_t k, double* out, hipStream_t s);

// Symmetric positive semidefinite EVD by one-sided block Jacobi, on the Cholesky factor of K or on K (jacobi.hip).
// K (k x k, column-major, not modified): V holds the eigenvectors (column-major) and lam the eigenvalues (unsorted,
// non-negative).  Returns sweeps used.
int jacobi_evd(const double* K, double* V, double* lam, int k, bool on_factor, hipStream_t s, int max_sweeps = 40);

// Lower Cholesky factor of the symmetric positive definite A (k x k, column-major, lower part
// read; A is overwritten).  L receives the factor (upper part zeroed).  Returns 0 on success or
// (j+1) for the first non-positive or non-finite pivot j.
int cholesky_lower(double* A, double* L, int k, hipStream_t s);

// X = L^{-1} for lower-triangular L (column-major); X is row-major, its upper part zeroed.
void lower_inverse(const double* L, double* X, int k, hipStream_t s);

}  // namespace krr
