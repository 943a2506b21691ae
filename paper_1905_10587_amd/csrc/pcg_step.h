// The scalar steps of the conjugate gradient recurrence inside its reduction kernels, and the halt gate of its captured
// cycles.
#pragma once

#include "krr_internal.h"

namespace krr {

// Halt gate of the graph-captured cycles.  *halt is 0, or u + 1 once the status of the cycle's iteration u
// has asked the host for a decision (a convergence claim or a breakdown); a gated kernel of stage `stage`
// does nothing when a status of an earlier stage has halted the cycle (kernels of iteration u up to its
// status have stage u + 1, the direction update after it u + 2).  halt == nullptr: never closed.
struct Gate {
  const int* halt = nullptr;
  int stage = 0;
  __device__ bool closed() const {
    if (!halt) return false;
    const int h = __hip_atomic_load(halt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return h != 0 && h < stage;
  }
};

// Scalar work done by the final reduction kernel on the column's sum v (saves a launch per scalar step):
//   kGamma:  gamma_c = rho_c / v for active columns (0 otherwise), breakdown flag if v <= 0 or not finite;
//   kBeta:   beta_c = v / rho_c for active columns (0 otherwise; v is the new r^T z);
//   kStatus: the status of iteration it for the host, stored into host-mapped memory,
//            hs = [rr = v (R) | gamma (R) | beta of the previous iteration (R) | claim (R) | flags (2)],
//            claim_c = 1 when column c is active, it >= next_check_c and sqrt(v) / ||y_c|| <= tol (its
//            recursive residual claims convergence); a claim or the breakdown flag closes the halt gate
//            (when there is one) at this kernel's stage;
//   kCheck:  the squared true residual norms of a check, also stored into hs (R).
// it = *it_base + it_off (it_base may be null: it = it_off).
struct DotEpilogue {
  enum Mode { kNone = 0, kGamma = 1, kBeta = 2, kStatus = 3, kCheck = 4 };
  int mode = kNone;
  const double* rho = nullptr;
  const int* active = nullptr;
  double* gamma = nullptr;
  double* beta = nullptr;
  int* flags = nullptr;
  double* hs = nullptr;
  const int* next_check = nullptr;
  const double* ynorm = nullptr;
  double tol = 0.0;
  const int* it_base = nullptr;
  int it_off = 0;
  int* halt = nullptr;
};

// The epilogue of column c's sum v (thread-level; out[c] = v first).  Returns gamma_c (kGamma) or beta_c
// (kBeta), 0 otherwise.
__device__ __forceinline__ double dot_epilogue(const DotEpilogue& e, const Gate& gate, int c, int R, double v,
                                               double* __restrict__ out) {
  out[c] = v;
  if (e.mode == DotEpilogue::kGamma) {
    double g = 0.0;
    if (e.active[c]) {
      if (!(v > 0.0) || !isfinite(v)) atomicOr(e.flags, 1);
      else g = e.rho[c] / v;
    }
    e.gamma[c] = g;
    return g;
  } else if (e.mode == DotEpilogue::kBeta) {
    double b = 0.0;
    if (e.active[c]) b = e.rho[c] != 0.0 ? v / e.rho[c] : 0.0;
    e.beta[c] = b;
    return b;
  } else if (e.mode == DotEpilogue::kStatus) {
    const int it = (e.it_base ? *e.it_base : 0) + e.it_off;
    const bool claim = e.active[c] && it >= e.next_check[c] && sqrt(v) / e.ynorm[c] <= e.tol;
    e.hs[c] = v;
    e.hs[R + c] = e.gamma[c];
    e.hs[2 * R + c] = e.beta[c];
    e.hs[3 * R + c] = claim ? 1.0 : 0.0;
    const int broke = c == 0 ? __hip_atomic_load(e.flags + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    if (c == 0) {
      e.hs[4 * R] = (double)e.flags[0];
      e.hs[4 * R + 1] = (double)broke;
    }
    if (e.halt && (claim || broke)) __hip_atomic_store(e.halt, gate.stage, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (e.mode == DotEpilogue::kCheck) {
    e.hs[c] = v;
  }
  return 0.0;
}

}  // namespace krr
