// The vector work of an iteration of one preconditioned column, in launches that share their passes (pcg_fused.hip).
#pragma once

#include "kmv.h"
#include "pcg_step.h"
#include "precond.h"

namespace krr {

// One column of at most this many rows: there an iteration is bound by its launches rather than by the passes over W.
constexpr int64_t kFusedRows = 32768;

struct FusedIteration {
  DevBuf<double> pq_part;   // p^T q per kDotRows rows, written by the product's last kernel
  void init(const krr_precond& P, int b, bool use32, int64_t n, hipStream_t s);
  // gamma = rho / p^T q (eg), x += gamma p, r -= gamma q, r^T r and the status (es); next: also W^T r.
  void step(double* x, double* r, const double* p, const double* q, double* pq, double* rr, const DotEpilogue& eg,
            const DotEpilogue& es, bool next, Gate gate, hipStream_t s);
  // z = M^{-1} r, rho_new = r^T z and beta (eb), pout = z + beta pin, also staged into V.  after_step: W^T r is there.
  void direction(const double* r, double* z, const double* pin, double* pout, double* rho_new, const DotEpilogue& eb,
                 bool after_step, StagedVec& V, const int64_t* perm, Gate gate, hipStream_t s);

 private:
  const krr_precond* P_ = nullptr;
  int b_ = 0;
  bool use32_ = false, few_ = false;
  int64_t n_ = 0;
  int rows_ = 0, nb_ = 0, wz_ = 0, shares_ = 1;   // rows and blocks of the pass W^T r, blocks of the pass W z,
                                                     // shares that z is left in
  DevBuf<double> rr_part_, rho_part_, partial_, t_, z_;
  void step_wt(double* x, double* r, const double* p, const double* q, double* pq, const DotEpilogue& eg, bool step,
               bool wt, Gate gate, hipStream_t s);
  void reduce(double* rr, const DotEpilogue& es, bool status, bool wt, Gate gate, hipStream_t s);
};

}  // namespace krr
