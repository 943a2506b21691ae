// C ABI: krr_kernel_mv (the paper's FIG(targets, sources, h, V), Sec. 2.4, computed exactly).
#include "kmv.h"

namespace krr {

void validate_common(int64_t m, int64_t n, int32_t d, double eps) {
  KRR_REQUIRE(m >= 1 && n >= 1, "point counts must be >= 1");
  KRR_REQUIRE(d >= 1 && d <= KRR_MAX_D, "d must be in [1, KRR_MAX_D]");
  KRR_REQUIRE(eps > 0 && std::isfinite(eps), "eps must be positive and finite");
}

void validate_prec(int32_t prec) {
  KRR_REQUIRE(prec == KRR_FP64 || prec == KRR_FP32 || prec == KRR_MIXED, "unknown precision");
}

// Few FP64 pairs go straight from the caller's arrays.  Not where the result overlaps an input: staging copies first, and
// so allows that.
static bool kmv_takes_small(const double* Xt, int64_t m, const double* Xs, int64_t n, int d, const double* V, int R,
                            int deriv, int prec, const double* U, int64_t ldu) {
  if (!kmv_prefers_small(m, n, d, R, deriv, prec)) return false;
  const double* end = U + (m - 1) * ldu + (deriv == 2 ? 2 : 1) * R;
  auto apart = [&](const double* p, int64_t count) { return end <= p || p + count <= U; };
  return apart(Xt, m * d) && apart(Xs, n * d) && apart(V, n * R);
}

// Full MVM from raw FP64 inputs.  scan: the sources' scan (nullptr: made here).  Both point sets (shared
// centre) and the vectors are staged, unless the product is a small one.
void kernel_mv_raw(const double* Xt, int64_t m, const double* Xs, int64_t n, int d, double eps, const double* V,
                   int R, const double* shift, int deriv, int prec, double* U, int64_t ldu, hipStream_t s,
                   const PointScan* scan) {
  const bool same = (Xt == Xs) && (m == n);
  if (kmv_takes_small(Xt, m, Xs, n, d, V, R, deriv, prec, U, ldu)) {
    kmv_small(Xt, m, Xs, n, d, eps, V, R, shift, deriv, U, ldu, nullptr, 0, s);
    return;
  }
  PointScan own;
  if (!scan) {
    const ScanInput in{Xs, n, d, "Xs"};
    scan_inputs(&in, 1, 0, &own, padded_dim(d), s);
    scan = &own;
  }
  Staged S, T;
  // square one-column mixed products may be staged in spatial order for exact far-tile culling
  const bool sort = same && prec == KRR_MIXED && R == 1 && deriv == 0 && cull_wanted(*scan, n, d, eps);
  const bool block = kmv_uses_block(prec, d, R, deriv);
  const int parts = block ? kStageSplit : kStageDirect;
  StageBatch batch;
  stage_points(S, Xs, n, d, eps, prec, scan, same, true, s, sort, parts, &batch);
  if (!same) stage_points(T, Xt, m, d, eps, prec, scan, true, false, s, false, parts, &batch);
  StagedVec SV;
  stage_vectors(SV, V, n, S.npad, R, prec, s, block, S.perm.p, nullptr, 0, &batch);
  batch.launch(s);
  kmv_launch(same ? S : T, S, SV, deriv, shift, V, prec, U, ldu, s);
}

}  // namespace krr

extern "C" int krr_kernel_mv(const double* Xt, int64_t m, const double* Xs, int64_t n, int32_t d, double eps,
                             const double* V, int32_t R, const double* shift, int32_t deriv, int32_t prec,
                             double* U, void* stream) {
  return krr::guarded([&] {
    krr::validate_common(m, n, d, eps);
    krr::validate_prec(prec);
    KRR_REQUIRE(Xt && Xs && V && U, "null pointer argument");
    KRR_REQUIRE(R >= 1 && R <= 256, "R must be in [1, 256]");
    KRR_REQUIRE(deriv >= 0 && deriv <= 2, "deriv must be 0, 1 or 2");
    KRR_REQUIRE(shift == nullptr || m == n, "shift requires targets == sources");
    if (shift)
      for (int c = 0; c < R; ++c) KRR_REQUIRE(std::isfinite(shift[c]), "shift must be finite");
    hipStream_t s = (hipStream_t)stream;
    const bool same = Xt == Xs && m == n;
    const int64_t ldu = deriv == 2 ? 2 * (int64_t)R : R;
    krr::ScanInput in[3] = {{Xt, m, d, "Xt"}, {Xs, n, d, "Xs"}, {V, n, R, "V"}};
    if (same) in[1] = in[2];
    const int count = same ? 2 : 3;
    if (krr::kmv_takes_small(Xt, m, Xs, n, d, V, R, deriv, prec, U, ldu)) {
      // needs only the flags of the scan, on the device: one synchronisation, after the product
      krr::ScanTicket t = krr::scan_launch(in, count, -1, nullptr, 0, true, s);
      krr::kmv_small(Xt, m, Xs, n, d, eps, V, R, shift, deriv, U, ldu, t.flags.p, (int)t.flags.n, s);
      KRR_CHECK_HIP(hipStreamSynchronize(s));
      krr::scan_wait(t);
    } else {
      krr::PointScan scan;
      krr::scan_inputs(in, count, same ? 0 : 1, &scan, krr::padded_dim(d), s);
      krr::kernel_mv_raw(Xt, m, Xs, n, d, eps, V, R, shift, deriv, prec, U, ldu, s, &scan);
    }
    return (int)KRR_OK;
  });
}
