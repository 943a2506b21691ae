// FP32 direct-difference kernel instantiations.
#include "kmv_dispatch.h"
#include "kmv_kernels.h"

namespace krr {

template <int D, int TM, int RC, int DV>
static void go32(const KmvGrid& g, const float* xt, const float* xs, const float* v,
                 double* part, hipStream_t s) {
  auto go = [&](auto dr) {
    constexpr int DR = decltype(dr)::value;
    if (g.occ) {
      KRR_CHECK_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(g.occ, k_kmv_f32<D, TM, RC, DV, DR>, 256, 0));
      return;
    }
    hipLaunchKernelGGL((k_kmv_f32<D, TM, RC, DV, DR>), g.grid, dim3(256), 0, s, xt, xs, v, g.Rp, g.src_len, g.n_src,
                       part, g.mpad, g.Rout);
  };
  // Chunks of eight columns keep the staged width of up to eight coordinates: a call of 4000, 20011 and 60000 points with 5
  // to 8 columns takes 60, 264 and 1880 us over six coordinates and 67, 277 and 1906 over the real five, and 62, 284 and
  // 2186 over eight against 62, 292 and 2297 over seven.  One coordinate of two is the other way by 1, 3 and 5%.
  if constexpr (TM == 1 && (RC < 8 || D > 8)) with_coordinates<D>(g.d, go);
  else go(std::integral_constant<int, D>{});
}

#define KRR_DV(D, TM, RC)                                   \
  if (DV == 0) { go32<D, TM, RC, 0>(g, xt, xs, v, part, s); return true; } \
  if (DV == 2) { go32<D, TM, RC, 2>(g, xt, xs, v, part, s); return true; }
#define KRR_RC(D, TM) \
  if (RC == 1) { KRR_DV(D, TM, 1) } if (RC == 4) { KRR_DV(D, TM, 4) } if (RC == 8) { KRR_DV(D, TM, 8) }
#define KRR_TM3(D) \
  if (TM == 1) { KRR_RC(D, 1) } if (TM == 2) { KRR_RC(D, 2) } if (TM == 4) { KRR_RC(D, 4) }
#define KRR_TM1(D) \
  if (TM == 1) { KRR_RC(D, 1) }

bool launch_kmv_f32(int D, int TM, int RC, int DV, const KmvGrid& g, const float* xt, const float* xs,
                    const float* v, double* part, hipStream_t s) {
  switch (D) {
    case 2: KRR_TM3(2) break;
    case 3: KRR_TM3(3) break;
    case 4: KRR_TM3(4) break;
    case 6: KRR_TM3(6) break;
    case 8: KRR_TM3(8) break;
    case 16: KRR_TM3(16) break;
    case 32: KRR_TM1(32) break;
    case 64: KRR_TM1(64) break;
    case 128: KRR_TM1(128) break;
  }
  return false;
}

}  // namespace krr
