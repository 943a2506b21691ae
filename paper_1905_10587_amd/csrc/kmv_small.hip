// FP64 products of few pairs, straight from the caller's arrays: no staged copies, no padding of the targets, and one
// launch where a block can take all sources of its targets.
#include "kmv.h"
#include "kmv_kernels.h"

namespace krr {

namespace {

// The most targets a thread holds: 32 coordinates (scalar registers) and 16 sums.
constexpr int most_targets(int D, int NC) {
  int tg = 8;
  while (tg > 1 && (tg * D > 32 || tg * NC > 16)) tg /= 2;
  return tg;
}

// Whether a scan queued before has found a value that is not finite (flags of its blocks; nbad 0: none to ask).  All
// threads of a block take part.
__device__ __forceinline__ bool refused(const int* bad, int nbad) {
  int b = 0;
  for (int i = threadIdx.x; i < nbad; i += 256) b |= bad[i];
  return __syncthreads_or(b) != 0;
}

// TG targets to G threads (G = 64, four groups a block, up to 512 sources; else 256): thread g of the group every G-th
// source from g on, for all TG targets.  The sums are added over a wave, each exchange halving the number of sums that a
// lane holds, then over the four waves in order.  grid.y splits the sources; with one split the result is written with
// its ridge term, else part[split][target][column].
// Bound by latency: a pair is 2 d + 17 FP64 operations, and 2000 x 2000 pairs are 63 a thread, one wave to a SIMD.  So a
// source is loaded once for TG targets, whose chains are independent, and nothing in the loop branches (coordinates and
// columns past d and R are loaded again from index 0): 11 us for 2000 x 2000 and 5 us for 16 x 2000 points, d = 3 (staged: 131 and 211 us a call; now 36 and 32).
template <int D, int TG, int RC, int DV>
__global__ __launch_bounds__(256) void k_kmv_small(const double* __restrict__ Xt, int64_t m, const double* __restrict__ Xs,
                                                   int64_t n, int d, double neg_c, const double* __restrict__ V, int R,
                                                   int64_t len, int G, ColumnShift sh, const int* __restrict__ bad,
                                                   int nbad, double* __restrict__ U, int64_t ldu,
                                                   double* __restrict__ part) {
  constexpr int NO = DV == 2 ? 2 : 1;
  constexpr int NC = RC * NO;    // sums per target: K columns, then K' columns
  constexpr int NV = TG * NC;    // a power of two, at most 16
  __shared__ double red[4][NV];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t i0 = G == 64 ? ((int64_t)blockIdx.x * 4 + wave) * TG : (int64_t)blockIdx.x * TG;
  const int64_t j0 = (int64_t)blockIdx.y * len, j1 = j0 + len < n ? j0 + len : n;
  double x[TG][D];
#pragma unroll
  for (int t = 0; t < TG; ++t) {
    const double* p = Xt + (i0 + t < m ? i0 + t : m - 1) * d;
#pragma unroll
    for (int k = 0; k < D; ++k) x[t][k] = p[k < d ? k : 0];
  }
  double acc[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) acc[c] = 0.0;
#pragma unroll (TG > 2 ? 2 : 4)
  for (int64_t j = j0 + (G == 64 ? lane : tid); j < j1; j += G) {
    double y[D], v[RC];
#pragma unroll
    for (int k = 0; k < D; ++k) y[k] = Xs[j * d + (k < d ? k : 0)];
#pragma unroll
    for (int c = 0; c < RC; ++c) v[c] = V[j * R + (c < R ? c : 0)];   // (columns past R are not written)
#pragma unroll
    for (int t = 0; t < TG; ++t) {
      double d2 = 0.0;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const double df = k < d ? x[t][k] - y[k] : 0.0;
        d2 = __builtin_fma(df, df, d2);
      }
      const double q = d2 * neg_c;
      const double e = exp2_neg_f64(q);
      const double ed = -kLn2 * q * e;   // (D^2/eps) K
#pragma unroll
      for (int c = 0; c < RC; ++c) {
        double* a = acc + t * NC + c;
        a[0] = __builtin_fma(DV == 1 ? ed : e, v[c], a[0]);
        if (DV == 2) a[RC] = __builtin_fma(ed, v[c], a[RC]);
      }
    }
  }
  int idx = 0;   // the sum that this lane ends up with
#pragma unroll
  for (int h = NV / 2, o = 1; h >= 1; h /= 2, o *= 2) {
    const bool up = (lane & o) != 0;
    idx += up ? h : 0;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const double keep = up ? acc[i + h] : acc[i], give = up ? acc[i] : acc[i + h];
      acc[i] = keep + __shfl_xor(give, o);
    }
  }
#pragma unroll
  for (int o = NV; o < 64; o *= 2) acc[0] += __shfl_xor(acc[0], o);
  if (lane < NV) red[wave][idx] = acc[0];
  if (refused(bad, nbad)) return;   // (its barrier also orders red)
  const int mine = G == 64 ? wave * 64 : 0;
  if (tid < mine || tid >= mine + NV) return;
  const int w = tid - mine, t = w / NC, c = w % NC, col = c % RC;
  const int64_t i = i0 + t;
  if (i >= m || col >= R) return;
  const double s = G == 64 ? red[wave][w] : ((red[0][w] + red[1][w]) + red[2][w]) + red[3][w];
  const int oc = c < RC ? col : R + col;
  if (gridDim.y > 1) part[((int64_t)blockIdx.y * m + i) * (R * NO) + oc] = s;
  else U[i * ldu + oc] = sh.on && c < RC ? __builtin_fma(sh.v[col], V[i * R + col], s) : s;
}

__global__ __launch_bounds__(256) void k_small_finish(const double* __restrict__ part, int S, int64_t m, int cols, int R,
                                                      ColumnShift sh, const double* __restrict__ V,
                                                      const int* __restrict__ bad, int nbad, double* __restrict__ U,
                                                      int64_t ldu) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (refused(bad, nbad) || t >= m * cols) return;
  const int64_t i = t / cols;
  const int c = (int)(t % cols);
  double s = 0.0;
#pragma unroll 8
  for (int p = 0; p < S; ++p) s += part[(int64_t)p * m * cols + t];
  U[i * ldu + c] = sh.on && c < R ? __builtin_fma(sh.v[c], V[i * R + c], s) : s;
}

struct SmallArgs {
  const double* Xt;
  int64_t m;
  const double* Xs;
  int64_t n;
  int d;
  double neg_c;
  const double* V;
  int R, deriv;
  ColumnShift sh;
  const int* bad;
  int nbad;
  double* U;
  int64_t ldu;
  hipStream_t s;
};

template <int D, int TG, int RC, int DV>
void go_small(const SmallArgs& a) {
  const int G = a.n <= 512 ? 64 : 256;
  const int64_t gx = ceil_div(a.m, TG * (256 / G));
  // one split up to 64 pairs a thread; more only while blocks are wanting, of 8 sources a thread at least
  const int64_t per = ceil_div(a.n, G);
  int64_t S = 1;
  if (per * TG > 64) S = std::max<int64_t>(1, std::min(ceil_div(1024, gx), per / 8));
  const int64_t len = ceil_div(a.n, S);
  S = ceil_div(a.n, len);
  kmv_record_launch(KmvLaunchInfo{-1, (int)len, 0, 0, round_up(a.m, kRowPad), 0});
  const int cols = a.R * (DV == 2 ? 2 : 1);
  DevBuf<double> part(S > 1 ? (size_t)(S * a.m * cols) : 0, a.s);
  hipLaunchKernelGGL((k_kmv_small<D, TG, RC, DV>), dim3((unsigned)gx, (unsigned)S), dim3(256), 0, a.s, a.Xt, a.m, a.Xs, a.n,
                     a.d, a.neg_c, a.V, a.R, len, G, a.sh, a.bad, a.nbad, a.U, a.ldu, part.p);
  KRR_LAUNCH_CHECK();
  if (S > 1) {
    hipLaunchKernelGGL(k_small_finish, dim3((unsigned)ceil_div(a.m * cols, 256)), dim3(256), 0, a.s, (const double*)part.p,
                       (int)S, a.m, cols, a.R, a.sh, a.V, a.bad, a.nbad, a.U, a.ldu);
    KRR_LAUNCH_CHECK();
  }
}

template <int D, int RC, int DV>
void go_small_t(const SmallArgs& a) {
  // one target a thread while that leaves blocks wanting (two for each compute unit)
  if (a.m <= 512) go_small<D, 1, RC, DV>(a);
  else go_small<D, most_targets(D, DV == 2 ? 2 * RC : RC), RC, DV>(a);
}

template <int D>
void go_small_d(const SmallArgs& a) {
  if (a.R > 4) go_small_t<D, 8, 0>(a);
  else if (a.R > 1) go_small_t<D, 4, 0>(a);
  else if (a.deriv == 1) go_small_t<D, 1, 1>(a);
  else if (a.deriv == 2) go_small_t<D, 1, 2>(a);
  else go_small_t<D, 1, 0>(a);
}

}  // namespace

bool kmv_small_fits(int64_t m, int64_t n, int d, int R, int deriv, int prec) {
  // 8 M pairs at d <= 8 and one column: there a call takes 52 us, and the staged path's four to six launches 56 (4000 x
  // 4000, d = 3).  Wide points and more columns leave fewer targets to a thread: at 2890 x 2890, d = 16 it is 163 us.
  const int64_t most = ((int64_t)1 << 23) >> ((d > 8 ? 3 : 0) + (R > 1 ? 1 : 0));
  return prec == KRR_FP64 && d <= 16 && (R == 1 || (R <= 8 && deriv == 0)) && m <= most / n;
}

bool kmv_prefers_small(int64_t m, int64_t n, int d, int R, int deriv, int prec) {
  return kmv_small_fits(m, n, d, R, deriv, prec) && kmv_get_override(d, R, prec) < 0;
}

void kmv_small(const double* Xt, int64_t m, const double* Xs, int64_t n, int d, double eps, const double* V, int R,
               const double* shift, int deriv, double* U, int64_t ldu, const int* bad, int nbad,
               hipStream_t s) {
  SmallArgs a{Xt, m, Xs, n, d, -kLog2e / eps, V, R, deriv, {}, bad, nbad, U, ldu, s};
  a.sh.on = shift != nullptr && deriv != 1;
  for (int c = 0; a.sh.on && c < R; ++c) a.sh.v[c] = shift[c];
  if (d <= 2) go_small_d<2>(a);
  else if (d <= 3) go_small_d<3>(a);
  else if (d <= 4) go_small_d<4>(a);
  else if (d <= 6) go_small_d<6>(a);
  else if (d <= 8) go_small_d<8>(a);
  else go_small_d<16>(a);
}

}  // namespace krr
