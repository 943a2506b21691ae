// Symmetric positive semidefinite eigendecomposition of the anchor block K_SS by one-sided block Jacobi, in two forms:
//
//   on the Cholesky factor (FP64 handles): K = L L^T and L R = U diag(sigma) with R orthogonal give
//     K = U diag(sigma^2) U^T, so the eigenvectors are the rotated columns themselves, normalised, and the rotations
//     are never accumulated (half the memory traffic); the factor is also much closer to orthogonal columns than K is
//     (random anchors, k = 150 .. 1600: 10 to 13 sweeps against 15 to 19);
//   on K itself, K R = U diag(lambda) with R = U accumulated (handles with an FP32 copy of the factor).  The FP32
//     rounding of W turns the last bits of the eigenvectors into differences of up to 1e-9 in an applied vector, so
//     these handles keep this form, whose sums and products are taken in a fixed order that no launch choice changes.
#include <cstring>

#include "dense.h"

namespace krr {

typedef double f64x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kW = 8;          // columns per block
constexpr int kC2 = 2 * kW;    // columns of a block pair

__device__ __forceinline__ void wave_lds_fence() {   // LDS written by this wave's lanes is read by its other lanes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1 / x and 1 / sqrt(x) to a unit or two in the last place (hardware estimate, two Newton steps), x normal
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
  return __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = __builtin_fma(0.5 * y, __builtin_fma(-x * y, y, 1.0), y);
  return __builtin_fma(0.5 * y, __builtin_fma(-x * y, y, 1.0), y);
}

struct Rotation {
  double c, s, t;   // t = 0: none
};

// The rotation that orthogonalises two columns of squared norms a, b and inner product g (none at a cosine of 1e-15
// or below).  IEEE: t, c and s by correctly rounded operations (the form on K, see above); otherwise the same root
// without the division by g and with the short reciprocals (a rotation step is a serial chain of these: k = 150,
// 13.9 -> 8.4 us a round), c then corrected.  |W W^T - K| over anchors alone, 1000 points, d = 4: 1.6e-14 (c as the
// reciprocal root leaves it: 2.8e-13; IEEE operations, which round 1 + t^2, its root and the quotient: 3.0e-13).
constexpr double kTol2 = 1e-30;
template <bool IEEE>
__device__ __forceinline__ Rotation rotation(double a, double b, double g) {
  Rotation r{1.0, 0.0, 0.0};
  if (g * g > kTol2 * (a * b)) {
    if (IEEE) {
      const double zeta = (b - a) / (2.0 * g);
      r.t = copysign(1.0, zeta) / (fabs(zeta) + sqrt(__builtin_fma(zeta, zeta, 1.0)));
      r.c = 1.0 / sqrt(__builtin_fma(r.t, r.t, 1.0));
    } else {
      const double d = b - a, h = 2.0 * g;
      const double q = __builtin_fma(d, d, h * h);
      r.t = copysign(1.0, d) * h * rcp_nr(__builtin_fma(q, rsqrt_nr(q), fabs(d)));
      // c to half a unit: a Newton step on the error of its square against 1 + t^2 = w + dw.  t's own rounding leaves a
      // rotation a rotation, but a c one unit off scales both columns, and a column goes through thousands of steps.
      const double w = __builtin_fma(r.t, r.t, 1.0), dw = __builtin_fma(r.t, r.t, 1.0 - w);
      const double c = rsqrt_nr(w), c2 = c * c, e = __builtin_fma(c, c, -c2);
      r.c = __builtin_fma(0.5 * c, __builtin_fma(-c2, dw, __builtin_fma(-c2, w, 1.0)) - e * w, c);
    }
    r.s = r.c * r.t;
  }
  return r;
}

// (u, v) = (c x - s y, s x + c y), the rounding of each stated
__device__ __forceinline__ void turn(const Rotation& r, double x, double y, double& u, double& v) {
  u = __builtin_fma(r.c, x, -(r.s * y));
  v = __builtin_fma(r.s, x, r.c * y);
}

// Round r of the circle method over NB column blocks: pair i is (P, Q), P < Q.
__device__ __forceinline__ void block_pair(int i, int r, int NB, int& P, int& Q) {
  if (i == 0) { P = r; Q = NB - 1; }
  else { P = (r + i) % (NB - 1); Q = (r - i + NB - 1) % (NB - 1); }
  if (P > Q) { const int t = P; P = Q; Q = t; }
}
// a block past k is all zeros: its partner has nothing to rotate across, and rotates its own pairs in round 0
__device__ __forceinline__ bool idle_pair(int Q, int r, int k) { return Q * kW >= k && r != 0; }

// One round.  Storage: block b holds its 8 columns
// row by row, A[(b kp + row) 8 + column], kp rows (zero past k), so that a row of a pair is two 64-byte runs.
//
// A workgroup forms the Gram matrix G = S^T S of its pair's 16 columns S (matrix cores: a lane's element is both
// operands; rows t = g mod 16 form one sum, the 16 sums are added in a fixed tree, so the result does not depend on
// NW), one wave runs one sweep of rotations on G in LDS, accumulating J, and S J is written back.  Jh (when the
// rotations are accumulated): J of every pair of the round is stored there for k_apply_rotations.
// Pairs that meet in round 0 rotate all their column pairs (15 steps of 8), later rounds the 64 cross pairs (8 steps
// of 8); a step is one LDS round trip of that wave, without barriers: lane (a, b) holds the 2 x 2 block of G between
// the column pairs a and b and rows a, a + 8 of J.
//
// What bounds it: the rounds of a sweep are serial, and a round is latency (launch, two passes over 128 KB a
// workgroup at k = 1000, 8 rotation steps), with NB / 2 workgroups on 256 CUs; hence as many waves per workgroup as
// the rows feed (NW), all loads of a wave issued together, and those of the second pass before the rotations.  The
// write-back is the largest part (7.8 of 18.5 us at k = 1000 from one workgroup), so that gridDim.y workgroups share
// it, each forming the Gram matrix and the rotations for itself; the columns therefore go from A to another buffer
// O (with 4: 14.8 us; k = 150: 9.0 -> 8.3), past the caches at the largest sizes (14.2).
template <int NW, bool KEEP>
__global__ __launch_bounds__(64 * NW) void k_jacobi_pair(const double* __restrict__ A, double* __restrict__ O,
                                                         double* __restrict__ Jh, int k, int kp, int NB, int r,
                                                         unsigned long long* __restrict__ offmax) {
  __shared__ double red[16][256];
  __shared__ double G[kC2][kC2 + 1], J[kC2][kC2 + 1];
  __shared__ double offw[4];
  int P, Q;
  block_pair(blockIdx.x, r, NB, P, Q);
  const int tid = threadIdx.x, lane = tid & 63;
  if (idle_pair(Q, r, k)) {
    if (blockIdx.y == 0)
      for (int e = tid; e < kp * kW; e += 64 * NW) O[(int64_t)P * kp * kW + e] = A[(int64_t)P * kp * kW + e];
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int64_t op = (int64_t)P * kp * kW, oq = (int64_t)Q * kp * kW;
  const int64_t mine = (r16 < kW ? op : oq) + (r16 & (kW - 1));   // this lane's column of the pair
  // first pass: Gram sums of the row groups g = wave + NW h (rows g + 16 m, four to an MFMA), 16 loads at a time
  constexpr int GP = 16 / NW, UG = 16 / GP;
  f64x4 acc[GP];
#pragma unroll
  for (int h = 0; h < GP; ++h) acc[h] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int m0 = 0; 16 * m0 < kp; m0 += 4 * UG) {
    double x[GP][UG];
#pragma unroll
    for (int u = 0; u < UG; ++u)
#pragma unroll
      for (int h = 0; h < GP; ++h) {
        const int row = wave + NW * h + 16 * (m0 + 4 * u + kq);
        x[h][u] = row < kp ? A[mine + (int64_t)row * kW] : 0.0;
      }
#pragma unroll
    for (int u = 0; u < UG; ++u) {
      if (16 * (m0 + 4 * u) < kp) {
#pragma unroll
        for (int h = 0; h < GP; ++h) acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[h][u], x[h][u], acc[h], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int h = 0; h < GP; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave + NW * h][(4 * e + kq) * 16 + r16] = acc[h][e];
  // second pass's operands, issued under the rotations: of the 16-row tiles y, y + gridDim.y, .. of this workgroup,
  // wave w takes every NW-th; a lane's row r16 of the tile, columns kq, kq + 4 of either block
  constexpr int TP = 4;
  const int ntile = kp / 16, sp = gridDim.y;
  const int t0 = (int)blockIdx.y + sp * wave;
  auto fetch = [&](int t, double (&x)[4]) {
    const int64_t o = (int64_t)(16 * t + r16) * kW + kq;
    x[0] = A[op + o];
    x[1] = A[op + o + 4];
    x[2] = A[oq + o];
    x[3] = A[oq + o + 4];
  };
  double sa[TP][4];
#pragma unroll
  for (int u = 0; u < TP; ++u)
    if (t0 + sp * NW * u < ntile) fetch(t0 + sp * NW * u, sa[u]);
  __syncthreads();
  if (tid < 256) {
    double v[4];
#pragma unroll
    for (int w = 0; w < 4; ++w)
      v[w] = (red[4 * w][tid] + red[4 * w + 1][tid]) + (red[4 * w + 2][tid] + red[4 * w + 3][tid]);
    G[tid >> 4][tid & 15] = ((v[0] + v[1]) + v[2]) + v[3];
    J[tid >> 4][tid & 15] = (tid >> 4) == (tid & 15) ? 1.0 : 0.0;
  }
  __syncthreads();
  if (tid < 256) {   // the fresh Gram's largest relative off-diagonal entry
    const int gi = tid >> 4, gj = tid & 15;
    double off = 0.0;
    if (gi < gj) {
      const double den = sqrt(G[gi][gi] * G[gj][gj]);
      off = den > 0 ? fabs(G[gi][gj]) / den : 0.0;
    }
    for (int o = 32; o > 0; o >>= 1) {
      const double t = __shfl_xor(off, o);
      off = t > off ? t : off;
    }
    if (lane == 0) offw[wave] = off;
  }
  __syncthreads();
  if (wave == 0) {
    double m = offw[0];
    for (int w = 1; w < 4; ++w) m = offw[w] > m ? offw[w] : m;
    if (lane == 0 && blockIdx.y == 0) atomicMax(offmax, (unsigned long long)__double_as_longlong(m));
    if (m * m > kTol2) {
      const int a = lane >> 3, b = lane & 7;
      const bool full = r == 0;
      const int nround = full ? kC2 - 1 : kW;
      auto pair = [&](int slot, int ir, int& p, int& q) {
        if (!full) { p = slot; q = kW + ((slot + ir) & (kW - 1)); return; }
        if (slot == 0) { p = ir; q = kC2 - 1; }
        else {
          p = ir + slot; p = p >= kC2 - 1 ? p - (kC2 - 1) : p;
          q = ir - slot; q = q < 0 ? q + (kC2 - 1) : q;
        }
        if (p > q) { const int t = p; p = q; q = t; }
      };
#pragma unroll 1
      for (int ir = 0; ir < nround; ++ir) {
        int pa, qa, pb, qb;
        pair(a, ir, pa, qa);
        pair(b, ir, pb, qb);
        const double ba = G[pb][pb], bb = G[qb][qb], bg = G[pb][qb];
        double x = G[pa][pb], y = G[pa][qb], z = G[qa][pb], w = G[qa][qb];
        const double j0 = J[a][pb], j1 = J[a][qb], j2 = J[a + kW][pb], j3 = J[a + kW][qb];
        const Rotation rb = rotation<KEEP>(ba, bb, bg);
        Rotation ra;   // pair a's rotation from lane (0, a)
        ra.c = __shfl(rb.c, a);
        ra.s = __shfl(rb.s, a);
        double x1, y1, z1, w1;
        turn(rb, x, y, x1, y1);   // columns: G <- G R
        turn(rb, z, w, z1, w1);
        turn(ra, x1, z1, x, z);   // rows: G <- R^T G
        turn(ra, y1, w1, y, w);
        if (a == b && rb.t != 0.0) {   // the rotated 2 x 2 block by the stable formulas
          x = __builtin_fma(-rb.t, bg, ba);
          w = __builtin_fma(rb.t, bg, bb);
          y = 0.0;
          z = 0.0;
        }
        double i0, i1, i2, i3;
        turn(rb, j0, j1, i0, i1);
        turn(rb, j2, j3, i2, i3);
        wave_lds_fence();   // every lane's reads are done
        G[pa][pb] = x;
        G[pa][qb] = y;
        G[qa][pb] = z;
        G[qa][qb] = w;
        J[a][pb] = i0;
        J[a][qb] = i1;
        J[a + kW][pb] = i2;
        J[a + kW][qb] = i3;
        wave_lds_fence();
      }
    }
  }
  __syncthreads();
  if (KEEP && blockIdx.y == 0 && tid < 256) Jh[((int64_t)r * (NB / 2) + blockIdx.x) * 256 + tid] = J[tid >> 4][tid & 15];
  // second pass: S <- S J
  double jb[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) jb[kc] = J[4 * kc + kq][r16];
  auto apply = [&](int t, const double (&x)[4]) {
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) d = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kc], jb[kc], d, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double* o = O + mine + (int64_t)(16 * t + 4 * e + kq) * kW;
      if (NW == 16) __hip_atomic_store(o, d[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else *o = d[e];
    }
  };
#pragma unroll
  for (int u = 0; u < TP; ++u)
    if (t0 + sp * NW * u < ntile) apply(t0 + sp * NW * u, sa[u]);
  for (int t = t0 + sp * NW * TP; t < ntile; t += sp * NW) {
    double x[4];
    fetch(t, x);
    apply(t, x);
  }
}

// V <- V J for every pair of the rounds [r0, r1) (J from k_jacobi_pair, round r's at Jh + (r - r0) NB / 2 matrices).
// The rows of V are independent, so that a workgroup takes `rows` (1 or 4) of them through all the rounds in LDS, one
// barrier a round, instead of a pass over V in every round (k = 1000: 7 us a round).  A wave takes pairs w, w + 16,
// ..: a 4 x 16 by 16 x 16 product as four v_mfma_f64_4x4x4 (operand A: lane l holds row l % 4, column 4 kc + l / 16,
// the same in its four blocks; B: J[4 kc + l / 16][l % 16]; result: row l / 16, column l % 16), the J of its next pairs
// loaded while the current ones are applied.  Four rows because every workgroup reads all of J: 252 workgroups at
// k = 1000 (with 16 rows in 63 workgroups: 3.6 us a round).  V: NB kW columns of kp rows, column-major.
__global__ __launch_bounds__(1024) void k_apply_rotations(double* __restrict__ V, const double* __restrict__ Jh, int k,
                                                          int kp, int NB, int r0, int r1, int rows) {
  extern __shared__ double vs[];   // column c at rows c
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int row0 = blockIdx.x * rows, ncol = NB * kW, np = NB / 2;
  for (int e = tid; e < rows * ncol; e += 1024) vs[e] = V[(int64_t)(e / rows) * kp + row0 + e % rows];
  const int vr = rows == 4 ? lane & 3 : 0;
  auto loadj = [&](int r, int i, double (&j)[4]) {
    const double* p = Jh + ((int64_t)(r - r0) * np + i) * 256 + r16;
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) j[kc] = p[(4 * kc + kq) * 16];
  };
  double jn[4] = {0.0, 0.0, 0.0, 0.0};
  if (wave < np) loadj(r0, wave, jn);
  __syncthreads();
  for (int r = r0; r < r1; ++r) {
    for (int i = wave; i < np; i += 16) {
      double j[4];
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) j[kc] = jn[kc];
      if (i + 16 < np) loadj(r, i + 16, jn);
      else if (r + 1 < r1) loadj(r + 1, wave, jn);
      int P, Q;
      block_pair(i, r, NB, P, Q);
      if (idle_pair(Q, r, k)) continue;
      double d = 0.0;
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) {
        const int c = (kc < 2 ? P * kW : Q * kW - kW) + 4 * kc + kq;
        d = __builtin_amdgcn_mfma_f64_4x4x4f64(vs[c * rows + vr], j[kc], d, 0, 0, 0);
      }
      const int c = (r16 < kW ? P * kW : Q * kW - kW) + r16;
      if (kq < rows) vs[c * rows + kq] = d;
    }
    __syncthreads();
  }
  for (int e = tid; e < rows * ncol; e += 1024) V[(int64_t)(e / rows) * kp + row0 + e % rows] = vs[e];
}

// Work copy for the factorisation: lower triangle of the symmetric K plus shift on the diagonal
__global__ void k_shifted(const double* __restrict__ K, int k, double shift, double* __restrict__ A) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)k * k) return;
  A[t] = K[t] + (t % k == t / k ? shift : 0.0);
}

// M (column-major) into the blocked storage of k_jacobi_pair, zero past k
__global__ void k_to_blocks(const double* __restrict__ M, int k, int kp, int NB, double* __restrict__ A) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)NB * kp * kW) return;
  const int c = (int)(t % kW), row = (int)((t / kW) % kp);
  const int64_t col = t / ((int64_t)kW * kp) * kW + c;
  A[t] = row < k && col < k ? M[col * k + row] : 0.0;
}
// identity, column-major, kp rows
__global__ void k_identity(int k, int kp, int ncol, double* __restrict__ V) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < (int64_t)ncol * kp) V[t] = t % kp == t / kp && t % kp < k ? 1.0 : 0.0;
}

// One column of the result per block.  With the rotations R (kp rows): lambda = |A column|, eigenvector = R column; without:
// lambda = |A column|^2 - shift (at least 0), eigenvector = A column normalised.  V column-major.
__global__ __launch_bounds__(256) void k_columns_to_evd(const double* __restrict__ A, const double* __restrict__ R, int k,
                                                        int kp, double shift, double* __restrict__ V,
                                                        double* __restrict__ lam) {
  __shared__ double red[256];
  const int col = blockIdx.x;
  const int64_t o = (int64_t)(col / kW) * kp * kW + col % kW;
  double s = 0.0;
  for (int t = threadIdx.x; t < k; t += 256) s = __builtin_fma(A[o + (int64_t)t * kW], A[o + (int64_t)t * kW], s);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double s2 = red[0];
  const double inv = s2 > 0.0 ? 1.0 / sqrt(s2) : 0.0;
  if (threadIdx.x == 0) lam[col] = R ? sqrt(s2) : s2 > shift ? s2 - shift : 0.0;
  for (int t = threadIdx.x; t < k; t += 256)
    V[(int64_t)col * k + t] = R ? R[(int64_t)col * kp + t] : A[o + (int64_t)t * kW] * inv;
}

template <bool KEEP>
void jacobi_round(const double* A, double* O, double* Jh, int k, int kp, int NB, int r, unsigned long long* off,
                  hipStream_t s) {
  // four workgroups a pair while that fits the CUs once
  const dim3 g((unsigned)(NB / 2), (unsigned)std::max(1, std::min(4, 256 / (NB / 2))));
  // a wave per 64 rows of a pair at most (k = 1000: 36.6 us a round with 4 waves, 16 with 16)
  if (kp <= 256) hipLaunchKernelGGL((k_jacobi_pair<4, KEEP>), g, dim3(256), 0, s, A, O, Jh, k, kp, NB, r, off);
  else if (kp <= 512) hipLaunchKernelGGL((k_jacobi_pair<8, KEEP>), g, dim3(512), 0, s, A, O, Jh, k, kp, NB, r, off);
  else hipLaunchKernelGGL((k_jacobi_pair<16, KEEP>), g, dim3(1024), 0, s, A, O, Jh, k, kp, NB, r, off);
}

}  // namespace

int jacobi_evd(const double* K, double* V, double* lam, int k, bool on_factor, hipStream_t s, int max_sweeps) {
  const unsigned nk = (unsigned)ceil_div((int64_t)k * k, 256);
  const int kp = (int)round_up(k, 16);
  int NB = (int)ceil_div(k, kW);
  NB = std::max(2, NB + (NB & 1));
  const size_t nblocked = (size_t)NB * kp * kW;
  const unsigned gb = (unsigned)ceil_div((int64_t)nblocked, 256);
  DevBuf<double> A(nblocked, s), A2(nblocked, s), R(on_factor ? 0 : nblocked, s);
  double shift = 0.0;
  if (on_factor) {
    // A numerically singular block (its smallest eigenvalues are rounding noise) is factored with a shift of a few
    // roundings of its largest possible row sum, taken off the eigenvalues again; the shift grows until the
    // factorisation succeeds.  K's roundings and its own are below k^2 u, which the fourth shift exceeds up to k = 60000
    // (the refusal after eight is for a block that is no kernel matrix).
    DevBuf<double> C((size_t)k * k, s), L((size_t)k * k, s);
    for (int attempt = 0;; ++attempt) {
      hipLaunchKernelGGL(k_shifted, dim3(nk), dim3(256), 0, s, K, k, shift, C.p);
      KRR_LAUNCH_CHECK();
      if (cholesky_lower(C.p, L.p, k, s) == 0) break;
      KRR_REQUIRE(attempt < 8, "anchor kernel block is not positive semidefinite");
      shift = shift == 0.0 ? 4.5e-16 * k : 32.0 * shift;
    }
    hipLaunchKernelGGL(k_to_blocks, dim3(gb), dim3(256), 0, s, (const double*)L.p, k, kp, NB, A.p);
  } else {
    hipLaunchKernelGGL(k_to_blocks, dim3(gb), dim3(256), 0, s, K, k, kp, NB, A.p);
    hipLaunchKernelGGL(k_identity, dim3(gb), dim3(256), 0, s, k, kp, NB * kW, R.p);
  }
  KRR_LAUNCH_CHECK();
  // the rotations of `chunk` rounds (64 MB at most) are kept, then applied to rows of R that fit in LDS
  const int64_t jround = (int64_t)(NB / 2) * 256;
  const int chunk = (int)std::min<int64_t>(NB - 1, std::max<int64_t>(1, ((int64_t)8 << 20) / jround));
  DevBuf<double> Jh(on_factor ? 0 : (size_t)(chunk * jround), s);
  const int rows = (size_t)4 * NB * kW * sizeof(double) <= 150 * 1024 ? 4 : 1;
  const size_t lds = (size_t)rows * NB * kW * sizeof(double);
  if (!on_factor) {
    KRR_REQUIRE(lds <= 160 * 1024, "k too large for the eigendecomposition");
    KRR_CHECK_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_apply_rotations),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  }
  DevBuf<unsigned long long> off(1, s);
  // A sweep's measure is the largest cosine that it met before its rotations.  The last sweep has to start at 1e-13: the
  // quadratic convergence that would allow more needs relative gaps that a block near the identity (points far apart:
  // cosines of 1e-11 and gaps no larger) does not have.
  constexpr double kStop = 1e-13;
  double *cur = A.p, *next = A2.p;
  int sweep = 0;
  for (; sweep < max_sweeps; ++sweep) {
    KRR_CHECK_HIP(hipMemsetAsync(off.p, 0, sizeof(unsigned long long), s));
    for (int r0 = 0; r0 < NB - 1; r0 += on_factor ? NB - 1 : chunk) {
      const int r1 = on_factor ? NB - 1 : std::min(r0 + chunk, NB - 1);
      for (int r = r0; r < r1; ++r) {
        if (on_factor) jacobi_round<false>(cur, next, nullptr, k, kp, NB, r, off.p, s);
        else jacobi_round<true>(cur, next, Jh.p - (int64_t)r0 * jround, k, kp, NB, r, off.p, s);
        std::swap(cur, next);
      }
      if (!on_factor)
        hipLaunchKernelGGL(k_apply_rotations, dim3((unsigned)ceil_div(kp, rows)), dim3(1024), lds, s, R.p,
                           (const double*)Jh.p, k, kp, NB, r0, r1, rows);
      KRR_LAUNCH_CHECK();
    }
    unsigned long long h = 0;
    KRR_CHECK_HIP(hipMemcpyAsync(&h, off.p, sizeof(h), hipMemcpyDeviceToHost, s));
    KRR_CHECK_HIP(hipStreamSynchronize(s));
    double offv;
    std::memcpy(&offv, &h, sizeof(offv));
    if (offv <= kStop) { ++sweep; break; }
  }
  hipLaunchKernelGGL(k_columns_to_evd, dim3((unsigned)k), dim3(256), 0, s, (const double*)cur, (const double*)R.p, k, kp,
                     shift, V, lam);
  KRR_LAUNCH_CHECK();
  return sweep;
}

}  // namespace krr
