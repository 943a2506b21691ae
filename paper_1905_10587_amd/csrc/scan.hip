// Input scan (see scan.h).  Every entry point reads its inputs once to reject NaN and Inf, and the operators need the
// points' mean (the centre of the FP32 and split copies) and box (far-tile culling, the FP64 exponent's bound).  One
// kernel does all of it: blocks take chunks of the inputs, a thread one coordinate (coalesced: consecutive threads,
// consecutive values), a second, one-block kernel adds the blocks' results in order, and both write what the host reads
// to host-mapped memory.  (One block per coordinate, as before, took 125 us for the mean and 83 us for the box at n = 1e5, d = 8; and
// each check, box and copy was a synchronisation of its own: 5 in a call of 16 predictions.)
#include "scan.h"

#include <algorithm>
#include <mutex>

namespace krr {

namespace {

constexpr int kMaxBlocks = 512;   // per input
constexpr int kSegs = 4;
constexpr int kPart = 3 * KRR_MAX_D;
static_assert(HostWords::kCount >= kSegs + kPart, "the scan's results");

struct Seg {
  const double* p;
  int64_t count, chunk;
  int d, first, blocks;
};
struct ScanArgs {
  Seg seg[kSegs];
  int nseg, stats;   // stats: the input with box and mean (-1: none)
};

// lane reductions of one coordinate's threads (g = thread / d, G of them) through LDS
__device__ __forceinline__ void combine(double* sum, double* lo, double* hi, int t, int g, int G, int d, int top) {
  for (int w = top; w > 0; w >>= 1) {
    __syncthreads();
    if (g < w && g + w < G) {
      sum[t] += sum[t + w * d];
      lo[t] = fmin(lo[t], lo[t + w * d]);
      hi[t] = fmax(hi[t], hi[t + w * d]);
    }
  }
  __syncthreads();
}

// Block b of its input: values [b chunk, (b + 1) chunk).  host[input] = 1 where a value is not finite (cleared by the
// host before the launch); input a.stats (chunk a multiple of d): part[b] = sums, minima, maxima per coordinate.
__global__ __launch_bounds__(256) void k_scan(ScanArgs a, double* __restrict__ part, double* __restrict__ host,
                                              int* __restrict__ flags) {
  __shared__ double sum[256], lo[256], hi[256];
  __shared__ int any;
  int s = 0;
  while (s + 1 < a.nseg && (int)blockIdx.x >= a.seg[s + 1].first) ++s;
  const Seg& g = a.seg[s];
  const int64_t b = (int)blockIdx.x - g.first;
  const int64_t beg = b * g.chunk, end = beg + g.chunk < g.count ? beg + g.chunk : g.count;
  const int t = threadIdx.x;
  if (t == 0) any = 0;
  __syncthreads();
  int bad = 0;
  if (s == a.stats) {
    const int d = g.d, G = 256 / d, S = G * d;
    double su = 0.0, l = INFINITY, h = -INFINITY;
    if (t < S) {
#pragma unroll 4
      for (int64_t e = beg + t; e < end; e += S) {
        const double v = g.p[e];
        bad |= !isfinite(v);
        su += v;
        l = fmin(l, v);
        h = fmax(h, v);
      }
    }
    sum[t] = su;
    lo[t] = l;
    hi[t] = h;
    int top = 1;
    while (2 * top < G) top *= 2;
    combine(sum, lo, hi, t, t < S ? t / d : 256, G, d, G > 1 ? top : 0);
    if (t < d) {
      double* o = part + b * kPart;
      o[t] = sum[t];
      o[KRR_MAX_D + t] = lo[t];
      o[2 * KRR_MAX_D + t] = hi[t];
    }
  } else {
#pragma unroll 4
    for (int64_t e = beg + t; e < end; e += 256) bad |= !isfinite(g.p[e]);
  }
  if (bad) any = 1;   // (the same value from every thread)
  __syncthreads();
  if (t == 0 && any) host[s] = 1.0;
  if (t == 0 && flags) flags[blockIdx.x] = any;
}

// host + kSegs = [lo | hi | mean] (KRR_MAX_D each) of input a.stats
__global__ __launch_bounds__(256) void k_scan_final(ScanArgs a, const double* __restrict__ part, double* __restrict__ center,
                                                    int dpad, double* __restrict__ host) {
  __shared__ double sum[256], lo[256], hi[256];
  const Seg& sg = a.seg[a.stats];
  const int t = threadIdx.x, d = sg.d, G = 256 / d, g = t / d;
  double su = 0.0, l = INFINITY, h = -INFINITY;
  if (g < G) {
#pragma unroll 4
    for (int b = g; b < sg.blocks; b += G) {
      const double* o = part + (int64_t)b * kPart + t % d;
      su += o[0];
      l = fmin(l, o[KRR_MAX_D]);
      h = fmax(h, o[2 * KRR_MAX_D]);
    }
  }
  sum[t] = su;
  lo[t] = l;
  hi[t] = h;
  int top = 1;
  while (2 * top < G) top *= 2;
  combine(sum, lo, hi, t, g < G ? g : 256, G, d, G > 1 ? top : 0);
  if (t < d) {
    const double mean = sum[t] / (double)(sg.count / d);
    host[kSegs + t] = lo[t];
    host[kSegs + KRR_MAX_D + t] = hi[t];
    host[kSegs + 2 * KRR_MAX_D + t] = mean;
    if (center) center[t] = mean;
  } else if (center && t < dpad) {
    center[t] = 0.0;
  }
}

struct WordPool {
  std::mutex mu;
  std::vector<double*> free;
};
WordPool& word_pool() {
  static WordPool* p = new WordPool;   // (never destroyed: a scan may end during exit)
  return *p;
}

}  // namespace

HostWords::HostWords(hipStream_t s) : s_(s) {
  WordPool& p = word_pool();
  {
    std::lock_guard<std::mutex> l(p.mu);
    if (!p.free.empty()) {
      w_ = p.free.back();
      p.free.pop_back();
      return;
    }
  }
  KRR_CHECK_HIP(hipHostMalloc((void**)&w_, sizeof(double) * kCount, hipHostMallocPortable));
}

HostWords::~HostWords() {
  if (!w_) return;
  if (busy_) (void)hipStreamSynchronize(s_);
  try {
    WordPool& p = word_pool();
    std::lock_guard<std::mutex> l(p.mu);
    p.free.push_back(w_);
  } catch (...) {   // (no memory for the list)
    (void)hipHostFree(w_);
  }
}

ScanTicket scan_launch(const ScanInput* in, int count, int stats, PointScan* ps, int dpad, bool flags, hipStream_t s) {
  KRR_REQUIRE(count >= 1 && count <= kSegs && stats < count && dpad <= 256, "internal: bad scan");
  ScanTicket tk;
  tk.count = count;
  tk.stats = stats;
  tk.ps = ps;
  tk.host = HostWords(s);
  double* host = tk.host.get();
  ScanArgs a{};
  a.nseg = count;
  a.stats = stats;
  int blocks = 0;
  for (int i = 0; i < kSegs; ++i) host[i] = 0.0;
  for (int i = 0; i < count; ++i) {
    tk.in[i] = in[i];
    Seg& g = a.seg[i];
    g.p = in[i].p;
    g.d = in[i].d;
    g.count = in[i].rows * (int64_t)in[i].d;
    const int64_t b = std::min<int64_t>(kMaxBlocks, std::max<int64_t>(1, ceil_div(g.count, 2048)));
    g.chunk = ceil_div(in[i].rows, b) * in[i].d;   // whole rows
    g.blocks = (int)ceil_div(g.count, g.chunk);
    g.first = blocks;
    blocks += g.blocks;
  }
  DevBuf<double> part(stats >= 0 ? (size_t)a.seg[stats].blocks * kPart : 0, s);
  if (flags) tk.flags.alloc(blocks, s);
  if (stats >= 0 && dpad > 0) ps->center.alloc(dpad, s);
  tk.host.busy();
  hipLaunchKernelGGL(k_scan, dim3((unsigned)blocks), dim3(256), 0, s, a, part.p, host,
                     tk.flags.p);
  if (stats >= 0)
    hipLaunchKernelGGL(k_scan_final, dim3(1), dim3(256), 0, s, a, (const double*)part.p, ps->center.p, dpad, host);
  KRR_LAUNCH_CHECK();
  return tk;
}

void scan_wait(ScanTicket& t) {
  t.host.done();
  for (int i = 0; i < t.count; ++i)
    if (t.host.get()[i] != 0.0) throw Error{KRR_EINVAL, std::string(t.in[i].name) + " contains NaN or Inf"};
  if (t.stats < 0) return;
  const int d = t.in[t.stats].d;
  const double* h = t.host.get() + kSegs;
  t.ps->lo.assign(h, h + d);
  t.ps->hi.assign(h + KRR_MAX_D, h + KRR_MAX_D + d);
  t.ps->mean.assign(h + 2 * KRR_MAX_D, h + 2 * KRR_MAX_D + d);
}

void scan_inputs(const ScanInput* in, int count, int stats, PointScan* ps, int dpad, hipStream_t s) {
  ScanTicket t = scan_launch(in, count, stats, ps, dpad, false, s);
  KRR_CHECK_HIP(hipStreamSynchronize(s));
  scan_wait(t);
}

void check_finite_device(const double* p, int64_t count, const char* what, hipStream_t s) {
  if (count <= 0) return;
  const ScanInput in{p, count, 1, what};
  scan_inputs(&in, 1, -1, nullptr, 0, s);
}

}  // namespace krr
