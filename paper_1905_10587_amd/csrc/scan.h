// One pass over a call's inputs: the check that they are finite, and the box and mean of its points.
#pragma once

#include <utility>
#include <vector>

#include "krr_internal.h"

namespace krr {

struct ScanInput {
  const double* p;    // rows x d [dev]
  int64_t rows;
  int d;
  const char* name;
};

// Box and mean of a point set, per coordinate (host), and the mean on the device (padded with zeros).
struct PointScan {
  std::vector<double> lo, hi, mean;
  DevBuf<double> center;
};

// Pinned words that kernels on the stream write and the host reads, from a pool (any thread, any device): as many sets as
// have ever been in use at once.  Given back at the end; where kernels may still write to them (an exception between
// busy() and done()), only after the stream has been waited for.
class HostWords {
 public:
  static constexpr int kCount = 4 + 3 * KRR_MAX_D;   // doubles
  HostWords() = default;
  explicit HostWords(hipStream_t s);
  HostWords(HostWords&& o) noexcept : w_(o.w_), s_(o.s_), busy_(o.busy_) { o.w_ = nullptr; }
  HostWords& operator=(HostWords&& o) noexcept {
    std::swap(w_, o.w_);
    std::swap(s_, o.s_);
    std::swap(busy_, o.busy_);
    return *this;
  }
  ~HostWords();
  double* get() const { return w_; }
  void busy() { busy_ = true; }
  void done() { busy_ = false; }

 private:
  double* w_ = nullptr;
  hipStream_t s_ = nullptr;
  bool busy_ = false;
};

// Scans up to 4 inputs; scan_wait (after the stream has been synchronised) throws KRR_EINVAL naming the first input with
// a NaN or an Inf.  stats >= 0: also fills ps for inputs[stats], its center with dpad values (dpad 0: no device copy).
struct ScanTicket {
  ScanInput in[4];
  int count = 0, stats = -1;
  PointScan* ps = nullptr;
  HostWords host;
  DevBuf<int> flags;   // on the device, one per block of the scan: not finite (where asked for)
};
ScanTicket scan_launch(const ScanInput* in, int count, int stats, PointScan* ps, int dpad, bool flags, hipStream_t s);
void scan_wait(ScanTicket& t);

// Both with the synchronisation between them.
void scan_inputs(const ScanInput* in, int count, int stats, PointScan* ps, int dpad, hipStream_t s);

}  // namespace krr
