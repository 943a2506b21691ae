// One pass over a call's inputs: the check that they are finite, and the box and mean of its points.
#pragma once

#include <memory>
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

// Scans up to 4 inputs; scan_wait (after the stream has been synchronised) throws KRR_EINVAL naming the first input with
// a NaN or an Inf.  stats >= 0: also fills ps for inputs[stats], its center with dpad values (dpad 0: no device copy).
struct ReturnWords {
  void operator()(double* p) const;
};
struct ScanTicket {
  ScanInput in[4];
  int count = 0, stats = -1;
  PointScan* ps = nullptr;
  std::unique_ptr<double, ReturnWords> host;   // pinned result words, given back with the ticket
  DevBuf<int> flags;   // on the device, one per block of the scan: not finite (where asked for)
};
ScanTicket scan_launch(const ScanInput* in, int count, int stats, PointScan* ps, int dpad, bool flags, hipStream_t s);
void scan_wait(const ScanTicket& t);

// Both with the synchronisation between them.
void scan_inputs(const ScanInput* in, int count, int stats, PointScan* ps, int dpad, hipStream_t s);

}  // namespace krr
