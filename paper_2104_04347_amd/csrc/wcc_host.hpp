// wcc_host.hpp -- small states and status reports between host and device
// through pinned host memory that kernels read and write directly
// (wcc_host.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "wcc_internal.hpp"

namespace wcc {

// One staging buffer: a status report, then up to kStageRows bytes of state.
constexpr size_t kStageBytes = size_t(2) << 20;
constexpr size_t kStageHead = 1024;
constexpr size_t kStageRows = kStageBytes - kStageHead;

// A staging buffer on loan from the process for one call that works on
// `stream`: taken when first needed, given back at the end of the call, so that
// a context holds none between calls.  A call that ends with work on the buffer
// still enqueued (an error half way) waits for the stream first.  The process
// keeps at most eight buffers for later calls and makes another where more
// calls are at work at once; safe from several threads.
class StageLoan {
 public:
  explicit StageLoan(hipStream_t stream) : stream_(stream) {}
  ~StageLoan();
  StageLoan(const StageLoan&) = delete;
  StageLoan& operator=(const StageLoan&) = delete;
  // The buffer, or null where no pinned memory is to be had (the caller then
  // copies directly).
  char* get();
  // Work on the buffer has been enqueued / waited for.
  void enqueued() { busy_ = true; }
  void waited() { busy_ = false; }

 private:
  hipStream_t stream_;
  char* mem_ = nullptr;
  bool busy_ = false;
};

// The control block with smax[s] replaced by the largest partial entry of
// slot s, written to the head of a staging buffer; complete once the stream
// has been synchronised.
hipError_t launch_report(const Ctrl* ctrl, const unsigned long long* parts, char* stage, hipStream_t s);

// Rows of a state: row r of a state of nc components and P + 1 rows each is
// component r / (P + 1), derivative k = r % (P + 1); point values in p[c][ld],
// derivatives in d[c][k - 1][ld].
template <class R>
struct Rows {
  double* p;
  R* d;
  int64_t ld;
  int32_t nc, P;
  int32_t n;               // cells
};

// Copy rows between the staging buffer (dense doubles [c][k][n] after its
// head) and the device.
template <class R>
hipError_t launch_rows_in(const Rows<R>& rows, const char* stage, hipStream_t s);
template <class R>
hipError_t launch_rows_out(const Rows<R>& rows, char* stage, hipStream_t s);

inline bool stage_fits(int64_t nc, int64_t P, int64_t n) { return (size_t)(nc * (P + 1) * n) * 8 <= kStageRows; }

}  // namespace wcc
