// wcc_host.hip -- small states and status reports between host and device.
//
// A state is nc (P + 1) padded rows on the device.  As one asynchronous copy a
// row from or to pageable memory it cost 5 to 18 us a row, and the control
// block and the 64 partial maxima two more copies each time the host looked:
// for a mesh of a few hundred cells more than its half-steps.  States of up to
// 2 MiB go through a pinned buffer instead, packed and unpacked by one kernel
// over the bus, and a report is one kernel of one wave.  Measured at 40 x 40
// cells, 24 rows (2D Euler, P = 2): write 168 -> 34 us, read 433 -> 52 us.  Larger
// states keep the copies, which run at the bus's rate there.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "wcc_host.hpp"
#include "wcc_tile.hpp"

namespace wcc {

namespace {
constexpr int kKept = 8;
// plain data, never destroyed: usable until the process ends
std::mutex g_stage_mu;
char* g_stages[kKept];
int g_stage_n = 0;
}  // namespace

char* StageLoan::get() {
  if (mem_) return mem_;
  {
    std::lock_guard<std::mutex> lk(g_stage_mu);
    if (g_stage_n > 0) return mem_ = g_stages[--g_stage_n];
  }
  void* s = nullptr;
  if (hipHostMalloc(&s, kStageBytes, hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return mem_ = static_cast<char*>(s);
}

StageLoan::~StageLoan() {
  if (!mem_) return;
  if (busy_) (void)hipStreamSynchronize(stream_);
  {
    std::lock_guard<std::mutex> lk(g_stage_mu);
    if (g_stage_n < kKept) {
      g_stages[g_stage_n++] = mem_;
      return;
    }
  }
  (void)hipHostFree(mem_);
}

__global__ __launch_bounds__(64) void k_report(const Ctrl* ctrl, const unsigned long long* parts, Ctrl* out) {
  const int lane = threadIdx.x;
  constexpr int words = (int)(sizeof(Ctrl) / sizeof(unsigned long long));
  static_assert(words <= 64, "one word a lane");
  // The entries' largest as unsigned integers, the order in which the kernels'
  // atomics raised them: a NaN is above every number (wave_max passes NaNs over).
  unsigned long long e[3], top[3];
  bool nan = false;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    e[s] = parts[(s * kSmaxParts + lane) * kSmaxStride];
    nan |= e[s] > 0x7ff0000000000000ull;
    top[s] = (unsigned long long)__double_as_longlong(wave_max(__longlong_as_double((long long)e[s])));
  }
  if (__ballot(nan) != 0) {
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const unsigned long long who = __ballot(e[s] > 0x7ff0000000000000ull);
      if (who != 0) top[s] = __shfl(e[s], __ffsll((long long)who) - 1);
    }
  }
  if (lane < words) {
    constexpr int first = (int)(offsetof(Ctrl, smax) / sizeof(unsigned long long));
    unsigned long long w = reinterpret_cast<const unsigned long long*>(ctrl)[lane];
#pragma unroll
    for (int s = 0; s < 3; ++s)
      if (lane == first + s) w = top[s];
    reinterpret_cast<unsigned long long*>(out)[lane] = w;
  }
}

hipError_t launch_report(const Ctrl* ctrl, const unsigned long long* parts, char* stage, hipStream_t s) {
  hipLaunchKernelGGL(k_report, dim3(1), dim3(64), 0, s, ctrl, parts, reinterpret_cast<Ctrl*>(stage));
  return hipGetLastError();
}

template <class R, bool IN>
__global__ __launch_bounds__(256) void k_rows(const Rows<R> a, double* host) {
  const int row = (int)blockIdx.y, c = row / (a.P + 1), k = row - c * (a.P + 1);
  double* h = host + (int64_t)row * a.n;
  for (int j = (int)(blockIdx.x * blockDim.x + threadIdx.x); j < a.n; j += (int)(gridDim.x * blockDim.x)) {
    if (k == 0) {
      double* d = a.p + (int64_t)c * a.ld + j;
      if (IN) *d = h[j]; else h[j] = *d;
    } else {
      R* d = a.d + (int64_t)(c * a.P + (k - 1)) * a.ld + j;
      if (IN) *d = (R)h[j]; else h[j] = (double)*d;
    }
  }
}

template <class R, bool IN>
static hipError_t launch_rows(const Rows<R>& rows, char* stage, hipStream_t s) {
  if (rows.n < 1 || !stage_fits(rows.nc, rows.P, rows.n)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)std::min(64, (rows.n + 255) / 256), (unsigned)(rows.nc * (rows.P + 1)));
  hipLaunchKernelGGL((k_rows<R, IN>), grid, dim3(256), 0, s, rows, reinterpret_cast<double*>(stage + kStageHead));
  return hipGetLastError();
}

template <class R>
hipError_t launch_rows_in(const Rows<R>& rows, const char* stage, hipStream_t s) {
  return launch_rows<R, true>(rows, const_cast<char*>(stage), s);
}
template <class R>
hipError_t launch_rows_out(const Rows<R>& rows, char* stage, hipStream_t s) {
  return launch_rows<R, false>(rows, stage, s);
}

template hipError_t launch_rows_in<double>(const Rows<double>&, const char*, hipStream_t);
template hipError_t launch_rows_in<float>(const Rows<float>&, const char*, hipStream_t);
template hipError_t launch_rows_out<double>(const Rows<double>&, char*, hipStream_t);
template hipError_t launch_rows_out<float>(const Rows<float>&, char*, hipStream_t);

}  // namespace wcc
