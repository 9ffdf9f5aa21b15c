// wcc_march.hpp -- many half-steps of a small instance in one launch
// (wcc_march.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "wcc_internal.hpp"

namespace wcc {

template <class R>
struct MarchArgs {
  double* p[2];           // point values of the two meshes, [c][j]
  R* d[2];                // derivatives, [c][k-1][j]
  int32_t ld;             // row length (cells)
  int32_t N;
  int32_t bc;
  int32_t parity;         // mesh of the state at the start
  int32_t slot;           // ring slot of the first half-step
  int32_t steps;          // half-steps to take (fewer at the end time or after a raised flag)
  double dx;
  Phys<R> ph;
  Ctrl* ctrl;
  unsigned long long* parts;
};

// Half-steps one launch may take: about 10 ms at the largest mesh.
constexpr int kMarchSteps = 4096;

// Wave tiles (one wave each) that one work-group marches.  The state of that
// many tiles, twice, fits its 160 KB of LDS, and up to there a half-step is
// faster than as a launch of its own (us, binary64 unless noted, march
// against launches, full work-group):
//   Euler   P = 1: 16 tiles 4.21 / 4.40;  P = 2: 12 tiles 4.41 / 5.06;
//           P = 3: 8 tiles 3.96 / 5.67 (one wave per SIMD: 2.54 / 5.41);
//           P = 4: 8 tiles 4.92 / 6.55;  FP32-mixed P = 3, 12 tiles 4.20 / 5.00
//   scalar  16 tiles: Burgers P = 1 1.83 / 3.74, P = 4 3.15 / 4.18
// With four waves of the higher degrees on a SIMD the one compute unit's issue
// rate costs what the launches did.
constexpr int march_tiles(int eq, int P, int elem_bytes) {
  return eq != kEuler || P <= 1 ? 16 : (P == 2 || elem_bytes == 4 ? 12 : 8);
}

// Whether this library holds the kernels of this form (the diagnostic one, which
// records launches, does not).
bool march_built();

template <class R>
hipError_t launch_march(const MarchArgs<R>& a, int eq, int P, bool lim, hipStream_t s);

}  // namespace wcc
