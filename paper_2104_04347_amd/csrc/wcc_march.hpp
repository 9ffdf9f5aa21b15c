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

// Half-steps one launch may take: 16 to 20 ms at the largest meshes, 4 ms at one
// tile of a scalar equation.
constexpr int kMarchSteps = 4096;

// Wave tiles (one wave each) that one work-group marches.  The state of that
// many tiles, twice, fits its 160 KB of LDS, and up to there a half-step is
// faster than as a launch of its own (us, binary64 unless noted, march
// against launches of the default shape, full work-group):
//   Euler   P = 0: 16 tiles 1.96 / 3.69;  P = 1: 16 tiles 4.30 / 4.39;
//           P = 2: 12 tiles 4.41 / 4.97;
//           P = 3: 8 tiles 3.91 / 5.51 (one wave per SIMD: 2.49 / 5.18);
//           P = 4: 8 tiles 4.85 / 6.25
//           FP32-mixed P = 1: 16 tiles 3.22 / 4.05;  P = 2, 3, 4: 12 tiles
//           3.20 / 4.46, 3.99 / 4.94, 5.05 / 5.59
//   scalar  16 tiles: Burgers P = 1 1.81 / 3.64, P = 3 2.58 / 3.84,
//           P = 4 3.11 / 4.06; advection P = 4 2.67 / 3.98
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
