// wcc_march.hip -- many half-steps of a small instance in one launch.
//
// A half-step of a few hundred cells is 1 to 3 us of work on a handful of
// wavefronts, but as a launch of its own it costs 4 to 6 us: dispatch, the
// ring and the state read from beyond the (invalidated) caches, the wave
// speeds reduced through memory for the next launch.  Here one work-group
// keeps the whole state in LDS and takes many half-steps: each wave owns one
// 63-cell tile (the same per-cell code as wcc_kernels.hip, so the same bits),
// the new cells go to the other of two LDS buffers, and one barrier a
// half-step publishes them together with the waves' largest speeds.  The time
// control of step_time runs in every wave on the same values; the ring in
// memory is read at the start and written at the end, as that many launches
// would leave it.
//
// What bounds it: the dependent binary64 chains of one cell, then the compute
// unit's issue rate.  Counters (Euler, P = 3, 915 vector instructions a wave and
// half-step): with one wave per SIMD 2.5 us, vector issue 0.65 of the time; with
// two 3.9 us, 0.82; P = 1 with four 4.3 us, 0.94.  Advection P = 2, one wave:
// 1.0 us, 0.48.  (march_tiles in wcc_march.hpp.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wcc_cell.hpp"
#include "wcc_internal.hpp"
#include "wcc_march.hpp"
#include "wcc_tile.hpp"

namespace wcc {

template <int EQ, int P, class R>
struct MarchState {
  static constexpr int NC = ncomp<EQ>();
  static constexpr int kCells = march_tiles(EQ, P, sizeof(R)) * 63 + 1;
  double p[NC][kCells];
  R d[P > 0 ? NC * P : 1][kCells];
};

template <int EQ, int P, bool LIM, class R>
__global__ __launch_bounds__(march_tiles(EQ, P, sizeof(R)) * 64) void k_march(const MarchArgs<R> a) {
  constexpr int NC = ncomp<EQ>();
  __shared__ MarchState<EQ, P, R> state[2];
  __shared__ double red_s[2][16];
  __shared__ unsigned red_f[2][16];
  __shared__ double ghost[2][3];
  const StepIn ring = step_load(a.ctrl, a.parts, a.slot);
  const int lane = threadIdx.x & 63, tile = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
            nw = blockDim.x >> 6;
  auto cells = [&](int parity) { return a.bc == kPeriodic || parity ? a.N : a.N + 1; };

  // the state into the LDS buffer of its mesh
  const int n0 = cells(a.parity);
  for (int j = threadIdx.x; j < n0; j += blockDim.x) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      state[a.parity].p[c][j] = a.p[a.parity][(int64_t)c * a.ld + j];
#pragma unroll
      for (int k = 0; k < P; ++k) state[a.parity].d[c * P + k][j] = a.d[a.parity][(int64_t)(c * P + k) * a.ld + j];
    }
  }
  if (threadIdx.x < 6) ghost[threadIdx.x / 3][threadIdx.x % 3] = a.ctrl->ghost[threadIdx.x / 3][threadIdx.x % 3];
  __syncthreads();

  // the old cell of this lane, as fetch_tile maps it
  auto fetch = [&](int parity, TileIn<EQ, P, R>& in) {
    int g;
    const int o = map_old(tile * 63 + lane - parity, cells(parity), a.N, a.bc, parity, g);
    const MarchState<EQ, P, R>& s = state[parity];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      in.p[c] = s.p[c][o];
      in.d[c][0] = (R)0;
#pragma unroll
      for (int k = 1; k <= P; ++k) in.d[c][k] = s.d[c * P + (k - 1)][o];
    }
    if (g) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        in.p[c] = ghost[g - 1][c];
#pragma unroll
        for (int k = 1; k <= P; ++k) in.d[c][k] = (R)0;
      }
    }
  };

  double t = ring.t, smax = wave_max(__longlong_as_double((long long)ring.smax));
  unsigned flags = ring.flags;
  int parity = a.parity, taken = 0;
  TileIn<EQ, P, R> in;
  fetch(parity, in);
  // every wave sees the same t, smax and flags, so all leave together
  while (taken < a.steps && flags == 0u && t < ring.t_end) {
    double dt = div_rn(ring.cfl * a.dx, smax);
    const double rem = ring.t_end - t;
    if (dt >= rem) {
      dt = rem;
      t = ring.t_end;
    } else {
      t = t + dt;
    }
    const double lam = div_rn(dt, a.dx);
    const int n_new = cells(1 - parity);
    double sp = 0.0;
    unsigned fl = 0u;
    if (tile * 63 < n_new) {
      double pn[NC];
      R dn[NC][P + 1];
      auto reread = [&](TileIn<EQ, P, R>& x) { fetch(parity, x); };   // the old state's buffer is still whole
      if (tile_cells<EQ, P, LIM, R>(a.ph, n_new, tile, in, reread, lam, (R)(-lam), lane, sp, fl, pn, dn)) {
        MarchState<EQ, P, R>& s = state[1 - parity];
        const int j = tile * 63 + lane;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          s.p[c][j] = pn[c];
#pragma unroll
          for (int k = 1; k <= P; ++k) s.d[c * P + (k - 1)][j] = dn[c][k];
        }
      }
    }
    sp = wave_max(sp);
    fl = wave_or(fl);
    if (lane == 0) {
      red_s[parity][tile] = sp;
      red_f[parity][tile] = fl;
    }
    // One barrier a half-step: what it publishes is overwritten two
    // half-steps later, after every wave has passed the next barrier and so
    // has read it.
    __syncthreads();
    const double mine = (lane & 15) < nw ? red_s[parity][lane & 15] : 0.0;
    const unsigned fmine = (lane & 15) < nw ? red_f[parity][lane & 15] : 0u;
    parity ^= 1;
    ++taken;
    fetch(parity, in);
    smax = wave_max(mine);
    flags = wave_or(fmine);
  }

  // the state and the ring as `steps` launches leave them
  if (taken > 0) {
    const int n = cells(parity);
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        a.p[parity][(int64_t)c * a.ld + j] = state[parity].p[c][j];
#pragma unroll
        for (int k = 0; k < P; ++k) a.d[parity][(int64_t)(c * P + k) * a.ld + j] = state[parity].d[c * P + k][j];
      }
    }
  }
  if (tile == 0) {
    const int s1 = (a.slot + a.steps) % 3, s2 = s1 == 2 ? 0 : s1 + 1;
    // (no half-step taken: the slot's entries move on as they are)
    a.parts[(s1 * kSmaxParts + lane) * kSmaxStride] =
        taken == 0 ? ring.smax : (lane == 0 ? (unsigned long long)__double_as_longlong(smax) : 0ull);
    a.parts[(s2 * kSmaxParts + lane) * kSmaxStride] = 0ull;
    if (lane == 0) {
      a.ctrl->t[s1] = t;
      a.ctrl->flags[s1] = flags;
      a.ctrl->flags[s2] = 0u;
      a.ctrl->steps_done = ring.done + taken;
    }
  }
}

namespace {

template <int EQ, int P, class R>
hipError_t march_lim(const MarchArgs<R>& a, bool lim, int threads, hipStream_t s) {
  if (lim && P >= 1)
    hipLaunchKernelGGL((k_march<EQ, P, (P >= 1), R>), dim3(1), dim3(threads), 0, s, a);
  else
    hipLaunchKernelGGL((k_march<EQ, P, false, R>), dim3(1), dim3(threads), 0, s, a);
  return hipGetLastError();
}

template <int EQ, class R>
hipError_t march_p(const MarchArgs<R>& a, int P, bool lim, hipStream_t s) {
  const int nmax = a.bc == kPeriodic ? a.N : a.N + 1, tiles = (nmax + 62) / 63;
  if (tiles > march_tiles(EQ, P, sizeof(R)) || a.steps < 1 || a.steps > kMarchSteps) return hipErrorInvalidValue;
  switch (P) {
    case 0: return march_lim<EQ, 0, R>(a, false, tiles * 64, s);
    case 1: return march_lim<EQ, 1, R>(a, lim, tiles * 64, s);
    case 2: return march_lim<EQ, 2, R>(a, lim, tiles * 64, s);
    case 3: return march_lim<EQ, 3, R>(a, lim, tiles * 64, s);
    case 4: return march_lim<EQ, 4, R>(a, lim, tiles * 64, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool march_built() { return true; }

template <class R>
hipError_t launch_march(const MarchArgs<R>& a, int eq, int P, bool lim, hipStream_t s) {
  switch (eq) {
    case kAdvection: return march_p<kAdvection, R>(a, P, lim, s);
    case kBurgers: return march_p<kBurgers, R>(a, P, lim, s);
    case kEuler: return march_p<kEuler, R>(a, P, lim, s);
  }
  return hipErrorInvalidValue;
}

template hipError_t launch_march<double>(const MarchArgs<double>&, int, int, bool, hipStream_t);
template hipError_t launch_march<float>(const MarchArgs<float>&, int, int, bool, hipStream_t);

}  // namespace wcc
