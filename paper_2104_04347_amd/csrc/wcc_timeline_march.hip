// wcc_timeline_march.hip -- stands in for wcc_march.hip in libwcc_timeline.so:
// the diagnostic library records the waves of each half-step's launch, so it has
// no form that runs many half-steps in one, and small meshes take the same
// kernels as larger ones there.
#include "wcc_march.hpp"

namespace wcc {

bool march_built() { return false; }

template <class R>
hipError_t launch_march(const MarchArgs<R>&, int, int, bool, hipStream_t) {
  return hipErrorNotSupported;
}

template hipError_t launch_march<double>(const MarchArgs<double>&, int, int, bool, hipStream_t);
template hipError_t launch_march<float>(const MarchArgs<float>&, int, int, bool, hipStream_t);

}  // namespace wcc
