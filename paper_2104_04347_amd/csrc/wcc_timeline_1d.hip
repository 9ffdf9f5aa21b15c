// wcc_timeline_1d.hip -- diagnostic build of the 1D half-step kernels (64-cell wave tiles) with per-wave timestamps
// (linked into libwcc_timeline.so in place of wcc_kernels.hip; see wcc_timeline.hpp).
#include "wcc_timeline.hpp"

#define step_load(...) step_load_tl(__VA_ARGS__)
#define publish(...) publish_tl(__VA_ARGS__)
#include "wcc_kernels.hip"
#undef step_load
#undef publish

WCC_TIMELINE_ENTRY_POINTS(1d)
