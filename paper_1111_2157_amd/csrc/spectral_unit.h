// Body of a spectral instantiation unit: SPEC_NAME launches spec_kernel<SPEC_NBP,
// ncls, SPEC_WS>, a grid of one item each (items null) or a drain of a queue.
#include "spectral_lane_impl.h"

namespace dmft {
hipError_t SPEC_NAME(int ncls, const DysonArgs& a, const void* items, int n_items, const DysonArgs* args, int* counter,
                     int grid, hipStream_t s) {
  const SpecItem* it = reinterpret_cast<const SpecItem*>(items);
#define SPEC_CASE(NC)                                                                                           \
  case NC:                                                                                                      \
    hipLaunchKernelGGL((spec_kernel<SPEC_NBP, NC, SPEC_WS>), dim3(grid), dim3(256), 0, s, a, it, n_items, args, \
                       counter);                                                                                \
    break;
#define SPEC_LANE_CASE(NC)                                                                                        \
  case NC:                                                                                                       \
    hipLaunchKernelGGL((spec_lane_kernel<SPEC_NBP, NC, SPEC_WS>), dim3(grid), dim3(64), 0, s, a, it, n_items, args, \
                       counter);                                                                                 \
    break;
  switch (ncls) {
    SPEC_LANE_CASE(4)
    SPEC_LANE_CASE(5)
    SPEC_CASE(6)
    SPEC_CASE(8)
    SPEC_CASE(10)
    SPEC_CASE(12)
    SPEC_CASE(14)
    SPEC_CASE(16)
    default: return hipErrorInvalidValue;
  }
#undef SPEC_CASE
#undef SPEC_LANE_CASE
  return hipGetLastError();
}
}  // namespace dmft
