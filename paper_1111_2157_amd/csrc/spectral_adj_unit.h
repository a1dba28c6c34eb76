// Body of an instantiation unit of the spectral trace and adjoint kernels:
// SPEC_NAME launches spec_adj_kernel<SPEC_NBP, ncls, what>, one item per work-group.
#include "spectral_adj_impl.h"

namespace dmft {
hipError_t SPEC_NAME(int ncls, int what, const DysonArgs& a, int grid, hipStream_t s) {
#define SPEC_WHAT(NC, W) hipLaunchKernelGGL((spec_adj_kernel<SPEC_NBP, NC, W>), dim3(grid), dim3(256), 0, s, a)
#define SPEC_CASE(NC)                    \
  case NC:                               \
    if (what == SPEC_TRACE)              \
      SPEC_WHAT(NC, SPEC_TRACE);         \
    else if (what == SPEC_ADJ)           \
      SPEC_WHAT(NC, SPEC_ADJ);           \
    else if (what == SPEC_GEN)           \
      SPEC_WHAT(NC, SPEC_GEN);           \
    else if (what == SPEC_GEN_N)         \
      SPEC_WHAT(NC, SPEC_GEN_N);         \
    else                                 \
      SPEC_WHAT(NC, SPEC_GEN_G);         \
    break;
  switch (ncls) {
    SPEC_CASE(5)
    SPEC_CASE(8)
    SPEC_CASE(10)
    SPEC_CASE(14)
    case 16:
      if (what != SPEC_TRACE) return hipErrorInvalidValue;
      SPEC_WHAT(16, SPEC_TRACE);
      break;
    default: return hipErrorInvalidValue;
  }
#undef SPEC_CASE
#undef SPEC_WHAT
  return hipGetLastError();
}
}  // namespace dmft
