// Dispatch of the low-rank Dyson kernel (lowrank_impl.h) over the padded
// band-window sizes; the kernels are instantiated in lowrank_{16,32,48,64}.hip.
#include <hip/hip_runtime.h>

#include "dmft_internal.h"

namespace dmft {

hipError_t launch_lowrank_16(int var, const DysonArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_lowrank_32(int var, const DysonArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_lowrank_48(int var, const DysonArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_lowrank_64(int var, const DysonArgs& a, dim3 grid, hipStream_t s);
int lowrank_variants_16(int kind, int* out, int max);
int lowrank_variants_32(int kind, int* out, int max);
int lowrank_variants_48(int kind, int* out, int max);
int lowrank_variants_64(int kind, int* out, int max);
hipError_t launch_lowrank_pair64(const DysonArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_lowrank_p3(int nbp, const DysonArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_spectral(int nbp, int ncls, const DysonArgs& a, const void* items, int n_items,
                           const DysonArgs* args, int* counter, int grid, hipStream_t s);

hipError_t launch_lowrank(int nbp, int var, const DysonArgs& a, dim3 grid, hipStream_t s) {
  if (var == kLowrankPairVariant) return nbp == 64 ? launch_lowrank_pair64(a, grid, s) : hipErrorInvalidValue;
  if (var == kLowrankP3Variant) return lowrank_p3_fits(nbp, a.nc) ? launch_lowrank_p3(nbp, a, grid, s) : hipErrorInvalidValue;
  switch (nbp) {
    case 16: return launch_lowrank_16(var, a, grid, s);
    case 32: return launch_lowrank_32(var, a, grid, s);
    case 48: return launch_lowrank_48(var, a, grid, s);
    case 64: return launch_lowrank_64(var, a, grid, s);
    default: return hipErrorInvalidValue;
  }
}

int lowrank_variants(int nbp, int kind, int* out, int max) {
  if (max <= 0) return 0;
  switch (nbp) {
    case 16:
    case 32:
    case 48: {
      int n = nbp == 16 ? lowrank_variants_16(kind, out, max)
              : nbp == 32 ? lowrank_variants_32(kind, out, max) : lowrank_variants_48(kind, out, max);
      if (kind == 0 && n < max) out[n++] = kLowrankP3Variant;
      return n;
    }
    case 64: {
      int n = lowrank_variants_64(kind, out, max);
      if (kind == 0 && n < max) out[n++] = kLowrankPairVariant;
      if (kind == 0 && n < max) out[n++] = kLowrankP3Variant;
      return n;
    }
    default: return 0;
  }
}

// Classes of the batched low-rank pass: the spectral kernel of each padded size
// and orbital count.
int lr_nc_class(int, int nc) { return spec_ncls(nc); }

int lr_class_wgs_per_cu(int nbp, int ncls) { return spec_wgs_per_cu(nbp, ncls); }

hipError_t launch_lr_class(int nbp, int ncls, const void* items, int n_items, const DysonArgs* args, int* counter,
                           int grid, hipStream_t s) {
  return launch_spectral(nbp, ncls, DysonArgs{}, items, n_items, args, counter, grid, s);
}

}  // namespace dmft
