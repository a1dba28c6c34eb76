// Instantiation unit of the spectral trace and adjoint kernels (spectral_adj_impl.h)
// for band windows padded to 16.
#define SPEC_NBP 16
#define SPEC_NAME launch_spectral_adj_16
#include "spectral_adj_unit.h"
