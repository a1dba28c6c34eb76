// Instantiation unit of the spectral trace and adjoint kernels (spectral_adj_impl.h)
// for band windows padded to 64.
#define SPEC_NBP 64
#define SPEC_NAME launch_spectral_adj_64
#include "spectral_adj_unit.h"
