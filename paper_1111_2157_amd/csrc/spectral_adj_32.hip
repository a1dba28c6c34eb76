// Instantiation unit of the spectral trace and adjoint kernels (spectral_adj_impl.h)
// for band windows padded to 32.
#define SPEC_NBP 32
#define SPEC_NAME launch_spectral_adj_32
#include "spectral_adj_unit.h"
