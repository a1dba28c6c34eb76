// Instantiation unit of the spectral kernel (spectral_impl.h) without the sums
// (G_loc only) for band windows padded to 64.
#define SPEC_NBP 64
#define SPEC_NAME launch_spectral_gloc_64
#define SPEC_WS false
#include "spectral_unit.h"
