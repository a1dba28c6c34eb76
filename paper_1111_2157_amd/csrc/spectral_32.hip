// Instantiation unit of the spectral density kernel (spectral_impl.h) for band
// windows padded to 32: one kernel per padded orbital count.
#define SPEC_NBP 32
#define SPEC_NAME launch_spectral_32
#define SPEC_WS true
#include "spectral_unit.h"
