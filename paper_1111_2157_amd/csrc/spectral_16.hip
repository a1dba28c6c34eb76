// Instantiation unit of the spectral density kernel (spectral_impl.h) for band
// windows padded to 16: one kernel per padded orbital count.
#define SPEC_NBP 16
#define SPEC_NAME launch_spectral_16
#define SPEC_WS true
#include "spectral_unit.h"
