// Instantiation unit of the spectral density kernel (spectral_impl.h) for band
// windows padded to 48: one kernel per padded orbital count.
#define SPEC_NBP 48
#define SPEC_NAME launch_spectral_48
#define SPEC_WS true
#include "spectral_unit.h"
