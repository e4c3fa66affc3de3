// Fused z passes of the lengths in PSATD_Z_E.
#include "zfused_kernel.hpp"

PSATD_Z_DEFINE(e, PSATD_Z_E)
