// Fused z passes of the lengths in PSATD_Z_D.
#include "zfused_kernel.hpp"

PSATD_Z_DEFINE(d, PSATD_Z_D)
