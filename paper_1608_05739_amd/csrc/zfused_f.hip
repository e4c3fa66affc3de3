// Fused z passes of the lengths in PSATD_Z_F.
#include "zfused_kernel.hpp"

PSATD_Z_DEFINE(f, PSATD_Z_F)
