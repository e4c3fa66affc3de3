// Fused z passes of the lengths in PSATD_Z_C.
#include "zfused_kernel.hpp"

PSATD_Z_DEFINE(c, PSATD_Z_C)
