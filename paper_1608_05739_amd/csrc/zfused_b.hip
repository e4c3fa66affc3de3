// Fused z passes of the lengths in PSATD_Z_B.
#include "zfused_kernel.hpp"

PSATD_Z_DEFINE(b, PSATD_Z_B)
