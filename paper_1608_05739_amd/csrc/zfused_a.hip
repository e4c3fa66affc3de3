// Fused z passes of the lengths in PSATD_Z_A.
#include "zfused_kernel.hpp"

PSATD_Z_DEFINE(a, PSATD_Z_A)
