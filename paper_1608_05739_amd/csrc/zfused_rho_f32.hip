// Fused z passes of a family of lengths in one launch: rho form, FP32.
#include "zfused_family.hpp"

PSATD_ZS_DEFINE(rho_f32, float, kRho)
