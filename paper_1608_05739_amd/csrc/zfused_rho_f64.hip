// Fused z passes of a family of lengths in one launch: rho form, FP64.
#include "zfused_family.hpp"

PSATD_ZS_DEFINE(rho_f64, double, kRho)
