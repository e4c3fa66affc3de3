// Fused z passes of a family of lengths in one launch: J form, FP64.
#include "zfused_family.hpp"

PSATD_ZS_DEFINE(j_f64, double, kJForm)
