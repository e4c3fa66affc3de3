// Fused z passes of a family of lengths in one launch: J form, FP32.
#include "zfused_family.hpp"

PSATD_ZS_DEFINE(j_f32, float, kJForm)
