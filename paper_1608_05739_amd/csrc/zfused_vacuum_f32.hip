// Fused z passes of a family of lengths in one launch: vacuum, FP32.
#include "zfused_family.hpp"

PSATD_ZS_DEFINE(vacuum_f32, float, kVacuum)
