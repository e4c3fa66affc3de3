// Fused z passes of a family of lengths in one launch: vacuum, FP64.
#include "zfused_family.hpp"

PSATD_ZS_DEFINE(vacuum_f64, double, kVacuum)
