// Line passes of the lengths in PSATD_LINE_MID.
#include "lines_kernel.hpp"

PSATD_LINE_DEFINE(mid, PSATD_LINE_MID)
