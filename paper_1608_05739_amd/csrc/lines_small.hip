// Line passes of the lengths in PSATD_LINE_SMALL.
#include "lines_kernel.hpp"

PSATD_LINE_DEFINE(small, PSATD_LINE_SMALL)
