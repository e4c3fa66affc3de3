// Line passes of the lengths in PSATD_LINE_LONG.
#include "lines_kernel.hpp"

PSATD_LINE_DEFINE(long, PSATD_LINE_LONG)
