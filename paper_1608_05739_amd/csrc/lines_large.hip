// Line passes of the lengths in PSATD_LINE_LARGE.
#include "lines_kernel.hpp"

PSATD_LINE_DEFINE(large, PSATD_LINE_LARGE)
