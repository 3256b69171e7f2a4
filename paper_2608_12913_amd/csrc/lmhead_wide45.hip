// lmhead_wide_kernel with 4 and 5 row blocks per wave (128 and 160 rows per workgroup).
#define DCD_WIDE_LO 4
#define DCD_WIDE_LAUNCH launch_lmhead_wide45
#include "lmhead_wide.hip"
