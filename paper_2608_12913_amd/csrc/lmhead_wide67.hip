// lmhead_wide_kernel with 6 and 7 row blocks per wave (192 and 224 rows per workgroup).
#define DCD_WIDE_LO 6
#define DCD_WIDE_LAUNCH launch_lmhead_wide67
#include "lmhead_wide.hip"
