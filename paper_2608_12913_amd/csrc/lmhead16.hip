// The streaming LM-head kernel with 16 rows per workgroup: the source of lmhead.hip
// compiled with that row shape.
#define DCD_STREAM_ROWS 16
#include "lmhead.hip"
