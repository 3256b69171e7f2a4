// The streaming LM-head kernel with 32 rows per workgroup: the source of lmhead.hip
// compiled with that row shape.
#define DCD_STREAM_ROWS 32
#include "lmhead.hip"
