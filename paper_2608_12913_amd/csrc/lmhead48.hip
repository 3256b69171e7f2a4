// The streaming LM-head kernel with 48 rows per workgroup: the source of lmhead.hip
// compiled with that row shape.
#define DCD_STREAM_ROWS 48
#include "lmhead.hip"
