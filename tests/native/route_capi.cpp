// The LM-head route of a problem (csrc/route.h) for the tests: rows per workgroup of the
// streaming kernel, or minus the row blocks per wave of the many-row kernel.
#include "route.h"

extern "C" int dcd_test_route(int R, int vocab, int dp, int dq, int bf16, int full) {
    const int ntiles = (vocab + dcd::kTileTokens - 1) / dcd::kTileTokens;
    const dcd::Route r =
        dcd::lmhead_route(dcd::RouteProblem{R, ntiles, dp, dq, bf16 ? dcd::kBF16 : dcd::kF32, full != 0});
    return r.wide_rb ? -r.wide_rb : r.stream_rows;
}
