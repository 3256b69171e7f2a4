// Which LM-head kernel a problem takes and in which row shape: plain host code, also built
// into the tests, which check that a case runs the shape it is meant for.
#pragma once

namespace dcd {

constexpr int kTileTokens = 256;       // tokens per vocabulary tile (every LM-head kernel)
constexpr int kStreamRowsSmall = 64;   // the streaming kernel's largest shape that keeps both heads' logits in registers
constexpr int kStreamRowsLarge = 128;  // its largest shape (bf16: the most rows it takes)
constexpr int kCus = 256;              // compute units of an MI355X
constexpr int kXcds = 8;               // in XCDs; workgroup id modulo 8 is its XCD
constexpr int kWideMinRows = 512;      // rows from which fp32 takes at most 64 rows per workgroup
constexpr long long kMaxGroups = 0x7fffffffLL;

enum ElemType { kF32 = 0, kBF16 = 1 };

struct RouteProblem {
    int R;          // rows (batch x nodes)
    int ntiles;     // vocabulary tiles
    int dp, dq;     // hidden sizes
    int dtype;      // ElemType
    bool full;      // untruncated target
};

// One of the two is 0: rows per workgroup of the streaming kernel (16, 32, 48, 64 or 128), or
// row blocks per wave of the many-row kernel (4 to 9: 32 rows per workgroup each).  Times below:
// whole greedy steps on one MI355X.
struct Route {
    int stream_rows, wide_rb;
};

inline int row_blocks_of(int R, int rows) { return (R + rows - 1) / rows; }

// workgroups of the streaming kernel with `rows` rows each: the row blocks of a vocabulary tile
// go to one XCD, the tiles to the XCDs in turn
inline long long stream_groups_per_xcd(int ntiles, int R, int rows) {
    return (long long)((ntiles + kXcds - 1) / kXcds) * row_blocks_of(R, rows);
}
inline long long stream_groups(int ntiles, int R, int rows) {
    return kXcds * stream_groups_per_xcd(ntiles, R, rows);
}

// fp32.  The matrix cores bound it (the fp32 rate is a sixteenth of bf16's), so padding rows
// cost as much as real ones; but workgroups of few rows also wait longer for loads, and several
// row blocks read every weight again through L2.  The shape of the least estimated time is
// taken, from coefficients measured per shape (us):
//   chunk   per 128-byte K chunk and workgroup a CU has to do (0.43 per 16 rows is the fp32
//           matrix rate), with the mean of the busiest CU's count and the average one
//   round   per chunk and round of the workgroups that share a CU (`resident`, bounded by their
//           registers): the load latency that one batch in flight leaves exposed
//   stream  per chunk and 65,536 tokens: what the weight stream adds to the matrix time
//   group   per workgroup: its epilogues; masked: the mask's part, where short workgroups meet at
//           the row bounds' atomics
//   once    prologue and the rest
// Measured in all shapes at 2,738 points (1 to 2048 rows, 1,000 to 128,256 tokens, heads of 64/64
// to 8192/4096, masked and not): the choice takes more than 3% longer than the best shape at
// 142 of them, more than 5% at 62 (heads narrower than 512, or rows that are no multiple of 128
// bytes).  Against 64 rows (to 64 rows and from 512) or 128 (between) it is 1.51 times as fast in
// the geometric mean and more than 3% slower at 14 points (at most 9%, 4.5 us).  4096/2048-wide
// heads, in 16, 32, 48, 64 and 128 rows: 64 rows of 128,256 tokens 1152, 1012, 1367, 909 us; 112
// rows 1891, 1803, 2003, 1683, 1596; 304 rows 4800, 4364, 4519, 4041, 4631; 64 rows of 32,003
// tokens 333, 294, 397, 473; 8 rows of 128,256 tokens 485, 560, 751, 892.  Heads of 96/32, masked, 49
// rows of 128,256 tokens: 89, 62, 73, 47.
struct Fp32Shape {
    int rows, resident;
    double chunk, round, stream, group, masked, once;
};
constexpr Fp32Shape kFp32Shapes[] = {
    {128, 2, 3.68, 0.436, 0.26, 13.2, 0.0, 15.1}, {64, 2, 1.70, 0.681, 0.183, 7.05, 0.0, 3.74},
    {48, 2, 1.41, 0.518, 0.195, 5.93, 0.371, 4.0}, {32, 3, 0.857, 0.473, 0.398, 2.80, 0.913, 2.76},
    {16, 4, 0.464, 0.411, 0.504, 1.25, 1.4, 1.68},
};

inline double fp32_cost(const RouteProblem &p, const Fp32Shape &s) {
    const auto chunks_of = [](int d) { return ((long long)d * 4 + 127) / 128; };
    const double chunks = (double)(chunks_of(p.dp) + chunks_of(p.dq));
    const long long groups = stream_groups_per_xcd(p.ntiles, p.R, s.rows), cus = kCus / kXcds;
    const long long busiest = (groups + cus - 1) / cus, rounds = (busiest + s.resident - 1) / s.resident;
    const double average = (double)groups / (double)cus, work = ((double)busiest + (average > 1.0 ? average : 1.0)) / 2;
    return chunks * (s.chunk * work + s.round * (double)rounds + s.stream * p.ntiles / 256.0) +
           (p.full ? s.group : s.group + s.masked) * work + s.once;
}

inline int fp32_stream_rows(const RouteProblem &p) {
    int best = kStreamRowsSmall;
    double least = -1.0;
    for (const Fp32Shape &s : kFp32Shapes) {
        // (the 128-row shape parks the expert logits in the workspace, which has room for them there)
        if (s.rows == kStreamRowsLarge && (p.R <= kStreamRowsSmall || p.R >= kWideMinRows)) continue;
        if (stream_groups(p.ntiles, p.R, s.rows) > kMaxGroups) continue;
        const double cost = fp32_cost(p, s);
        if (least < 0.0 || cost < least) best = s.rows, least = cost;
    }
    return best;
}

// bf16: the weight stream bounds it, so rows share a workgroup where the tiles alone fill
// the chip.  Where they do not, the smallest shape that still gives every workgroup a CU of
// its own is the fastest, as each has less to stage, read and reduce: 64 rows, 4096/2048,
// 8,000 tokens 116 us with 64, 71 with 16; 32,003 tokens 123 and 114 (32 rows; 16 rows make
// two rounds, 136); 128 rows, 32,003 tokens 165 with 128, 126 with 64.  Otherwise the
// smallest shape that holds the rows: 6 untruncated rows, 128,256 tokens 253 us with 64,
// 243 with 16; 80 rows there 292 with 128, 341 in two blocks of 48.  Masked, 32 or more rows, and
// in narrow heads 64, as workgroups that end sooner meet at the row bounds' atomics.  128,256
// tokens, masked, 1, 17 and 33 rows with 32 (48 for 33 rows) against 64: heads of 144/64 (208
// columns) 54, 44, 42 and 44, 44, 41 us; 304/136 58, 53, 54 and 58, 55, 54; 448/192 42, 45, 52 and 48,
// 51, 53; 656/272 (928) 78, 78, 81 and 80, 78, 78; 768/384 59, 63, 68 and 64, 68, 69; 1024/512 74, 77, 81
// and 77, 80, 82; 4096/2048 within 1%.  The line at 1024 columns lies where none was slower any more.
//
// bf16 above 128 rows: the many-row kernel, except where 16 or 32 rows give every workgroup
// a CU of its own and a weight byte is re-read for at most 32 row blocks.  4096/2048-wide
// heads, many-row kernel against that: 200 rows of 1,024 tokens 94 and 73 us, 512 rows 104
// and 89, 1024 rows 128 and 121 (16 rows, 64 blocks: 135), 512 rows of 4,096 tokens 105 and
// 96, 200 rows of 8,000 tokens 93 and 83; in two rounds it is slower (304 rows there: 100
// and 117), with 48 or 64 rows too (107 and 117).
// LM heads over 128,256 tokens, 128 rows against the many-row kernel: 128 rows 295 and
// 308 us, 160 rows 480 and 325, 256 rows 505 and 400.
inline int bf16_stream_rows(const RouteProblem &p) {  // 0: the many-row kernel
    constexpr int shapes[] = {16, 32, 48, kStreamRowsSmall, kStreamRowsLarge};
    const bool many = p.R > kStreamRowsLarge;
    for (int rows : shapes) {
        const long long nrb = row_blocks_of(p.R, rows);
        if (rows <= (many ? 32 : kStreamRowsSmall) && nrb <= 32 && p.ntiles * nrb <= kCus) return rows;
    }
    if (many) return 0;
    const int least_rows = p.dp + p.dq >= 1024 ? 32 : kStreamRowsSmall;
    for (int rows : shapes)
        if (rows >= p.R && (p.full || rows >= least_rows)) return rows;
    return kStreamRowsLarge;  // (the last shape holds them)
}

// Row blocks per wave of the many-row kernel (32 * RB rows per workgroup): the workgroups run in
// rounds of one per CU, and a round takes about as long as RB row blocks and a constant part (the
// weights' share of a chunk, prologue, epilogues).  Over 132 to 2048 rows and vocabularies of
// 4,096 to 128,256 tokens the choice was within 4% of the best of the six shapes, mostly
// within 1%; the worst fixed shape is up to 2.5 times slower.
inline int wide_row_blocks(int ntiles, int R) {
    int best = 0;
    long long best_cost = 0;
    for (int rb = 4; rb <= 9; ++rb) {
        const long long groups = (long long)ntiles * row_blocks_of(R, 32 * rb);
        const long long cost = ((groups + kCus - 1) / kCus) * (2 * rb + 3);
        if (!best || cost < best_cost) best = rb, best_cost = cost;
    }
    return best;
}

inline Route lmhead_route(const RouteProblem &p) {
    if (p.dtype == kF32) return Route{fp32_stream_rows(p), 0};
    const int rows = bf16_stream_rows(p);
    return Route{rows, rows ? 0 : wide_row_blocks(p.ntiles, p.R)};
}

}  // namespace dcd
