// How the small-batch product's work is shared out over workgroups: plain host arithmetic, apart from
// the kernel so that it can be checked on its own.
#ifndef ENDOR_GEMM_PLAN_H_
#define ENDOR_GEMM_PLAN_H_

#include <cstdint>

#include "endor_gemm_units.h"

namespace endor_gemm_plan {

constexpr int kSegCols = 256;  // columns per round: a 64-bit bitmap word per lane
constexpr int kGemmWaves = 4;  // waves (groups of 16 rows) per workgroup; they share the tile of X
constexpr int kBlockRows = endor_gemm_units::kRows * kGemmWaves;

// Every workgroup gets the same number of consecutive rounds, counted row block by row block: so many
// that kResident workgroups do all of them at once (two per compute unit; three fit most forms, 52 KB of
// LDS and 125 to 183 registers each, but shared out for three 28672 x 8192 took 85 us, for two 80), and so many that a row block has at most kMaxParts
// parts.  Whole blocks, which need no second kernel, where that costs a workgroup no more than
// kWholeSlack rounds (the kernel takes about as long as two rounds).  Small products, kSmall rounds or
// fewer per workgroup, run as workgroups of two rounds.  These, and those that fit the chip at once,
// never reach into a second block: starting on a block takes as long as several rounds (2053 x 1031:
// 13.8 us, 19.7 us with workgroups that cross from block to block).
//
// For the same reason more row blocks than kResident, each of kNarrow rounds or fewer, are a workgroup
// each: a workgroup's starts on one block after the other are then hidden behind the others' work.
// Measured, 16 right-hand sides, consecutive rounds against a block a workgroup: 524288 x 256
// 144 / 88 us, 1000000 x 128 279 / 165, 262144 x 512 80 / 62, 131072 x 1024 59 / 51, 36864 x 1024
// 29 / 21, 36864 x 2048 38 / 33, 33000 x 3072 47 / 46; but 36000 x 3584 51.5 / 52.3 and 36864 x 4096
// 56.9 / 59.2.  (The kernel before this form, of which four workgroups fit a compute unit and three of
// this one, was slower everywhere else but took 146 us on 10^6 x 256 with one in ten kept: now 147.)
constexpr int64_t kResident = 256 * 2;
constexpr int64_t kMaxParts = 16;
constexpr int64_t kWholeSlack = 2;
constexpr int64_t kSmall = 4;
constexpr int64_t kNarrow = 12;
constexpr int64_t kMaxGrid = int64_t(1) << 23;  // workgroups: a launch has fewer than 2^32 threads

struct Plan {
    uint32_t blocks, segs, per_wg, rounds, wgs;
    bool split;  // some row block is shared
};

inline Plan make_plan(int64_t rows, int64_t cols) {
    Plan p;
    const int64_t blocks = (rows + kBlockRows - 1) / kBlockRows;
    int64_t segs = (cols + kSegCols - 1) / kSegCols;
    int64_t per = (blocks * segs + kResident - 1) / kResident;  // blocks * segs is below 2^27: rows*cols < 2^34
    per = (per + 1) & ~int64_t(1);
    if (per <= kSmall) per = segs < 2 ? segs : 2;
    const int64_t least = (segs + kMaxParts - 1) / kMaxParts;
    if (per < least) per = least;
    const int64_t parts = (segs + per - 1) / per;
    if (per <= kSmall || blocks * parts <= kResident) segs = parts * per;  // rounds past the last column have no bits
    const int64_t rounds = blocks * segs;
    const int64_t whole = (per + segs - 1) / segs * segs;
    if (whole - per <= kWholeSlack) per = whole;
    if (blocks > kResident && segs <= kNarrow) per = segs * ((blocks + kMaxGrid - 1) / kMaxGrid);
    p.blocks = static_cast<uint32_t>(blocks);
    p.segs = static_cast<uint32_t>(segs);
    p.per_wg = static_cast<uint32_t>(per);
    p.rounds = static_cast<uint32_t>(rounds);
    p.wgs = static_cast<uint32_t>((rounds + per - 1) / per);
    p.split = per % segs != 0;
    return p;
}

}  // namespace endor_gemm_plan

#endif  // ENDOR_GEMM_PLAN_H_
