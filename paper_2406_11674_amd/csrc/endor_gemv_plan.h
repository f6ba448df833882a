// How the vector products' work is shared out over segments, waves and workgroups: plain host arithmetic,
// apart from the kernel so that it can be checked on its own.
#ifndef ENDOR_GEMV_PLAN_H_
#define ENDOR_GEMV_PLAN_H_

#include <cstddef>
#include <cstdint>

namespace endor_gemv_plan {

constexpr int64_t kUnits = 256;    // compute units; one workgroup each (registers of all its waves)
constexpr size_t kLds = 160 * 1024;
constexpr size_t kTableBytes = 4224;  // the windows' selector tables

constexpr int waves_of(int steps) { return steps == 8 ? 12 : 16; }
// items of a workgroup, whose starts and sums take up to 16 KB of LDS (of 512, two vectors of 24576 would miss one
// panel of 8-step segments by 200 bytes)
constexpr int max_items(int steps, int rhs) { return steps == 8 && rhs == 2 ? 496 : 512; }
constexpr int64_t seg_cols(int steps) { return 512 * steps; }
// LDS of a workgroup beside x: tables, two segments' entries per wave, starts, ends and sums of its items
constexpr size_t lds_beside_x(int steps, int rhs) {
    return kTableBytes + size_t(waves_of(steps)) * 2 * 64 * steps * 4 + size_t(max_items(steps, rhs)) * (16 + 4 * rhs);
}
// segments of x that fit beside that
constexpr int64_t room_of(int steps, int rhs) {
    return static_cast<int64_t>((kLds - 64 - lds_beside_x(steps, rhs)) / (size_t(seg_cols(steps)) * 2 * rhs));
}
constexpr int most_steps(int rhs) { return rhs > 2 ? 4 : 8; }

constexpr int kMaxRhs = 4;

// Whether the vector form is the faster one for nb right-hand sides of the small-batch product.  Measured,
// us, the form on the matrix cores / this one:
//  - short rows, many of them: 36864 x 768 and one right-hand side 18.6 / 19 to 21, 131072 x 256 22 / 104;
//    12000 x 600 13 / 9.5, 20000 x 1200 24 / 16, 36864 x 1500 with two 29.6 / 27.4, with three 29.6 / 30.2;
//  - all of x has to fit LDS: two right-hand sides 4096 x 20000 39 / 28, 8192 x 28672 74 / 82; three
//    2000 x 16000 21.7 / 19.2, 4096 x 20000 39 / 46;
//  - four only pay on small matrices: 4096 x 4096 15 / 12, 12000 x 2500 27 / 22, 16384 x 4096 27 / 29,
//    36864 x 9216 107 / 117;
//  - else 28672 x 8192 with one to three 75 / 52, 59, 70; 4099 x 5005, three in ten kept, 18 / 12, 14, 15.
//  cols >= 8: shorter vectors are read element by element, which is there for one right-hand side only.
constexpr bool takes(int64_t rows, int64_t cols, int nb) {
    if (cols < 8 || nb > kMaxRhs || cols * nb > 48 * 1024) return false;
    if (nb == 4 && rows * cols > int64_t(1) << 25) return false;
    return rows <= 16384 || cols >= 1024 * (nb == 1 ? 1 : nb == 2 ? 1.4 : 2);
}

struct Plan {
    int steps;          // of 512 columns per segment
    int64_t parts;      // items per row and panel
    int64_t part_segs;  // segments per item
    int64_t panels;     // of parts * part_segs segments
    int64_t grid;       // workgroups
};

constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The plan with segments of that many steps and up to that many parts per row.  Where x does not fit LDS its
// panels are of about equal length: a wave walks every segment of every panel, whether it has columns or not.
// (4099 x 24576, two right-hand sides, 6 segments of which 5 fit: a panel of 5 and another of 5 with one
// segment to do took 61 us, one panel takes 32; 2000 x 100000 in panels that are filled in turn 69, of equal length 54.)
constexpr Plan plan_with(int64_t rows, int64_t cols, int rhs, int steps, int64_t parts) {
    const int64_t segs = ceil_div(cols, seg_cols(steps)), room = room_of(steps, rhs);
    Plan p{};
    p.steps = steps;
    if (parts > waves_of(steps)) parts = waves_of(steps);
    p.panels = ceil_div(segs, room);
    const int64_t panel_segs = ceil_div(segs, p.panels);
    for (;; --parts) {  // one part always fits
        p.part_segs = ceil_div(panel_segs, parts);
        p.parts = ceil_div(panel_segs, p.part_segs);
        if (p.parts * p.part_segs <= room) break;
    }
    // no more workgroups than there are eight items for (1000 x 3000: 8.6 us with one for every 8 rows, 9.1 for
    // every 16; 512 x 512: 8.4 for every 2, 7.6 for 8 or 16), and no more items per workgroup than LDS has room for
    int64_t grid = ceil_div(rows * p.parts, 8);
    if (grid > kUnits) grid = kUnits;
    if (grid > rows) grid = rows;
    const int64_t least = ceil_div(rows * p.parts, max_items(steps, rhs) - waves_of(steps));  // a workgroup has up to one row more than the average
    // a compute unit holds one workgroup: more than there are units in whole generations of about equal length
    // (131072 x 64 in 265 workgroups, 9 of them by themselves at the end, 90 us, in 512 51; 300000 x 100 in 605 135, in 768 109)
    if (grid < least) grid = least > kUnits ? ceil_div(least, kUnits) * kUnits : least;
    p.grid = grid;
    return p;
}

constexpr int64_t rows_per_unit(int64_t rows) { return ceil_div(rows, kUnits); }

// The length of a segment: the one with the least work per row, where a step (512 columns) counts 30 and a
// segment 40 beside its steps (the waves' vector instructions: 20 per step and 75 to 95 per segment, of which
// part hides).  Long segments have the least of it but fewer, longer ones per wave and more code, which
// shows at the start: 6 steps only where a compute unit has 50 of them (3000 x 3000: 8.7 us with 4 steps, 9.5
// with 6; 9216 x 9216 26 and 22), 8 where it has 100 (3000 x 20000: 18 us with 4 steps, 20 with 8; 8192 x
// 28672 53 and 50), or 70 of a sparse matrix, where the work counts and not the reading (20000 x 4000, a
// tenth kept, 22.4 with 4, 21.1 with 8; half kept 23.8 and 24.3), and for up to two right-hand sides (more do
// not fit the registers; nor do three and 6 steps).
//
// Parts: a row each for a wave from 12 rows per compute unit on; fewer are cut so that every wave has an
// item or two (600 x 36864: 22 us with rows whole, 14 to 15 with 11 parts; 2000 x 5000 9.3 whole, 8.9 with 3;
// from 24 rows on parts cost up to 2 us, as their starts have to be counted).
constexpr Plan make_plan(int64_t rows, int64_t cols, int64_t nnz, int rhs) {
    if (cols < 8) return plan_with(rows, cols, 1, 2, 1);
    const int64_t per = rows_per_unit(rows);
    const bool sparse = nnz < rows * cols / 4;
    int64_t best = -1;
    int steps = 2;
    for (int st = 2; st <= most_steps(rhs); st += 2) {
        const int64_t segs = ceil_div(cols, seg_cols(st)), cost = segs * (40 + 30 * st);
        if (segs * per < (st == 8 ? (sparse ? 70 : 100) : st == 6 ? 50 : 0)) continue;
        if (segs > room_of(st, rhs) && ceil_div(cols, seg_cols(4)) <= room_of(4, rhs)) continue;  // x fits, but not with these
        if (best < 0 || cost < best) {
            best = cost;
            steps = st;
        }
    }
    return plan_with(rows, cols, rhs, steps, per >= 12 ? 1 : (32 + per - 1) / per);
}

}  // namespace endor_gemv_plan

#endif  // ENDOR_GEMV_PLAN_H_
