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

constexpr int64_t ceil_div(int64_t a, int64_t b) {
    // the divisions of 64 bits are most of what a plan takes
    const uint64_t n = static_cast<uint64_t>(a + b - 1), d = static_cast<uint64_t>(b);
    return (n | d) >> 32 ? static_cast<int64_t>(n / d) : static_cast<uint32_t>(n) / static_cast<uint32_t>(d);
}

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

// What a plan costs: about 40 per percent of a microsecond.  A segment takes 90, and 30 a step with another 2 for
// each right-hand side, of a compute unit's vector units; 16 waves with the same number of segments use
// them fully, 12 are 3 % slower.  A workgroup ends with its longest wave, which alone runs at 3/8 of a wave's
// cost and waits 45 a segment for memory.  Longer segments are more code to fetch at the start (3 a step), parts
// of rows have their starts counted (15 for every four items of a wave), and a further panel of x is a start of
// its own (1000).
//
// Fitted to every plan of 310 products (200 shapes, 1 x 600 to 36864 x 8192, 0.1 to 0.8 kept, one to four
// right-hand sides): the plan it picks is 0.6 % slower than the best on average.  The rule before, by the work of
// a row alone, kept rows whole from 12 per compute unit on and had no term for the longest wave: 2000 x 28672,
// a tenth kept, 21 us where 17 is possible (8 steps, rows whole), 12000 x 2500 16.5 / 11.9 (6 steps), 3000 x
// 3000 8.4 / 7.0, 4099 x 15000 with three 28 / 24 (2 parts: 17 rows are two to a wave of 16, 34 halves three).
constexpr int64_t cost_of(int64_t rows, int rhs, const Plan &p) {
    const int64_t waves = waves_of(p.steps), items = ceil_div(rows, p.grid) * p.parts, segs = p.part_segs * p.panels;
    const int64_t segment = 90 + (30 + 2 * rhs) * p.steps;
    const int64_t work = items * segs * segment / 16, all = waves < 16 ? work + work / 32 : work;
    const int64_t longest = ceil_div(items, waves) * segs * (segment * 3 / 8 + 45);
    return ceil_div(p.grid, kUnits) * (all > longest ? all : longest) + 3 * p.steps +
           (p.parts > 1 ? 15 * ceil_div(items, 4 * waves) * p.panels : 0) + 1000 * (p.panels - 1);
}

constexpr Plan make_plan(int64_t rows, int64_t cols, int rhs) {
    if (cols < 8) return plan_with(rows, cols, 1, 2, 1);
    Plan best{};
    int64_t least = -1;
    for (int steps = cols > 4096 ? 4 : 2; steps <= most_steps(rhs); steps += 2) {  // 2 steps are for short rows
        // more than 32 rows per compute unit are never cut (9216 x 9216 in 3 parts 22, whole 19; a plan costs the
        // caller 0.1 to 0.3 us)
        const int64_t most = rows > 32 * kUnits ? 1 : waves_of(steps), segs = ceil_div(cols, seg_cols(steps));
        for (int64_t parts = 1, before = 0; parts <= most && parts <= segs; ++parts) {
            const Plan p = plan_with(rows, cols, rhs, steps, parts);
            if (p.parts == before) continue;
            before = p.parts;
            const int64_t cost = cost_of(rows, rhs, p);
            if (least < 0 || cost < least) {
                least = cost;
                best = p;
            }
        }
    }
    return best;
}

}  // namespace endor_gemv_plan

#endif  // ENDOR_GEMV_PLAN_H_
