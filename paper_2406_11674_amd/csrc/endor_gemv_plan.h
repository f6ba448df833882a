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

constexpr int64_t ceil_div(int64_t a, int64_t b) {
    // the divisions of 64 bits are most of what a plan takes
    const uint64_t n = static_cast<uint64_t>(a + b - 1), d = static_cast<uint64_t>(b);
    return (n | d) >> 32 ? static_cast<int64_t>(n / d) : static_cast<uint32_t>(n) / static_cast<uint32_t>(d);
}

constexpr int kMaxRhs = 4;

// Whether the vector form is the faster one for nb right-hand sides of the small-batch product.  The form on the
// matrix cores takes 16 rows of 256 columns in a round and starts slowly, this one takes a segment for every row
// however short the row is: so for narrow matrices it depends on the rows, up to `most` of them per compute unit for
// the widths below.
// Lines that do not begin at a bitmap word cost the matrix form more: a quarter more rows then.
// Measured, a tenth and 0.6 kept, us, the form on the matrix cores / this one:
//   64 columns  2000 rows, one vector, 7.3 / 6.9, two 7.3 / 7.3, 4099, three, 7.3 / 8.5, 16384, one, 7.3 / 11.7, four
//               7.4 / 14.7
//   512         9216, one 9 / 8.9, 12672, one, 8.9 / 11.0, four 9.2 / 13.7; 4099, three, 9.1 / 8.9
//   1024        16384, one, 11.8 to 13.7 / 12.1, 28672 14.9 / 17.3, 131072 48 / 61; 9216, four, 11.8 to 13 / 10.9
//   1300, 1536  20000, two, 22 to 25 / 19; 12672, three, 18 / 16, 28672, three, 22 to 26 / 29
//   2500        20000, three, 37 / 31, 28672 41 / 44 (a segment of 4 steps and one nearly empty)
//   wider       28672 x 8192 with one to three 75 / 50, 58, 70; 4099 x 5005, 0.3 kept, 18 / 12, 14, 15
// All of x has to fit LDS (two vectors of 8192 x 28672 74 / 82); four are left to the matrix cores from 2^25 elements on.
//  cols >= 8: shorter vectors are read element by element, which is there for one right-hand side only.
constexpr bool takes(int64_t rows, int64_t cols, int nb) {
    if (cols < 8 || nb > kMaxRhs || cols * nb > 48 * 1024) return false;
    if (nb == 4 && rows * cols > int64_t(1) << 25) return false;
    constexpr int kAny = 1 << 24;
    constexpr int most[6][kMaxRhs] = {{17, 8, 4, 0},     {36, 24, 18, 16},     {79, 44, 36, 36},
                                      {144, 79, 60, 40}, {kAny, kAny, 79, 79}, {kAny, kAny, 79, 50}};
    if (cols > 3072) return true;
    const int width = cols <= 256 ? 0 : cols <= 512 ? 1 : cols <= 1024 ? 2 : cols <= 1536 ? 3 : cols <= 2048 ? 4 : 5;
    const int64_t limit = most[width][nb - 1];
    return ceil_div(rows, kUnits) <= (cols % 64 ? limit + limit / 4 : limit);
}

struct Plan {
    int steps;          // of 512 columns per segment
    int64_t parts;      // items per row and panel
    int64_t part_segs;  // segments per item
    int64_t panels;     // of parts * part_segs segments
    int64_t grid;       // workgroups
};

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
    // (131072 x 64 in 265 workgroups, 9 of them by themselves at the end, 90 us, in 512 51; 300000 x 100 in 605 135, in
    // 768 109)
    if (grid < least) grid = least > kUnits ? ceil_div(least, kUnits) * kUnits : least;
    p.grid = grid;
    return p;
}

// The rows past a whole number for each workgroup go to workgroups at regular distances.  With the first ones having them,
// long runs of workgroups began at a common stride, and where that is an unlucky one all of them read the same channels of
// memory at a time: 9280 x 11648, 0.62 kept, 34.7 us, so 31.6 (9216 rows, 36 for each, 39); 9413 x 35233, 0.71 kept,
// 100.6, so 88.0.
//   more_share: ceil(2^32 * more / groups), more < groups; more_before: how many of the workgroups before have one more
constexpr uint32_t more_share(uint32_t more, uint32_t groups) {
    return static_cast<uint32_t>(((uint64_t(more) << 32) + groups - 1) / groups);
}
constexpr uint32_t more_before(uint32_t group, uint32_t share) { return static_cast<uint32_t>(uint64_t(group) * share >> 32); }

// What a plan costs, in units of some 7 ns.  A segment takes 90, and 30 a step with another 2 for each right-hand
// side, of a compute unit's vector units; 16 waves with the same number of segments use them fully, 12 are 3 %
// slower.  A workgroup ends with its longest wave, which alone runs at 3/8 of a wave's cost and waits 52 a
// segment for memory.  Longer segments are more code to fetch at the start (3 a step).  Parts of rows have their
// starts found, four items of a wave at a time (10; one vector's from the bitmap, 120 for 16384 columns), and
// a further panel of x is a start of its own (150).
//
// Fitted to every plan of 358 products (224 shapes, 1 x 600 to 36864 x 8192 and 1 x 2^22, 0.1 to 0.8 kept, one to
// four right-hand sides): the plan it picks is 0.75 % slower than the best on average.  The rule before, by the work of
// a row alone, kept rows whole from 12 per compute unit on and had no term for the longest wave: 2000 x 28672,
// a tenth kept, 21 us where 17 is possible (8 steps, rows whole), 12000 x 2500 16.5 / 11.9 (6 steps), 3000 x
// 3000 8.4 / 7.0, 4099 x 15000 with three 28 / 24 (2 parts: 17 rows are two to a wave of 16, 34 halves three),
// 3264 x 50000 97 / 43.
constexpr int64_t cost_of(int64_t rows, int rhs, const Plan &p) {
    const int64_t waves = waves_of(p.steps), items = ceil_div(rows, p.grid) * p.parts, segs = p.part_segs * p.panels;
    const int64_t segment = 90 + (30 + 2 * rhs) * p.steps;
    const int64_t work = items * segs * segment / 16, all = waves < 16 ? work + work / 32 : work;
    const int64_t longest = ceil_div(items, waves) * segs * (segment * 3 / 8 + 52);
    const int64_t start = 10 + (rhs == 1 ? 120 * p.parts * p.part_segs * seg_cols(p.steps) / 16384 : 0);
    return ceil_div(p.grid, kUnits) * (all > longest ? all : longest) + 3 * p.steps +
           (p.parts > 1 ? start * ceil_div(items, 4 * waves) * p.panels : 0) + 150 * (p.panels - 1);
}

constexpr Plan make_plan(int64_t rows, int64_t cols, int rhs) {
    if (cols < 8) return plan_with(rows, cols, 1, 2, 1);
    Plan best{};
    int64_t least = -1;
    // 2 steps are for short rows; three panels and more for the longest segments alone, which have the fewest of both (5 x
    // 1000000 145 us, with 4 steps 155, 40 x 500000 76, with 6 steps 85)
    const int longest = most_steps(rhs);
    const bool panels = ceil_div(cols, seg_cols(longest)) > 2 * room_of(longest, rhs);
    for (int steps = panels ? longest : cols > 4096 ? 4 : 2; steps <= longest; steps += 2) {
        if (least >= 0 && seg_cols(steps - 2) >= cols) break;  // a shorter segment already holds the row
        // more than 32 rows per compute unit are never cut (9216 x 9216 in 3 parts 22, whole 19; a plan costs the
        // caller 0.05 us, 512 x 512, to 0.8, 600 x 36864)
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
