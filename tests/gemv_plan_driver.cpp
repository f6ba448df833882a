// How the vector products share out their work (endor_gemv_plan.h), checked on the host over shapes of every
// kind.  Built and run by tests/test_gemv_plan.py; not part of the library.
#include <cstdint>
#include <cstdio>

#include "endor_gemv_plan.h"

using namespace endor_gemv_plan;

static uint64_t state = 0x243F6A8885A308D3ull;
static uint64_t rnd() {
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}
static int64_t size(int bits) {  // spread over its logarithm
    const int b = static_cast<int>(rnd() % (bits + 1));
    return 1 + static_cast<int64_t>(rnd() % (uint64_t(1) << b));
}

// What must hold of any plan; a complaint, or null.
static const char *check(int64_t rows, int64_t cols, int rhs, const Plan &p) {
    const int64_t seg = seg_cols(p.steps), segs = ceil_div(cols, seg), slots = p.panels * p.parts * p.part_segs;
    if (p.steps < 2 || p.steps > most_steps(rhs) || (p.steps & 1)) return "no such segment";
    if (p.parts < 1 || p.part_segs < 1 || p.parts > waves_of(p.steps)) return "parts";
    if (lds_beside_x(p.steps, rhs) + size_t(p.parts * p.part_segs * seg) * 2 * rhs > kLds) return "more LDS than there is";
    if (slots < segs) return "columns left out";
    if (p.grid < 1 || p.grid > rows || (rows < 2000000000 && p.grid * 64 * waves_of(p.steps) >= int64_t(1) << 32)) return "grid";
    if (ceil_div(rows, p.grid) * p.parts > max_items(p.steps, rhs)) return "more items than a workgroup has room for";
    if (p.grid > kUnits && p.grid % kUnits) return "a last generation of a few workgroups";
    // waves walk every slot
    if (slots - segs >= p.panels * p.parts + p.panels) return "a panel of segments without columns";
    return nullptr;
}

// Every row has one workgroup, none more than its share rounded up, and the larger ones lie at regular distances: a run of
// workgroups of one size is no longer than it has to be.
static const char *check_rows(int64_t rows, uint32_t groups) {
    const uint32_t each = static_cast<uint32_t>(rows / groups), more = static_cast<uint32_t>(rows % groups), share = more_share(more, groups);
    if (more_before(0, share) != 0 || more_before(groups, share) != more) return "rows left over";
    for (int k = 0; k < 64; ++k) {
        const uint32_t g = static_cast<uint32_t>(rnd() % groups), a = more_before(g, share), b = more_before(g + 1, share);
        if (b < a || b - a > 1 || each + (b - a) > ceil_div(rows, groups)) return "a workgroup's rows";
        const int64_t even = static_cast<int64_t>(static_cast<unsigned __int128>(rows) * g / groups) - int64_t(each) * g;
        if (a < even || a > even + 1) return "rows bunched";
    }
    return nullptr;
}

int main() {
    for (int rep = 0; rep < 100000; ++rep) {
        const int64_t rows = size(rep % 20 ? 18 : 31);
        const uint32_t groups = static_cast<uint32_t>(1 + rnd() % uint64_t(rep % 2 && rows > 256 ? 256 : rows));
        if (const char *bad = check_rows(rows, groups)) {
            std::printf("%s: %lld rows, %u workgroups\n", bad, (long long)rows, groups);
            return 1;
        }
    }
    for (int rep = 0; rep < 400000; ++rep) {
        const int rhs = 1 + static_cast<int>(rnd() % 4);
        int64_t rows = size(rep % 50 ? 18 : 31), cols = size(rep % 50 ? 18 : 33);
        if (rows > 0x7fffffff || cols > ((int64_t(1) << 34) - 1) / rows) continue;  // refused
        if (rhs > 1 && cols < 8) continue;
        Plan p = make_plan(rows, cols, rhs);
        const char *bad = check(rows, cols, rhs, p);
        // a product that is taken from the matrix cores has all of x in LDS
        if (!bad && rhs > 1 && takes(rows, cols, rhs) && p.panels != 1) bad = "x in panels";
        if (!bad && cols >= 8)
            for (int st = 2; st <= most_steps(rhs) && !bad; st += 2) {
                p = plan_with(rows, cols, rhs, st, 1 + rnd() % 16);
                bad = check(rows, cols, rhs, p);
            }
        if (bad) {
            std::printf("%s: %lld x %lld, %d right-hand sides: steps %d parts %lld x %lld, %lld panels, %lld workgroups\n", bad,
                        (long long)rows, (long long)cols, rhs, p.steps, (long long)p.parts, (long long)p.part_segs,
                        (long long)p.panels, (long long)p.grid);
            return 1;
        }
    }
    // products with few right-hand sides: narrow ones that the matrix cores do in half to four fifths of the time, and others
    const int64_t kNot[][3] = {{16384, 256, 1}, {16384, 64, 2},    {16384, 256, 4}, {9216, 64, 2},   {9216, 8, 4},
                               {4099, 64, 4},   {131072, 1024, 1}, {16384, 1024, 4}, {131072, 256, 1}};
    for (const auto &s : kNot)
        if (takes(s[0], s[1], static_cast<int>(s[2]))) {
            std::printf("%lld x %lld with %lld taken from the matrix cores\n", (long long)s[0], (long long)s[1], (long long)s[2]);
            return 1;
        }
    const int64_t kYes[][3] = {{1, 600, 4},     {2000, 64, 2},    {4099, 5005, 3},  {12000, 600, 1},
                               {4096, 4096, 4}, {28672, 8192, 3}, {4400, 24570, 2}};
    for (const auto &s : kYes)
        if (!takes(s[0], s[1], static_cast<int>(s[2]))) {
            std::printf("%lld x %lld with %lld left to the matrix cores\n", (long long)s[0], (long long)s[1], (long long)s[2]);
            return 1;
        }
    std::printf("ok\n");
    return 0;
}
