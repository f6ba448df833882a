// The address arithmetic of the small-batch product's value loads (endor_gemm_units.h), replayed on
// the host for every load of every round of small products: each must lie inside `values` (or be the dummy), and together they must bring
// every unit that lies inside `values`.  Built and run by tests/test_gemm_units.py; not part of the
// library.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "endor_gemm_plan.h"
#include "endor_gemm_units.h"

using namespace endor_gemm_units;

static uint64_t state = 0x243F6A8885A308D3ull;
static uint64_t rnd() {
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}

static long replayed = 0;

// Rows row0 .. of one wave over rounds [k0, k1): cnt[row][round] values each, row_begin[row] of them before a row's first round.
// Returns a complaint, or null.
template <int kClass>
static const char *wave(uint64_t vbeg, uint64_t vend, const std::vector<std::vector<uint32_t>> &cnt,
                        const std::vector<uint64_t> &row_begin, int row0, int k0, int k1) {
    using F = Fetch<kClass>;
    const int rows = static_cast<int>(cnt.size());
    uint64_t first[kRows];
    for (int r = 0; r < kRows; ++r) {
        const int row = row0 + r < rows ? row0 + r : rows - 1;
        first[r] = vbeg + 2 * row_begin[row];
        for (int k = 0; k < k0; ++k) first[r] += 2 * cnt[row][k];
    }
    const uint64_t base = first[0] & ~uint64_t(15);
    const Limits L = limits_of(vbeg, vend, base);
    uint32_t off[kRows] = {};
    const int count = k1 - k0;
    for (int k = 0; k < count; ++k) {
        Slice s[kRows];
        for (int r = 0; r < kRows; ++r) {
            const uint32_t c = row0 + r < rows ? cnt[row0 + r][k0 + k] : 0u;
            const uint32_t start = static_cast<uint32_t>(first[r] - base) + off[r];
            s[r] = slice_of(L, start, c);
            // a row goes element by element only where it does not begin in a unit that can be read whole,
            // or reaches over the end: no other row's position matters
            const uint64_t unit = base + (start & ~15u), inside = unit >= vbeg && unit < vend ? (vend - unit) >> 4 : 0;
            if (L.ready && s[r].whole != (inside < s[r].units ? inside : s[r].units)) return "units that could be read whole are not";
            off[r] += 2 * c;
        }
        if (!L.ready) {  // every load reads the dummy, every unit comes element by element
            if (vend >= base + 48) return "an array of whole units is not read by units";
            continue;
        }
        bool got[kRows][64] = {};
        auto load = [&](int r, uint32_t unit) {
            const uint64_t p = base + unit_offset(s[r].info, unit);
            ++replayed;
            const uint64_t slice = (first[r] + off[r] - 2 * (row0 + r < rows ? cnt[row0 + r][k0 + k] : 0u)) & ~uint64_t(15);
            if (unit < s[r].whole && p != slice + 16 * unit) return "a unit was read from another place";
            if (unit < 64) got[r][unit] = true;
            return p >= vbeg && p + 16 <= vend ? nullptr : "a unit outside the values was read";
        };
        for (int i = 0; i < kFetchLoads<kClass>; ++i)
            for (uint32_t lane = 0; lane < 64; ++lane) {
                const uint32_t l = fetch_lane<kClass>(lane);
                if (const char *bad = load(fetch_row<kClass>(i, l / F::kUnits), l % F::kUnits)) return bad;
            }
        for (int r = 0; r < kRows; ++r) {
            if (F::kTail)
                if (const char *bad = load(r, F::kUnits)) return bad;
            for (uint32_t u = 0; u < s[r].whole; ++u)
                if (!got[r][u] && (F::kTail || u < F::kUnits)) return "a unit was not asked for";
            if (s[r].whole > s[r].units || s[r].units > 33) return "too many units";
            const uint64_t end = base + unit_offset(s[r].info, 63) + 16;
            if (s[r].whole && (end > vend || base + unit_offset(s[r].info, 0) < vbeg)) return "a late unit lies outside";
        }
    }
    return nullptr;
}

// The partition of one shape: every round done once, the parts of a shared row block at most kMaxParts,
// their slots of the scratch all different, and no workgroup that takes blocks of few rounds one after
// the other while there are more blocks than workgroups on the chip.
static const char *partition(int64_t rows, int64_t cols) {
    using namespace endor_gemm_plan;
    const Plan p = make_plan(rows, cols);
    const int64_t need = (cols + kSegCols - 1) / kSegCols;
    if (int64_t(p.blocks) != (rows + kBlockRows - 1) / kBlockRows || p.segs < need) return "rounds are missing";
    if (int64_t(p.rounds) != int64_t(p.blocks) * p.segs || p.per_wg == 0) return "the rounds do not add up";
    if (int64_t(p.wgs) != (int64_t(p.rounds) + p.per_wg - 1) / p.per_wg) return "the workgroups do not add up";
    if ((int64_t(p.wgs) * 64 * kGemmWaves) >> 32) return "too many threads for a launch";
    if (p.split != (p.per_wg % p.segs != 0)) return "a split that is not announced";
    if (int64_t(p.blocks) > kResident && need <= kNarrow && p.per_wg != p.segs && p.blocks <= kMaxGrid) return "blocks of few rounds are chained";
    if (p.segs > need + p.per_wg) return "rounds of nothing";
    for (int64_t block : {int64_t(0), int64_t(p.blocks) / 2, int64_t(p.blocks) - 1}) {
        const int64_t first = block * p.segs / p.per_wg, last = ((block + 1) * p.segs - 1) / p.per_wg;
        if (last - first > kMaxParts) return "too many parts";
        if (p.split && last + block >= int64_t(p.wgs) + p.blocks) return "a part without a slot";
        if (block + 1 < int64_t(p.blocks) && ((block + 1) * p.segs) / p.per_wg + block + 1 <= last + block) return "a slot used twice";
    }
    return nullptr;
}

// Matrices larger than can be walked here: wherever a row of a range that is not far may stand, its units
// are all read whole, and the offsets of any range fit 32 bits.
static const char *extremes() {
    using namespace endor_gemm_plan;
    const uint64_t vbeg = 0x7f0000000000ull, vend = vbeg + (uint64_t(1) << 35);
    const Limits L = limits_of(vbeg, vend, vbeg);
    for (uint64_t delta : {uint64_t(0), uint64_t(14), kSpan - 2, kSpan, uint64_t(1) << 33})
        for (uint64_t width : {uint64_t(256), kSpan / 4, kSpan / 2, kSpan / 2 + 1, kSpan, 2 * kSpan}) {
            if (is_far(vbeg + delta, vbeg, static_cast<uint32_t>(width))) {
                if (delta < kSpan && 2 * width <= kSpan) return "a short range counts as far";
                continue;
            }
            for (uint64_t off : {uint64_t(0), width, 2 * width - 512}) {
                const Slice s = slice_of(L, static_cast<uint32_t>(delta + off), 256);
                if (s.whole != s.units) return "units of a long range are not read whole";
                if (unit_offset(s.info, 0) != ((delta + off) & ~uint64_t(15))) return "a unit of a long range is read from another place";
            }
        }
    const Plan p = make_plan(1, (int64_t(1) << 34) - 1);
    if (2 * uint64_t(p.per_wg) * kSegCols >> 32) return "offsets inside a range do not fit";
    return nullptr;
}

int main() {
    if (const char *bad = extremes()) {
        std::printf("%s\n", bad);
        return 1;
    }
    for (int64_t rows : {int64_t(1), int64_t(64), int64_t(65), int64_t(2053), int64_t(28672), int64_t(32768), int64_t(32769), int64_t(36864), int64_t(131072), int64_t(524289), int64_t(2147483632)})
        for (int64_t cols : {int64_t(1), int64_t(100), int64_t(256), int64_t(257), int64_t(768), int64_t(1031), int64_t(3072), int64_t(3073), int64_t(8192), int64_t(28672), int64_t(1) << 24, (int64_t(1) << 34) - 1}) {
            if (cols > ((int64_t(1) << 34) - 1) / rows) continue;
            if (const char *bad = partition(rows, cols)) {
                std::printf("%ld x %ld: %s\n", (long)rows, (long)cols, bad);
                return 1;
            }
        }
    int cases = 0;
    for (int rows : {1, 2, 16, 17, 40})
        for (int rounds : {1, 2, 3, 9})
            for (int shape = 0; shape < 7; ++shape)
                for (uint32_t align = 0; align < 16; align += 2)
                    for (int cut = 0; cut < 3; ++cut) {
                        std::vector<std::vector<uint32_t>> cnt(rows, std::vector<uint32_t>(rounds));
                        std::vector<uint64_t> begin(rows);
                        uint64_t nnz = 0;
                        for (int r = 0; r < rows; ++r) {
                            begin[r] = nnz;
                            for (int k = 0; k < rounds; ++k) {
                                uint32_t c = static_cast<uint32_t>(rnd() % 257);      // 0: any density
                                if (shape == 1) c = 256;                              // everything kept
                                if (shape == 2) c = 0;                                // nothing
                                if (shape == 3) c = r == 0 ? 0 : 120 + rnd() % 20;    // an empty first row
                                if (shape == 4) c = r == 0 ? k % 2 : 90;              // a first row of single values
                                if (shape == 5) c = rnd() % 3 ? 0 : rnd() % 40;       // sparse
                                if (shape == 6) c = r % 3 ? 0 : 128;                  // empty rows
                                cnt[r][k] = c;
                                nnz += c;
                            }
                        }
                        // cut: the array ends with the last value, in the middle (nnz too small), or at its 3rd value
                        const uint64_t have = cut == 0 ? nnz : cut == 1 ? nnz / 2 : nnz < 3 ? nnz : 3;
                        const uint64_t vbeg = 0x7f0000000000ull + align, vend = vbeg + 2 * have;
                        for (int row0 = 0; row0 < rows; row0 += kRows)
                            for (int k0 = 0; k0 < rounds; k0 += 4) {
                                const int k1 = k0 + 4 < rounds ? k0 + 4 : rounds;
                                const char *bad[3] = {wave<0>(vbeg, vend, cnt, begin, row0, k0, k1),
                                                      wave<1>(vbeg, vend, cnt, begin, row0, k0, k1),
                                                      wave<2>(vbeg, vend, cnt, begin, row0, k0, k1)};
                                for (int c = 0; c < 3; ++c)
                                    if (bad[c]) {
                                        std::printf("rows %d rounds %d shape %d values at %u mod 16, cut %d, row %d, round %d, class %d: %s\n",
                                                    rows, rounds, shape, align, cut, row0, k0, c, bad[c]);
                                        return 1;
                                    }
                                ++cases;
                            }
                    }
    std::printf("ok %d waves, %ld loads\n", cases, replayed);
    return 0;
}
