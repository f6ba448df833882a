// Which form a column-subset decompression takes, and with what: plain host arithmetic, apart from the kernels so that it
// can be checked on its own.
//
// Two kernels: workgroups that stay, a row after the other (endor_cols_stream.h), and a workgroup for every row, whose values
// are gathered from memory or staged in LDS.
#ifndef ENDOR_COLS_PLAN_H_
#define ENDOR_COLS_PLAN_H_

#include <cstddef>
#include <cstdint>

namespace endor_cols_plan {

constexpr int64_t kMB = int64_t(1) << 20;
constexpr int kBlock = 256;           // threads of a workgroup that has one row
constexpr uint32_t kLineBytes = 128;  // of the second-level cache
constexpr size_t kMaxColsLds = 40 * 1024, kMinColsStage = 6 * 1024, kLdsPerUnit = 160 * 1024;

// ---------------------------------------------------------------- a workgroup for every row: what it stages

// LDS for a row's bitmap, and the 1 bits before each piece of it.
constexpr size_t bitmap_lds(int64_t cols) { return static_cast<size_t>((cols + 63) / 64) * 4 * sizeof(uint32_t); }
// And for its values: room for an eighth more than a row has on average, and a spare unit.
constexpr size_t stage_bytes(int elem_bytes, int64_t row_values) {
    return (static_cast<size_t>(row_values) * 9 / 8 * elem_bytes + 256 + 15) & ~size_t(15);
}

constexpr bool rows_staged(int elem_bytes, int64_t rows, int64_t cols, int64_t nnz, int64_t nsel) {
    const size_t lds = bitmap_lds(cols), stage = stage_bytes(elem_bytes, nnz / rows);
    // Staging pays when most 64-byte lines of a row's values are wanted anyway (a sixteenth of the
    // columns; the gather then costs a cache access per value, staging one per 64 bytes), the row is
    // long enough for that to matter and short enough for four workgroups per compute unit.  Measured,
    // gather against staged: a tenth of 8192 x 28672 65 / 63 us, three tenths 135 / 114, 8-bit 50 / 41, one
    // in five kept 52 / 39, three tenths of 36864 x 9216 198 / 138; but 8192 x 28672 with four in five kept
    // (52 KB a row) 89 / 105, a fifth of 5003 x 3171 (4 KB) 11 / 13, a tenth of 30000 x 700 39 / 49.
    const bool rows_fit = nsel >= cols / 16 && lds + stage <= kMaxColsLds;
    // And there has to be a lot to read or to answer: otherwise a workgroup's wait for its row shows, while
    // the gather finds values that the memory-side cache holds.  A tenth of 2048 x 16384 9 / 12 us, three
    // tenths 17 / 19, half 25 / 25; 3000 x 36864, 8-bit (55 MB), a tenth 21 / 25, a fifth 43 / 35; 4096 x
    // 28672, one in five kept (47 MB), 0.07 of the columns 17 / 19, 0.15 37 / 29; 0.07 of 7200 x 12000,
    // 8-bit, 16 / 18; of 9216 x 9216, two in five kept (68 MB) 20 / 21, half kept (85 MB) 24 / 22.
    const int64_t asked = rows * nsel;
    const bool much = nnz * elem_bytes >= 72 * kMB || asked >= 14000000 || (rows >= 28 * 256 && asked >= 8000000);
    // Or all rows on the chip at once, none of them long: a fifth of 1024 x 16384, 8-bit, 9.5 / 8.3 us, half
    // 17 / 13; fp16, four in five kept (26 KB a row), a fifth 9.7 / 11.2.
    const bool at_once = rows <= 2048 && static_cast<size_t>(rows) * (lds + stage) <= 256 * kLdsPerUnit && nsel >= cols / 5 &&
                         nnz * elem_bytes <= rows * 20480;
    // A shorter row only where every thread of its workgroup has six queries or more, and there are 8 million hits in
    // all: otherwise the wait for the row outweighs the gather's accesses.  Fewer where `values` is larger than the
    // memory-side cache keeps.  By columns asked of a row, gather / staged: 17233 x 2473, 0.66 kept, 1162 35.4 / 44.3 us,
    // 20000 x 1500, 0.8 kept, 750 33 / 37, 9216 x 9216, 8-bit, 1474 (6.8 million) 22 / 25; 18432 x 4608, half kept, 1843 64 /
    // 47, 18923 x 15575, 8-bit, 0.14 kept, 4828 133 / 87, 28672 x 8192, 8-bit, 2457 110 / 80; 95868 x 3763, 8-bit (238 MB), 940
    // 194 / 168.  Over 285 calls (rows of 250 bytes to 6 KB) the choice is 0.6 % slower than the better form on average; by
    // hits of a row alone, 600 or 300, it was 1.9 %.
    const double hits = static_cast<double>(nsel) * static_cast<double>(nnz) / static_cast<double>(cols);
    const bool most_asked = hits >= 8e6 && (nsel >= 6 * kBlock || (nnz * elem_bytes >= 128 * kMB && hits >= rows * 300.0));
    const bool long_rows = stage >= kMinColsStage && (much || at_once);
    return rows > 1 && rows_fit && (long_rows || (stage < kMinColsStage && most_asked));
}

// ---------------------------------------------------------------- workgroups that stay

constexpr int kMaxStreamQueries = 12;  // of a thread; 16 take more registers than there are

// A workgroup of kThreads and the LDS it may take for 1024 / kThreads of them to share a compute unit.
template <int kThreads>
struct StreamShape {
    static constexpr int kWaves = kThreads / 64;
    static constexpr uint32_t kGroups = 256 * (1024 / kThreads);
    static constexpr uint32_t kUnits = 15 * kThreads / 4;  // 16-byte units of a row's values: 30 KB for 512 threads, 15 for 256
    static constexpr int kRounds = (kUnits + kThreads - 1) / kThreads;
    static constexpr int64_t kMaxCols = 64 * kThreads;     // a bitmap word a thread
};

template <int kThreads>
constexpr bool fits_stream(int64_t row_bytes, int64_t cols, int64_t nsel) {
    typedef StreamShape<kThreads> Sh;  // (512: three standard deviations of the longest rows)
    return row_bytes + 512 <= 16 * int64_t(Sh::kUnits) && cols <= Sh::kMaxCols && nsel <= kThreads * kMaxStreamQueries;
}

// Threads of such workgroups, 0 where a workgroup per row is the faster form.
//
// A step takes 0.9 us or more however little there is in it, and a workgroup two steps more than it has rows, the last of which
// may be of a few workgroups: of groups * steps places, how many have a row?  The other kernel is slow where it stages rows,
// where it gathers what the memory-side cache does not keep, and where a thread takes a second round of queries (1537 columns).
// So, a workgroup per row / staying, us:
//   256 threads, rows that would be staged: five queries a thread, 9782 x 8261, 1239 columns, 29 / 25, 12538 x 3715, 1523, 36 / 28
//     gathered: the same from 105 MB of values and output on (8-bit 70), 27893 x 4938, 1264 columns, 72 / 54, 17637 x 4565, 1233,
//       45 / 37, 8-bit 23844 x 3531, 1395, 60 / 41, but 13120 x 5120, 1280 (86 MB), 25 / 30, 9088 x 2624, 1278 (49 MB), 18.4 / 22.1;
//       six queries where four in five places have a row, 14663 x 3546, 1624, 38 / 32; else a second round of the other
//       kernel, 6375 x 3321, 1577, 19.3 / 17.6, 8-bit 6469 x 12229, 1810, 20.0 / 16.9, 5718 x 11811, 1465, 16.4 / 18.8, and
//       not with nine queries, which take twelve, 5824 x 11712, 2249, 22.0 / 25.4, 6016 x 6656, 2110, 20.2 / 22.5
//   512 threads, rows of 20 KB and more: three queries a thread, 8192 x 28672, a tenth 63 / 55, a fifth 93 / 71; of 12 KB: four,
//       16384 x 16384, 0.07 of the columns 59 / 65, a tenth 62 / 66, 0.3 of them 100 / 96, 6656 x 12224, 978, 22.0 / 27.2;
//       shorter ones: five
// Not where few columns are asked (less than a sixteenth: the gather reads less), nor for sparse 16-bit rows, of which the
// cache serves the gather (7232 x 8896, a tenth kept, 23 / 26), nor for 16-bit outputs of 96 MB and more of shorter rows or few
// queries, which the other kernel streams past the cache in whole lines (31040 x 9920, 0.3 kept, 115 / 122, 21632 x 13248, 2782
// columns, 106 / 116).
//
// Fitted to 1499 calls of both kernels (5500 to 36864 rows, 800 to 32768 columns, a sixteenth to half of them, a tenth to
// nine tenths kept, both widths, rows alike and not): taken for 429 of them, 1.15 times as fast on average, at worst 0.95;
// of 899 others for 259, 1.15 times, at worst 0.95.  Rows that are not alike do not all fit LDS near its limits: 447 calls of such
// rows (deviations of 3 to 10 of 100 columns) 1.15 times, but of 14.5 KB and more with 256 threads 1.01.  (Without the steps in it the rule lost 5 % and more, up to a fifth, on 21
// of the 470 that it took.)
constexpr int stream_threads(int elem_bytes, int64_t rows, int64_t cols, int64_t nnz, int64_t nsel) {
    const int64_t row_bytes = nnz / rows * elem_bytes;
    if (rows < 5500 || nsel < cols / 16) return 0;
    const bool narrow = fits_stream<256>(row_bytes, cols, nsel);
    if (!narrow && !fits_stream<512>(row_bytes, cols, nsel)) return 0;
    const int threads = narrow ? 256 : 512;
    const int64_t groups = narrow ? StreamShape<256>::kGroups : StreamShape<512>::kGroups;
    const int64_t places = groups * ((rows + groups - 1) / groups + 2);
    const int64_t half_queries = 2 * nsel / threads;
    if (elem_bytes == 2 && rows * nsel * elem_bytes >= 96 * kMB && (row_bytes < 16000 || half_queries < 15)) return 0;
    if (!narrow && row_bytes >= 12000) return half_queries >= (row_bytes >= 20000 ? 5 : 8) ? threads : 0;
    if (elem_bytes == 2 && nnz < rows * cols / 5) return 0;
    int least = rows >= 9000 && row_bytes >= 2500 ? 9 : 11;
    if (narrow && !rows_staged(elem_bytes, rows, cols, nnz, nsel)) {
        const int64_t share = rows * 100 / places, moved = nnz * elem_bytes + rows * nsel * elem_bytes;
        if (moved < (elem_bytes == 2 ? 105 : 70) * kMB) least = share >= 80 ? 11 : 12;
        if (share < 79 && elem_bytes == 2 && nsel > 8 * threads && half_queries < 19) return 0;
    }
    return half_queries >= least ? threads : 0;
}

// ---------------------------------------------------------------- plans

// Plain; past the memory-side cache; so, and each wave's part of a row in whole lines, where rows of the output do
// not begin at one.  A streamed store of parts of lines costs about a third more than one of whole ones: 8192 x
// 28672, four in five kept, 0.35 of the columns (rows of 20070 bytes) plain 157 us, streamed 179, in whole lines 153.
enum class Store { kPlain, kStreamed, kLines };

// Queries per thread and round.  A staged row takes 4 (6 against 4: 2048 x 16384, 8-bit, half, 20.6 / 19.3 us, 36864 x
// 9216, three tenths, 136 / 128; 12 cost it the occupancy, 28672 x 8192, three tenths, 111 / 94).  A gathered row takes 6
// (28672 x 8192, one in five kept, three tenths 134 / 125 before its stores were streamed), but 4 where
// the last of several rounds would be mostly empty with 6 (2048 x 16384, a tenth, 9.9 / 9.2).  3 for few queries
// (36864 x 2000, a tenth, 6 / 4 / 3: 47 / 47 / 44).
constexpr int cols_round(bool staged, int64_t nsel) {
    const int64_t rounds6 = (nsel + 6 * kBlock - 1) / (6 * kBlock), rounds4 = (nsel + 4 * kBlock - 1) / (4 * kBlock);
    return nsel <= 3 * kBlock ? 3 : staged || (rounds6 == rounds4 && rounds6 > 1) ? 4 : 6;
}

struct Plan {
    int threads;           // of workgroups that stay; 0: a workgroup for every row
    int round;             // queries of a thread; of a round, where a workgroup has one row
    bool staged;           // the row's values in LDS
    uint32_t stage_units;  // 16-byte units that the staging area holds
    size_t lds;
    Store store;
};

// `out`: the output's address.
constexpr Plan make_plan(int elem_bytes, int64_t rows, int64_t cols, int64_t nnz, int64_t nsel, uint64_t out) {
    Plan p{};
    p.threads = stream_threads(elem_bytes, rows, cols, nnz, nsel);
    if (p.threads != 0) {
        const int64_t queries = (nsel + p.threads - 1) / p.threads;
        p.round = queries <= 4 && p.threads == 512 ? 4 : queries <= 6 ? 6 : queries <= 8 ? 8 : kMaxStreamQueries;
        return p;
    }
    const size_t lds = bitmap_lds(cols), stage = stage_bytes(elem_bytes, nnz / rows);
    const bool staged = rows_staged(elem_bytes, rows, cols, nnz, nsel);
    p.staged = staged;
    p.stage_units = static_cast<uint32_t>(stage / 16);
    p.lds = lds + (staged ? stage : 0);
    // Streamed stores where values are gathered: the output then leaves the lines of `values`, which several
    // queries of a row share, in the memory-side cache.  28672 x 8192, one in five kept, a tenth of the columns
    // 57 / 44 us, three tenths 125 / 85, 36864 x 2000 three tenths 68 / 57.  Where rows are staged every line is
    // read once, and only an output that would fill that cache is streamed: 8192 x 28672, three tenths (141
    // MB) 113 / 101, half (235 MB) 152 / 134, but 4096 x 28672, one in five kept, three tenths (70 MB) 42.6 / 45.5.
    // Very small outputs and 8-bit ones are not: 1024 x 16384, a tenth (3 MB), 6.5 / 6.8; 8-bit +-2 % throughout.
    const int64_t out_bytes = rows * nsel * elem_bytes;
    const int round = cols_round(staged, nsel);
    p.round = round;
    if (elem_bytes == 2 && out_bytes >= (staged ? 96 * kMB : 8 * kMB)) {
        p.store = Store::kStreamed;
        if ((out | static_cast<uint64_t>(2 * nsel)) % kLineBytes) {
            // Rows that begin inside a line.  Whole lines, where the queries then take no round more, or one more of
            // at least four (28672 x 8192, four in five kept, 3055 columns 128 / 118, 17274 x 13952, half, 3069 82 / 77; but 36864 x
            // 9216, one in five, 2027 91 / 102).  A gathered row has to be long for it (28672 x 8192, one in five kept,
            // 1802 columns 79 / 80 us in lines; 9216 x 9216 2027 28.1 / 28.9, 3225 equal) and its output large (3200 x 8704,
            // 0.47 (26 MB) 19.1 / 19.8, 1000 x 20000 to 30000 15 to 19, 2 to 3 % slower; 3000 x 36864, 0.22 (49 MB) 57 / 54).
            const int64_t taken = (nsel + round * kBlock - 1) / (round * kBlock) * (round * kBlock);
            const bool room = nsel + int64_t(kLineBytes) / 2 <= taken;
            if (staged ? room || nsel > 2048 : room && nsel >= 3072 && out_bytes >= 32 * kMB) p.store = Store::kLines;
        }
    }
    return p;
}

}  // namespace endor_cols_plan

#endif  // ENDOR_COLS_PLAN_H_
