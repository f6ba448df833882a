// Which 16-byte units of `values` a wave of the small-batch product reads: plain address arithmetic,
// apart from the kernel so that it can be replayed on the host.
//
// A wave walks 16 rows of W, 256 columns (a round) at a time.  A row's slice of a round is the units
// that hold its values.  Units are read whole, so only those that lie inside `values` as a whole are
// read here; the others (at the array's ends) are put together element by element.
#ifndef ENDOR_GEMM_UNITS_H_
#define ENDOR_GEMM_UNITS_H_

#include <cstdint>

namespace endor_gemm_units {

constexpr int kRows = 16;  // rows of W per wave: the M of the matrix instruction

// How many units of a row's slice are asked for a round ahead, and how: kRowsPer rows per load
// instruction (neighbouring lanes take a row's neighbouring units, so an instruction covers whole
// cache lines and no line is asked for twice).  kTail: one more load brings unit kUnits of every row.
// A row with more units gets the rest when its round is staged.
template <int kClass>
struct Fetch;
template <>
struct Fetch<0> {  // 97 values per row and round
    enum { kUnits = 13, kRowsPer = 4, kTail = 0 };
};
template <>
struct Fetch<1> {  // 161 values
    enum { kUnits = 21, kRowsPer = 3, kTail = 0 };
};
template <>
struct Fetch<2> {  // all 256
    enum { kUnits = 32, kRowsPer = 2, kTail = 1 };
};

template <int kClass>
constexpr uint32_t fetch_lane(uint32_t lane) {  // lanes without a unit of their own repeat the last one
    return lane < Fetch<kClass>::kRowsPer * Fetch<kClass>::kUnits ? lane : Fetch<kClass>::kRowsPer * Fetch<kClass>::kUnits - 1;
}

template <int kClass>
constexpr int kFetchLoads = (kRows + Fetch<kClass>::kRowsPer - 1) / Fetch<kClass>::kRowsPer;

template <int kClass>
constexpr uint32_t fetch_row(int load, uint32_t row_of_load) {
    return (load + 1) * Fetch<kClass>::kRowsPer <= kRows || load * Fetch<kClass>::kRowsPer + row_of_load < kRows
               ? load * Fetch<kClass>::kRowsPer + row_of_load
               : kRows - 1;
}

constexpr uint64_t kSpan = uint64_t(1) << 28;  // bytes

// A row whose values of a range of `width` columns may lie too far from the wave's base (the unit of its
// first row's first value) for offsets of 32 bits: rows of more than some ten million columns, whose 16
// starts are far apart, and ranges of more than 2^27 columns.  Others stay below base + 2 * kSpan.
constexpr bool is_far(uint64_t first, uint64_t base, uint32_t width) {
    return first - base >= kSpan || 2 * uint64_t(width) > kSpan;
}

// What may be read around `base`, a 16-byte boundary: the unit of the first value of the wave's first
// row.  An array that is not 16-byte aligned begins inside that unit, which then is not read.
struct Limits {
    uint32_t lo, hi;  // offsets from base of the array's first byte (0 if it lies before base) and of its end
    uint32_t idle;    // the first unit that may be read: for a lane that has nothing to read
    bool ready;       // false: no unit can be read around this base
};

constexpr Limits limits_of(uint64_t vbeg, uint64_t vend, uint64_t base) {
    Limits L{};
    L.lo = base >= vbeg ? 0u : static_cast<uint32_t>(vbeg - base);  // a table that lies may put the base anywhere
    L.hi = vend <= base ? 0u : vend - base < 3 * kSpan ? static_cast<uint32_t>(vend - base) : static_cast<uint32_t>(3 * kSpan);
    if (base < vbeg && vbeg - base > 15) L.hi = 0;
    L.idle = L.lo ? 1u : 0u;
    L.ready = L.hi >= 16 * (L.idle + 1);
    return L;
}

// A row's slice of a round: cnt values from offset `start`.
struct Slice {
    uint32_t units;  // those that hold a value
    uint32_t whole;  // those that are read whole: from the first one up to the end of `values`; none in the round
                     // in which the row begins before the array's first whole unit
    uint32_t info;   // first unit << 6 | the last one to read, counted from it
};

constexpr Slice slice_of(const Limits &L, uint32_t start, uint32_t cnt) {
    Slice s{};
    const uint32_t shift = start & 15u, first = start & ~15u;
    s.units = cnt ? (shift + 2 * cnt + 15) >> 4 : 0u;
    const uint32_t room = first >= L.lo && L.hi > first ? (L.hi - first) >> 4 : 0u;  // whole units from here to the end of `values`
    s.whole = s.units < room ? s.units : room;
    s.info = s.whole ? (first << 2) | (s.whole - 1) : L.idle << 6;
    return s;
}

// Offset of the unit that a lane reads for unit `unit` of a slice: a lane without one of its own
// reads the slice's last one again.
constexpr uint32_t unit_offset(uint32_t info, uint32_t unit) {
    const uint32_t last = info & 63u;
    return ((info >> 6) + (unit < last ? unit : last)) << 4;
}

}  // namespace endor_gemm_units

#endif  // ENDOR_GEMM_UNITS_H_
