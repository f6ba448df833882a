// Which 16-byte units of a tile's slice of `values` lie inside the array as a whole: plain address arithmetic, apart
// from the kernels so that it can be replayed on the host.
//
// The slice is `units` units from a16, the 16-byte boundary at or below its first value.  Units [first, last) are read
// as one; the others reach over an end of the array [vbeg, vend), or lie outside it behind a table that is not the
// bitmap's, and are put together from their elements.
#ifndef ENDOR_VALUE_UNITS_H_
#define ENDOR_VALUE_UNITS_H_

#include <cstdint>

namespace endor_value_units {

constexpr bool all_inside(uint64_t a16, uint32_t units, uint64_t vbeg, uint64_t vend) {
    return a16 >= vbeg && a16 + 16 * uint64_t(units) <= vend;
}
constexpr uint32_t first_whole(uint64_t a16, uint32_t units, uint64_t vbeg) {
    const uint64_t skip = a16 < vbeg ? (vbeg - a16 + 15) >> 4 : 0;
    return skip < units ? static_cast<uint32_t>(skip) : units;
}
constexpr uint32_t end_of_whole(uint64_t a16, uint32_t units, uint64_t vbeg, uint64_t vend) {
    const uint64_t room = vend > a16 ? (vend - a16) >> 4 : 0;
    const uint32_t last = room < units ? static_cast<uint32_t>(room) : units, first = first_whole(a16, units, vbeg);
    return last > first ? last : first;
}

}  // namespace endor_value_units

#endif  // ENDOR_VALUE_UNITS_H_
