// Which bytes of `values` the vector products read for a segment: plain arithmetic, apart from the kernel
// so that it can be replayed on the host.
//
// The kernel reads 16 bytes for every bitmap byte, whatever number of values the byte takes.  Where all of a
// segment's windows lie inside the array (kWhole) they are read from the dword boundary below their first
// value.  At an end of the array (kEdge) a window is read from its first value itself, or from the last
// place from which 16 bytes can be read, and shifted down: one trip to memory like any other segment.  The
// last segment of every product is one of these.  Read element by element it took a trip per step, one
// after the other, when everything else had ended: 1 x 2000 6.5 us, now 5.0, 2000 x 2000 6.9 / 5.6, 2000 x
// 5000 8.3 / 7.3, 4096 x 4096 9.1 / 7.7.
// An array that holds no window at all, and offsets that point out of it, go element by element (kElements).
#ifndef ENDOR_GEMV_WINDOWS_H_
#define ENDOR_GEMV_WINDOWS_H_

#include <cstdint>

namespace endor_gemv_windows {

constexpr uint32_t kWhole = 0, kEdge = 1, kElements = 2;

// Positions are counted in values from `base`, 13 bits of an entry; a byte's entry is
//     shift (values to drop from the window's front) << 28 | position << 9 | the byte
constexpr uint32_t kMaxPosition = 0x1fff;

struct Windows {
    uint64_t base;   // address that positions count from
    uint32_t first;  // position of the segment's first value
    uint32_t limit;  // the last position a window can be read from
    uint32_t how;
    // an entry's window begins at base + ((entry >> 8) & offset_mask)
    uint32_t offset_mask;
};

// Segment of `cnt` (<= 4096) values at address vseg of the array [vbeg, vend): whether all of its windows lie inside.
constexpr bool is_whole(uint64_t vbeg, uint64_t vend, uint64_t vseg, uint32_t cnt) {
    return vseg <= vend && (vseg & ~uint64_t(3)) >= vbeg && vseg + 2 * uint64_t(cnt) + 20 <= vend;
}

constexpr Windows whole_windows(uint64_t vseg) {
    return {vseg & ~uint64_t(3), static_cast<uint32_t>(vseg >> 1) & 1u, kMaxPosition, kWhole, 2 * kMaxPosition & ~3u};
}

// where they do not
constexpr Windows end_windows(uint64_t vbeg, uint64_t vend, uint64_t vseg) {
    if (vseg < vbeg || vseg > vend || vend - vbeg < 16)
        return {vseg & ~uint64_t(3), static_cast<uint32_t>(vseg >> 1) & 1u, kMaxPosition, kElements, 0u};
    const uint64_t base = vseg - vbeg >= 16 ? vseg - 16 : vbeg, room = (vend - 16 - base) / 2;
    return {base, static_cast<uint32_t>(vseg - base) / 2, room < kMaxPosition ? static_cast<uint32_t>(room) : kMaxPosition, kEdge,
            2 * kMaxPosition};
}

constexpr uint32_t entry_of(uint32_t position, uint32_t byte) { return (position << 9) | byte; }

// the same entry, its window moved down to where it can be read
constexpr uint32_t edge_entry(uint32_t entry, uint32_t limit) {
    const uint32_t position = entry >> 9, byte = entry & 0xffu;
    if (position <= limit) return entry;
    const uint32_t shift = position - limit;
    return ((shift < 8 ? shift : 8u) << 28) | (limit << 9) | byte;
}

}  // namespace endor_gemv_windows

#endif  // ENDOR_GEMV_WINDOWS_H_
