// Replays on the host which units of a tile's slice of `values` are read as one (csrc/endor_value_units.h): all of
// them inside the array, none left out that is, for arrays at every alignment, slices over either end, over both, and
// slices anywhere, as a table that is not the bitmap's gives them.
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "endor_value_units.h"

using namespace endor_value_units;

static long checked = 0;

static bool check(uint64_t vbeg, uint64_t bytes, uint64_t vaddr, uint32_t cnt, uint32_t e) {
    const uint64_t vend = vbeg + bytes, a16 = vaddr & ~uint64_t(15);
    const uint32_t units = cnt ? static_cast<uint32_t>((vaddr - a16 + uint64_t(cnt) * e + 15) >> 4) : 0;
    const uint32_t first = first_whole(a16, units, vbeg), last = end_of_whole(a16, units, vbeg, vend);
    bool ok = first <= last && last <= units && all_inside(a16, units, vbeg, vend) == (units == 0 ? a16 >= vbeg && a16 <= vend : first == 0 && last == units);
    for (uint32_t u = 0; u < units; ++u) {
        const bool inside = a16 + 16 * uint64_t(u) >= vbeg && a16 + 16 * uint64_t(u) + 16 <= vend;
        ok = ok && inside == (u >= first && u < last);
    }
    ++checked;
    if (!ok) std::printf("vbeg %llu bytes %llu vaddr %llu cnt %u e %u: [%u, %u) of %u\n", (unsigned long long)vbeg, (unsigned long long)bytes,
                         (unsigned long long)vaddr, cnt, e, first, last, units);
    return ok;
}

int main() {
    bool ok = true;
    for (uint32_t e = 1; e <= 2; ++e)
        for (uint64_t off = 0; off < 16; off += e)
            for (uint64_t n : {0u, 1u, 2u, 7u, 8u, 9u, 15u, 16u, 17u, 31u, 40u, 513u, 4096u, 4097u}) {
                const uint64_t vbeg = 4096 + off, bytes = n * e;
                for (uint64_t at = 0; at <= n; at = at < 20 ? at + 1 : at * 2 + 3)
                    for (uint32_t cnt : {0u, 1u, 5u, 8u, 16u, 33u, 1024u, 4096u})
                        ok = check(vbeg, bytes, vbeg + at * e, cnt, e) && ok;
                for (uint32_t cnt : {1u, 8u, 4096u})  // behind the end, and far behind
                    ok = check(vbeg, bytes, vbeg + bytes + 1000 * e, cnt, e) && check(vbeg, bytes, vbeg + (uint64_t(1) << 35), cnt, e) && ok;
                ok = check(0, 0, off, 100, e) && ok;
            }
    std::printf("%ld slices\n", checked);
    return ok ? 0 : 1;
}
