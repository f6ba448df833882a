// The address arithmetic of the vector products' value loads (endor_gemv_windows.h), replayed on the host:
// every window must lie inside `values` and bring each bitmap byte the values it takes, and only an array
// without room for one window may be read element by element.  Built and run by tests/test_gemv_windows.py;
// not part of the library.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "endor_gemv_windows.h"

using namespace endor_gemv_windows;

static uint64_t state = 0x243F6A8885A308D3ull;
static uint64_t rnd() {
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}

static long windows = 0, edges = 0, elements = 0;

// A segment of the given bytes whose first value is number `first` of an array of nnz values at vbeg; value i is i.
static const char *segment(uint64_t vbeg, uint64_t nnz, uint64_t first, const std::vector<uint32_t> &bytes) {
    const uint64_t vend = vbeg + 2 * nnz, vseg = vbeg + 2 * first;
    uint32_t cnt = 0;
    for (uint32_t b : bytes) cnt += __builtin_popcount(b);
    const Windows whole = whole_windows(vseg);
    const bool all = is_whole(vbeg, vend, vseg, cnt);
    const Windows w = all ? whole : end_windows(vbeg, vend, vseg);
    if (w.how == kElements) {
        ++elements;
        return first <= nnz && nnz >= 8 ? "an array with room for a window is read element by element" : nullptr;
    }
    if (first > nnz) return "an offset behind the array leads to a read";
    edges += w.how == kEdge;
    uint32_t before = 0;
    uint64_t next_front = 0;  // of the window behind, going backwards
    std::vector<uint64_t> at(bytes.size());
    std::vector<uint32_t> entry(bytes.size());
    for (size_t i = 0; i < bytes.size(); ++i) {
        uint32_t e = entry_of(whole.first + before, bytes[i]);
        if (!all) e = edge_entry(e + ((w.first - whole.first) << 9), w.limit);
        entry[i] = e;
        at[i] = w.base + ((e >> 8) & w.offset_mask);
        if (at[i] < vbeg || at[i] + 16 > vend) return "a window reaches out of the array";
        if (w.how == kWhole && (at[i] & 3)) return "a window off its dword";
        if ((e & 0xff) != bytes[i]) return "an entry without its byte";
        before += __builtin_popcount(bytes[i]);
        ++windows;
    }
    // kWhole: a window's fifth dword is the next one's first, or the one at the segment's end
    const uint64_t end = (vseg + 2 * uint64_t(cnt)) & ~uint64_t(3);
    if (w.how == kWhole && (end < vbeg || end + 4 > vend)) return "the dword behind the segment reaches out of the array";
    before = 0;
    for (size_t i = bytes.size(); i-- > 0;) {
        const uint64_t after = i + 1 < bytes.size() ? next_front : end;
        uint32_t k0 = 0;
        for (size_t j = 0; j < i; ++j) k0 += __builtin_popcount(bytes[j]);
        for (uint32_t k = 0; k < static_cast<uint32_t>(__builtin_popcount(bytes[i])); ++k) {
            const uint64_t want = vseg + 2 * (k0 + k);
            if (want + 2 > vend) break;  // more bits than values: anything that is no read outside will do
            uint64_t got;
            if (w.how == kWhole) {
                const uint64_t byte = ((entry[i] >> 8) & 2) + 2 * k;
                got = byte < 16 ? at[i] + byte : after + byte - 16;
            } else {
                const uint64_t half = (entry[i] >> 28) + k;
                if (half >= 8) return "a value shifted out of its window";
                got = at[i] + 2 * half;
            }
            if (got != want) return "a byte gets another's value";
        }
        next_front = at[i];
    }
    return nullptr;
}

int main() {
    const char *bad = nullptr;
    for (int rep = 0; rep < 60000 && !bad; ++rep) {
        const uint64_t vbeg = 0x10000 + 2 * (rnd() % 16);
        const int steps = 2 << (rnd() % 3), density = static_cast<int>(rnd() % 10);
        std::vector<uint32_t> bytes(64 * steps, 0);
        const size_t used = rnd() % 3 ? rnd() % (bytes.size() + 1) : bytes.size();
        uint32_t cnt = 0;
        for (size_t i = 0; i < used; ++i) {
            for (int b = 0; b < 8; ++b)
                if (static_cast<int>(rnd() % 9) < density) bytes[i] |= 1u << b;
            cnt += __builtin_popcount(bytes[i]);
        }
        const uint64_t front = rnd() % 3 ? rnd() % 40 : rnd() % 20000, back = rnd() % 2 ? rnd() % 24 : rnd() % 20000;
        uint64_t nnz = front + cnt + back, first = front;
        switch (rnd() % 8) {
            case 0: nnz = front + rnd() % (cnt + 1); break;           // fewer values than bits
            case 1: first = nnz + 1 + rnd() % 10; break;              // an offset behind the array
            case 2: first = uint64_t(0) - 1 - rnd() % 5; break;       // and one before it
            default: break;
        }
        bad = segment(vbeg, nnz, first, bytes);
        if (bad)
            std::printf("%s: vbeg %llx nnz %llu first %llu cnt %u\n", bad, (unsigned long long)vbeg, (unsigned long long)nnz,
                        (unsigned long long)first, cnt);
    }
    if (bad) return 1;
    std::printf("ok %ld windows, %ld segments at an end, %ld element by element\n", windows, edges, elements);
    return 0;
}
