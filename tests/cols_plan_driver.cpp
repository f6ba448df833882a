// Which form a column subset takes (endor_cols_plan.h).  Built and run by tests/test_cols_plan.py; not part of the library.
// Checks what must hold of any plan over calls of every kind, then answers lines of
//     bytes of an element, rows, columns, values, columns asked, the output's address
// with
//     threads, round, staged, store
#include <cstdint>
#include <cstdio>

#include "endor_cols_plan.h"

using namespace endor_cols_plan;

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

// A complaint, or null.
static const char *check(int bytes, int64_t rows, int64_t cols, int64_t nsel, const Plan &p) {
    if (p.threads != 0) {
        if (p.threads != 256 && p.threads != 512) return "threads";
        if (cols > 64 * p.threads) return "more than a bitmap word a thread";
        if (int64_t(p.round) * p.threads < nsel || p.round > kMaxStreamQueries) return "queries without a thread";
        if (int64_t(bytes) * nsel > 0x7fffffff) return "a row of the output past 31 bits";
        return nullptr;
    }
    if (p.round != 3 && p.round != 4 && (p.round != 6 || p.staged)) return "no such round";
    if (p.store != Store::kPlain && bytes != 2) return "no such store";
    if (p.lds < static_cast<size_t>((cols + 63) / 64) * 16 + (p.staged ? size_t(p.stage_units) * 16 : 0)) return "LDS";
    if (p.staged && (p.lds > kMaxColsLds || rows == 1)) return "staged";
    return nullptr;
}

int main() {
    for (int rep = 0; rep < 1000000; ++rep) {
        const int bytes = 1 + static_cast<int>(rnd() % 2);
        const int64_t rows = size(rep % 20 ? 16 : 31), cols = size(18);
        if (rows > 0x7fffffff || cols > ((int64_t(1) << 34) - 1) / rows) continue;  // refused
        const int64_t nnz = static_cast<int64_t>(rnd() % static_cast<uint64_t>(rows * cols + 1)), most = (int64_t(1) << 34) / rows;
        int64_t nsel = rep % 10 ? 1 + static_cast<int64_t>(rnd() % static_cast<uint64_t>(cols)) : size(33);
        if (nsel > most) nsel = most;
        const Plan p = make_plan(bytes, rows, cols, nnz, nsel, bytes * rnd() % 4096);
        if (const char *bad = check(bytes, rows, cols, nsel, p)) {
            std::printf("%s: %d-byte %lld x %lld, %lld values, %lld columns\n", bad, bytes, (long long)rows, (long long)cols, (long long)nnz, (long long)nsel);
            return 1;
        }
    }
    long long bytes, rows, cols, nnz, nsel, out;
    while (std::scanf("%lld %lld %lld %lld %lld %lld", &bytes, &rows, &cols, &nnz, &nsel, &out) == 6) {
        const Plan p = make_plan(static_cast<int>(bytes), rows, cols, nnz, nsel, static_cast<uint64_t>(out));
        std::printf("%d %d %d %d\n", p.threads, p.round, p.staged ? 1 : 0, static_cast<int>(p.store));
    }
    return 0;
}
