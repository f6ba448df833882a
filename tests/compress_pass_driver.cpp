// How the one-pass compressor's workgroups share out their blocks (endor_compress_plan.h), replayed on the host with a
// thread for every wave: workgroups that start in any order, late, or only when others have ended.  Built and run by
// tests/test_compress_plan.py, by itself and under ThreadSanitizer: every access has the order that it has in the kernel,
// so what one wave reads of another's without having been given it is a race.  Not part of the library.
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <condition_variable>
#include <memory>
#include <thread>
#include <vector>

#include "endor_compress_plan.h"

using namespace endor_compress_plan;

namespace {

constexpr uint32_t kParty = 4, kPackers = 2;

void complain(const char *what, uint32_t a = 0, uint32_t b = 0) {
    std::printf("%s (%u, %u)\n", what, a, b);
    std::fflush(stdout);
    std::_Exit(1);
}

struct Rng {
    uint64_t s;
    uint32_t operator()(uint32_t n) {
        s = s * 6364136223846793005ull + 1442695040888963407ull;
        return static_cast<uint32_t>((s >> 33) % n);
    }
};

// what is in the table's memory
struct Shared {
    struct Party {
        std::atomic<uint64_t> span[kSpanSlots] = {};
        std::atomic<uint32_t> started{0}, first{0};
    };
    std::vector<Party> parties;
    std::vector<std::atomic<uint64_t>> words;
    std::vector<uint32_t> count;              // of a block's tiles, before the call
    std::vector<std::atomic<uint32_t>> packed;  // times, by all packing waves
    std::atomic<uint32_t> scanners{0};
    uint32_t groups, nblocks, most_polls;
    Shared(uint32_t g, uint32_t n, uint32_t polls)
        : parties((g + kParty - 1) / kParty), words(n), count(n * kPackers), packed(n), groups(g), nblocks(n), most_polls(polls) {}
};

// what is in a workgroup's LDS
struct Local {
    uint32_t count[kRing][kPackers] = {}, counted_block[kRing][kPackers] = {};
    std::atomic<uint32_t> arrived[kRing] = {};
    uint64_t first[kRing] = {};
    uint32_t block[kRing] = {};
    std::atomic<uint32_t> placed{0};
};

void breathe(Rng &r) {
    if (r(3) == 0) std::this_thread::yield();
}

void look_up(Shared &S, Local &L, uint32_t group, Rng r) {
    const uint32_t groups = S.groups, nblocks = S.nblocks, parties = static_cast<uint32_t>(S.parties.size());
    Shared::Party &own = S.parties[group / kParty];
    auto tell = [&](uint32_t placed) { L.placed.store(placed, std::memory_order_release); };
    const uint32_t registered = own.started.fetch_add(1, std::memory_order_relaxed);
    breathe(r);
    bool scans = registered == 0 && S.parties[0].first.fetch_add(1, std::memory_order_relaxed) == 0;
    auto started = [&]() {
        std::vector<uint32_t> here;
        for (auto &p : S.parties) here.push_back(p.started.load(std::memory_order_relaxed));
        return here;
    };
    auto give_out = [&](uint32_t number, uint32_t start, const std::vector<uint32_t> &here) {
        Span s{number, start, 0, 0, 0};
        for (uint32_t h : here) s.running += h;
        const Span all = s;
        for (uint32_t p = 0; p < parties; ++p) {
            s.here = here[p];
            S.parties[p].span[number % kSpanSlots].store(span_word(s), std::memory_order_relaxed);
            breathe(r);
            s.before += here[p];
        }
        return all;
    };
    uint32_t given = 0, given_start = 0, given_end = 0;
    if (scans) {
        std::vector<uint32_t> here;
        for (uint32_t polls = 0;; ++polls) {
            here = started();
            uint32_t running = 0;
            for (uint32_t h : here) running += h;
            if (has_waited(polls + (kMostPolls - S.most_polls), running, groups)) break;
            std::this_thread::yield();
        }
        given_end = span_end(give_out(0, 0, here), groups, nblocks);
    }
    Span span{};
    for (bool found = false; !found;) {
        uint64_t w[kSpanSlots];
        for (uint32_t i = 0; i < kSpanSlots; ++i) w[i] = own.span[i].load(std::memory_order_relaxed);
        for (uint32_t i = 0; i < kSpanSlots && !found; ++i) {
            span = span_of(w[i]);
            found = is_span(w[i]) && begins_with(span, w[(i + kSpanSlots - 1) % kSpanSlots], registered, nblocks);
        }
        if (!found) std::this_thread::yield();
    }
    Part part = part_of(span, group, registered, groups, nblocks);
    const bool whole = is_whole(span, groups);
    if (whole) scans = group == 0;
    if (scans && S.scanners.fetch_add(1, std::memory_order_relaxed) != 0) complain("two workgroups look the places up", group);
    auto next = [&](uint32_t b) -> uint32_t {
        if (b + part.stride < part.end || part.end >= nblocks) return b + part.stride;
        const uint32_t number = span.number + 1;
        for (;;) {
            const uint64_t w = own.span[number % kSpanSlots].load(std::memory_order_relaxed);
            span = span_of(w);
            if (is_span(w) && span.number == number) break;
            if (is_span(w) && span.number > number) complain("a span overwritten before it was read", number, span.number);
            if (scans) complain("the wave that gives spans out waits for one", number);
            std::this_thread::yield();
        }
        part = part_of(span, group, registered, groups, nblocks);
        return part.first;
    };
    uint32_t b0 = part.first, b1 = next(b0), b2 = next(b1);
    L.block[0] = b0;
    L.block[1] = b1;
    L.block[2] = b2;
    tell(1);
    uint32_t n = 0;
    auto place = [&](uint64_t w) {
        const uint32_t b3 = next(b2);
        L.block[(n + kHeld) % kRing] = b3;
        L.first[n % kRing] = word_upto(w) - word_own(w);
        tell(n + 2);
        ++n;
        b0 = b1;
        b1 = b2;
        b2 = b3;
    };
    if (!scans) {
        while (b0 < nblocks) {
            uint64_t w;
            while (!((w = S.words[b0].load(std::memory_order_acquire)) & kPlaced)) std::this_thread::yield();
            place(w);
        }
        return;
    }
    const uint32_t lanes = r(2) ? 64 : 1 + r(8);
    uint64_t before = 0;
    uint32_t pos = 0;
    auto give_out_due = [&]() {
        while (!whole && pos >= given_start && given_start < nblocks) {
            given_start = given_end;
            given_end = span_end(give_out(++given, given_start, started()), groups, nblocks);
        }
    };
    give_out_due();
    while (b0 < nblocks || pos < nblocks) {
        const uint64_t mine = S.words[b0 < nblocks ? b0 : nblocks - 1].load(std::memory_order_acquire);
        for (uint32_t i = 0; i < lanes && pos < nblocks; ++i, ++pos) {
            const uint64_t w = S.words[pos].load(std::memory_order_acquire);
            if (!(w & kCounted)) break;
            before += word_own(w);
            S.words[pos].store(placed_word(before, word_own(w)), std::memory_order_release);
        }
        give_out_due();
        if (b0 < nblocks && (mine & kPlaced)) place(mine);
        std::this_thread::yield();
    }
}

void pack_tiles(Shared &S, Local &L, uint32_t wave, const std::vector<uint64_t> &sums, Rng r) {
    const uint32_t nblocks = S.nblocks;
    auto until = [&](uint32_t placed) {
        while (L.placed.load(std::memory_order_acquire) < placed) std::this_thread::yield();
    };
    auto count = [&](uint32_t n, uint32_t block) {
        const uint32_t slot = n % kRing, own = block < nblocks ? S.count[block * kPackers + wave] : 0;
        breathe(r);
        struct Mem {
            Shared &S;
            Local &L;
            uint32_t slot, wave, block;
            void count(uint32_t v) {
                L.count[slot][wave] = v;
                L.counted_block[slot][wave] = block;
            }
            uint32_t arrive(uint32_t v) { return L.arrived[slot].fetch_add(v, std::memory_order_acq_rel); }
            void clear_arrived() { L.arrived[slot].store(0, std::memory_order_relaxed); }
            void publish(uint64_t w) {
                if (block < S.nblocks && S.words[block].exchange(w, std::memory_order_release) != 0) complain("a block counted twice", block);
            }
        };
        tile_counted(Mem{S, L, slot, wave, block}, kPackers, own);
    };
    auto pack = [&](uint32_t n, uint32_t block) {
        const uint32_t slot = n % kRing;
        uint64_t first = L.first[slot];
        for (uint32_t v = 0; v < wave; ++v) {
            if (L.counted_block[slot][v] != block) complain("another block's count", block, v);
            first += L.count[slot][v];
        }
        if (first != sums[block * kPackers + wave]) complain("a wrong place", block, wave);
        S.packed[block].fetch_add(1, std::memory_order_relaxed);
        breathe(r);
    };
    until(1);
    uint32_t b0 = L.block[0], b1 = L.block[1], b2 = L.block[2], n = 0;
    if (b0 >= nblocks) return;
    count(0, b0);
    while (b0 < nblocks) {
        count(n + 1, b1);
        until(n + 2);
        const uint32_t b3 = L.block[(n + kHeld) % kRing];
        pack(n, b0);
        if (b3 <= b2 && b3 < nblocks) complain("blocks out of order", b2, b3);
        b0 = b1;
        b1 = b2;
        b2 = b3;
        ++n;
    }
}

// `room`: workgroups that run at a time; the others start when one has ended.  Each starts after some time.
void call(uint32_t groups, uint32_t nblocks, uint32_t room, uint32_t most_polls, bool staggered, uint64_t seed) {
    Rng r{seed};
    Shared S(groups, nblocks, most_polls);
    std::vector<uint64_t> sums(nblocks * kPackers);
    uint64_t sum = 0;
    for (size_t i = 0; i < sums.size(); ++i) {
        sums[i] = sum;
        sum += S.count[i] = r(4) ? r(4097) : 0;
    }
    std::mutex m;
    std::condition_variable free;
    uint32_t running = 0;
    std::vector<std::thread> waves;
    std::vector<std::unique_ptr<Local>> locals;
    std::vector<uint32_t> order(groups);
    for (uint32_t i = 0; i < groups; ++i) order[i] = i;
    for (uint32_t i = groups; i-- > 1;) std::swap(order[i], order[r(i + 1)]);
    std::vector<std::atomic<uint32_t>> left(groups);
    for (uint32_t i = 0; i < groups; ++i) {
        const uint32_t group = order[i];
        {
            std::unique_lock<std::mutex> lock(m);
            free.wait(lock, [&] { return running < room; });
            ++running;
        }
        if (staggered)
            for (uint32_t k = r(60); k; --k) std::this_thread::yield();
        locals.push_back(std::make_unique<Local>());
        Local *L = locals.back().get();
        left[group] = 1 + kPackers;
        auto ended = [&, group] {
            if (left[group].fetch_sub(1) == 1) {
                std::lock_guard<std::mutex> lock(m);
                --running;
                free.notify_one();
            }
        };
        const uint64_t s = seed * 1000003 + group * 64;
        waves.emplace_back([&S, L, group, s, ended] {
            look_up(S, *L, group, Rng{s});
            ended();
        });
        for (uint32_t v = 0; v < kPackers; ++v)
            waves.emplace_back([&S, L, v, &sums, s, ended] {
                pack_tiles(S, *L, v, sums, Rng{s + v + 1});
                ended();
            });
    }
    for (auto &t : waves) t.join();
    for (uint32_t b = 0; b < nblocks; ++b)
        if (S.packed[b].load() != kPackers || word_upto(S.words[b].load()) != (b + 1 < nblocks ? sums[(b + 1) * kPackers] : sum)) complain("a block not done", b);
    if (S.scanners.load() != 1) complain("nobody looked the places up");
}

}  // namespace

int main(int argc, char **argv) {
    const uint32_t calls = argc > 1 ? static_cast<uint32_t>(std::atoi(argv[1])) : 1000;
    // a span's word holds what it is made from
    Rng r{7};
    for (int i = 0; i < 100000; ++i) {
        const Span a{r(1u << 18), r(1u << 20), r(1u << 10), r(1u << 10), r(1u << 5)}, b = span_of(span_word(a));
        if (!is_span(span_word(a)) || a.number != b.number || a.start != b.start || a.running != b.running || a.before != b.before || a.here != b.here)
            complain("a span's word", a.number, b.number);
    }
    for (uint32_t i = 0; i < calls; ++i) {
        const uint32_t groups = 2 + r(9), nblocks = groups + r(i % 8 ? 90 : 400);
        const uint32_t room = i % 3 == 0 ? groups : 1 + r(groups);
        call(groups, nblocks, room, i % 3 == 0 ? (i % 2 ? kMostPolls : 1) : 1 + r(kMostPolls), i % 4 != 0, i + 1);
    }
    std::printf("ok\n");
    return 0;
}
