// How the one-pass compressor shares out its blocks of tiles among the workgroups that run, and the words and slots in
// which they tell each other about them: plain arithmetic, apart from the kernel so that it can be replayed on the host.
#ifndef ENDOR_COMPRESS_PLAN_H_
#define ENDOR_COMPRESS_PLAN_H_

#include <cstdint>

namespace endor_compress_plan {

constexpr uint32_t kHeld = 3;          // blocks a workgroup holds
constexpr uint32_t kRing = kHeld + 1;  // a wave that has counted block n + 3 may find another at block n still

// A block's word: how many non-zeros it has, and once it is placed, how many there are up to its end.
constexpr uint64_t kCounted = uint64_t(1) << 62, kPlaced = uint64_t(1) << 63;
constexpr uint64_t counted_word(uint32_t own) { return kCounted | uint64_t(own) << 40; }
constexpr uint64_t placed_word(uint64_t upto, uint32_t own) { return kPlaced | uint64_t(own) << 40 | upto; }
constexpr uint32_t word_own(uint64_t w) { return static_cast<uint32_t>(w >> 40) & 0x3fffffu; }
constexpr uint64_t word_upto(uint64_t w) { return w & ((uint64_t(1) << 40) - 1); }

// A wave has counted its tile of a block: `own` non-zeros.  The waves that pack the block's later tiles read that when they have been
// told the block's place, by a wave that has it from the block's word, which another one completes, when the last wave to
// count has published it.  Every link of that chain hands on what the one before it has written: `arrive` gives out what its
// wave has written and takes in what those that arrived before it gave out, `publish` gives out, and whoever reads a
// word takes in.
template <class Mem>
constexpr void tile_counted(Mem mem, uint32_t tiles, uint32_t own) {
    mem.count(own);
    const uint32_t had = mem.arrive(own | 1u << 24);
    if (had >> 24 != tiles - 1) return;
    mem.clear_arrived();  // (before the word: the slot's next block is counted by waves that have been told this one's place)
    mem.publish(counted_word((had + own) & 0xffffffu));
}

// The first workgroup to register says how blocks are shared out when all are running, or after that many polls, 0.7 us
// each (by themselves all of them run within 10 us).
constexpr uint32_t kMostPolls = 32;
constexpr bool has_waited(uint32_t polls, uint32_t running, uint32_t groups) { return running >= groups || polls >= kMostPolls; }

// Blocks are shared out in spans, among the workgroups that were running when a span was given out: a workgroup has
// kSpanBlocks in each, at equal distances.  Once all are running a span takes the rest.  A span is given out when the
// places have reached the start of the one before it: a workgroup that has a place for a block and looks kHeld blocks
// ahead then finds it given out (or about to be, by a wave that waits for nobody).
constexpr uint32_t kSpanBlocks = kHeld + 1;
constexpr uint32_t kSpanSlots = 4;  // a span is read before the third one behind it can be reached

// A span, as it is told to the workgroups of a party.
struct Span {
    uint32_t number;
    uint32_t start;    // its first block; none: that was the last one
    uint32_t running;  // the workgroups that share it
    uint32_t before;   // those of the parties before
    uint32_t here;     // those of this party: the ones that registered first
};
// (blocks < 2^20, spans < 2^18, workgroups < 2^10, of a party < 2^5)
constexpr uint64_t span_word(const Span &s) {
    return uint64_t(1) << 63 | uint64_t(s.number) << 45 | uint64_t(s.here) << 40 | uint64_t(s.before) << 30 | uint64_t(s.running) << 20 | s.start;
}
constexpr bool is_span(uint64_t w) { return w >> 63; }
constexpr Span span_of(uint64_t w) {
    return Span{static_cast<uint32_t>(w >> 45) & 0x3ffffu, static_cast<uint32_t>(w) & 0xfffffu, static_cast<uint32_t>(w >> 20) & 0x3ffu,
                static_cast<uint32_t>(w >> 30) & 0x3ffu, static_cast<uint32_t>(w >> 40) & 0x1fu};
}
constexpr uint32_t span_end(const Span &s, uint32_t groups, uint32_t nblocks) {
    const uint32_t end = s.start + kSpanBlocks * s.running;
    return s.running >= groups || end > nblocks ? nblocks : end;
}
// all were running from the start: the first of the grid looks the places up and packs nothing
constexpr bool is_whole(const Span &s, uint32_t groups) { return s.number == 0 && s.running == groups; }

// A workgroup's blocks in a span: every stride-th from `first` to `end`.
struct Part {
    uint32_t first, stride, end;
};
// of the workgroup that is `group` of the grid and the `registered`-th of its party
constexpr Part part_of(const Span &s, uint32_t group, uint32_t registered, uint32_t groups, uint32_t nblocks) {
    if (is_whole(s, groups)) return Part{group ? group - 1 : nblocks, groups - 1, nblocks};
    return Part{s.start < nblocks ? s.start + s.before + registered : nblocks, s.running, span_end(s, groups, nblocks)};
}
// Whether a workgroup that has no span yet begins with this one: it is its first, or there are no more.  `word_before`: the
// one before in its slot, which has to be there to tell.
constexpr bool begins_with(const Span &s, uint64_t word_before, uint32_t registered, uint32_t nblocks) {
    if (registered >= s.here && s.start < nblocks) return false;
    const Span before = span_of(word_before);
    return s.number == 0 || (is_span(word_before) && before.number == s.number - 1 && registered >= before.here);
}

}  // namespace endor_compress_plan

#endif  // ENDOR_COMPRESS_PLAN_H_
