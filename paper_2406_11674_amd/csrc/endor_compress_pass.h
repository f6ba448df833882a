// The device compressor (Algorithm 1) in one pass over the dense matrix.  Included by endor_kernels.hip, whose
// types and loads it uses.
//
// Where a tile's values go is only known when every tile before it has been counted.  The two kernels that
// count and pack read the dense matrix twice; here a workgroup keeps its tiles in registers in between.  One
// workgroup per compute unit takes every groups-th block of tiles, one tile a wave.  A wave counts its tile
// of the next block, then packs its tile of this one, then asks for the block after the next: of three
// blocks, one is on its way from memory, one is counted and waits for its place, one is packed.
//
// Every block has a 64-bit word.  The last wave that has counted publishes the block's count there; one wave
// on the chip (of a workgroup that packs nothing) reads the words in order and completes them with the sums
// up to each; a wave of the block's own workgroup waits for that and tells the others through LDS.  What this
// takes, about 6 us, passes while the block before is packed and the one behind it arrives and is counted.
// (Numbers taken from one counter, instead of every groups-th block, were 25 us slower: additions to one
// address cost 25 to 50 ns each.)
//
// Where not all workgroups run, because other work holds compute units, blocks are given out a few a workgroup at a
// time, so that workgroups that start late, as the other work ends, share in what is left.  When those left instead, a
// call that had begun on a few units stayed on them: a pair of calls on two streams, 28672 x 8192 fp16, took 320 to 670
// us, at worst 1090, and 36864 x 9216 8-bit 320 to 820, at worst 1290, where it now takes 285 and 309, at worst 297 and
// 327 (of two passes 416 and 350).  (Numbers from a counter do not do here: workgroups that start one after the other take
// several in a row each, and every one waits for the last of the one before, 4 us a workgroup.)
//
// Every wait ends: only workgroups that have registered, and so are running, own blocks; the lowest block
// that is not counted belongs to one that waits for the places of lower blocks alone, and those are counted.
// The wave that looks places up gives the blocks out as it goes and waits for nothing but counts; with the last
// place it says that there are no more.
//
// Bound by memory: 28672 x 8192 fp16, half kept, 734 MB in 137 us, 5.4 TB/s; two passes take 199, loads
// and stores without the scatter 13 us less than this; 473 MB read, the matrix once, and 272 written, counted.  Of it, 10 us pass before the first values are written
// (the registration waits behind the first loads) and 6 after the last block has arrived.  Us a call, two
// passes / one: 28672 x 8192 fp16 a tenth, half, nine tenths kept 199 / 145, 220 / 165, 257 / 200;
// 8192 x 8192 85 / 77; 28672 x 8192 8-bit 148 / 132.
#ifndef ENDOR_COMPRESS_PASS_H_
#define ENDOR_COMPRESS_PASS_H_

namespace {

// Tiles of a block, one for each wave that packs.  With the wave that looks the places up the workgroup has 12
// waves, three a SIMD with up to 168 registers (three tiles of 16-bit elements are 96 of them; 8 waves kept too
// little in flight: 192 us where 12 took 171), or 16 of up to 128 for 8-bit elements (149 -> 137; 12: 147).
template <int E>
struct Blocks {
    static constexpr int kTiles = E == 2 ? 11 : 15;
    static constexpr int kThreads = 64 * (kTiles + 1);
    static constexpr int kPerChunk = (kTilesPerChunk + kTiles - 1) / kTiles;  // block words kept in a chunk's slice of the table
};
constexpr uint32_t kPackGroups = 256;  // workgroups: one a compute unit
using endor_compress_plan::counted_word;
using endor_compress_plan::kCounted;
using endor_compress_plan::kHeld;
using endor_compress_plan::kPlaced;
using endor_compress_plan::kRing;
using endor_compress_plan::kSpanSlots;
using endor_compress_plan::Part;
using endor_compress_plan::placed_word;
using endor_compress_plan::Span;
using endor_compress_plan::span_of;
using endor_compress_plan::word_own;
using endor_compress_plan::word_upto;

// The table's memory while the kernel runs, slice by slice: the words of some blocks, two parties, the counts of the
// chunk's tiles in 16 bits.
constexpr int kMaxPerChunk = Blocks<2>::kPerChunk > Blocks<1>::kPerChunk ? Blocks<2>::kPerChunk : Blocks<1>::kPerChunk;
constexpr int kPartyAt = 2 * kMaxPerChunk + 2 + 32;
constexpr int kCountsAt = kChunkStride - kTilesPerChunk / 2;
constexpr uint32_t kPassMinChunks = 16;  // whose slices hold all parties

template <int E>
__device__ __forceinline__ uint64_t *block_word(const MatParams &M, uint32_t block) {
    const uint32_t c = block / Blocks<E>::kPerChunk;
    return reinterpret_cast<uint64_t *>(M.tile_off + size_t(c) * kChunkStride + (c & 1)) + block % Blocks<E>::kPerChunk;
}

// Workgroups register in parties of 16: 256 additions to one counter take 25 us, to 16 counters two.
constexpr uint32_t kParty = 16;
constexpr uint32_t kParties = kPackGroups / kParty;
static_assert(kParty < 32 && kPackGroups < 1024 && kMaxElems / kTileElems / Blocks<2>::kTiles < int64_t(1) << 20, "a span's word");
struct alignas(8) Party {
    uint64_t span[kSpanSlots];
    uint32_t apart[32 - 2 * kSpanSlots];  // (a line of its own: the others' polls would hold the counter up)
    uint32_t started;  // workgroups of the party that run
    uint32_t first;    // (of the first party) parties that have asked who looks the places up
};
static_assert(kPartyAt % 2 == 0 && kPartyAt + int(sizeof(Party) / 4) < kCountsAt && kParties <= kPassMinChunks, "a party fits into a slice");
__device__ __forceinline__ Party *party(const MatParams &M, uint32_t p) {
    return reinterpret_cast<Party *>(M.tile_off + size_t(p) * kChunkStride + (p & 1) + kPartyAt);
}

template <class T>
__device__ __forceinline__ T peek(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class T>
__device__ __forceinline__ void publish(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// What a wave has written to LDS is given out with the next word it writes, and what others gave out taken in with a word it has
// read: a wait for the wave's own LDS accesses, none for memory.
__device__ __forceinline__ void give_out_lds() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent", "local"); }
__device__ __forceinline__ void take_in_lds() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent", "local"); }
__device__ __forceinline__ uint32_t first_lane(uint32_t v) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v))); }
__device__ __forceinline__ uint32_t lane_of(uint32_t v, uint32_t lane) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), lane)); }

// Words and parties of a chunk's slice empty.
__global__ __launch_bounds__(64) void endor_clear_blocks_kernel(MatParams M) {
    uint32_t *slice = M.tile_off + size_t(blockIdx.x) * kChunkStride;
    static_assert(kCountsAt == 129, "two stores a thread and one more");
    slice[threadIdx.x] = 0;
    slice[64 + threadIdx.x] = 0;
    if (threadIdx.x == 0) slice[128] = 0;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// `bytes` bytes from `p` on, both wave-uniform: loads outside bring 0, stores outside are dropped.  Loads and stores
// that would be under a test otherwise are unconditional this way, so the waits for what is in flight stay exact.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_range(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, static_cast<int>(bytes), 0x00020000);
}

// What a wave keeps of a tile between counting and packing it.
template <int E>
struct TileData {
    u32x4 d[Shape<E>::kSteps];
    uint32_t before;  // non-zeros of the tile before this lane's bitmap word
    uint32_t cnt;     // of the tile
};

template <int E>
struct alignas(16) PackScratch {
    static constexpr int kUnits = (E * (Shape<E>::kLaneElems - 1 + kTileElems) + 15) / 16;
    u32x4 stage[kUnits];
    uint64_t words[2][kTileWords];
    uint32_t start[kTileWords];
};

__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int E>
__global__ __launch_bounds__(Blocks<E>::kThreads, Blocks<E>::kThreads / 256) void endor_compress_kernel(CompressParams C, uint32_t nblocks) {
    using Sh = Shape<E>;
    constexpr uint32_t kTiles = Blocks<E>::kTiles;
    __shared__ PackScratch<E> s_scratch[kTiles];
    __shared__ uint32_t s_count[kRing][kTiles];
    __shared__ uint32_t s_arrived[kRing];  // waves that have counted their tile << 24 | its non-zeros
    __shared__ uint64_t s_first[kRing];    // non-zeros before the block
    // The workgroup's blocks: the first kHeld of them, then the n + kHeld-th by the time the n-th is placed.  (A slot is
    // written again when all waves have counted the block after the one it held, so they have read it.)
    __shared__ uint32_t s_block[kRing];
    __shared__ uint32_t s_placed;  // 1 when the first are known, then one more for every block that is placed
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    if (threadIdx.x < kRing) s_arrived[threadIdx.x] = 0;
    if (threadIdx.x == 0) s_placed = 0;
    __syncthreads();

    if (wave == kTiles) {
        auto tell = [&](uint32_t placed) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            if (lane == 0) __hip_atomic_store(&s_placed, placed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        // Who takes part: the first to register gives the first span out when all are running or have been waited for.  Where
        // all are, the first of the grid looks the places up; else the one that gave it out does, beside its own blocks.
        const uint32_t groups = gridDim.x;
        Party *own_party = party(C.table, blockIdx.x / kParty);
        uint32_t registered = 0, scans = 0;
        if (lane == 0) {
            registered = __hip_atomic_fetch_add(&own_party->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (registered == 0) scans = __hip_atomic_fetch_add(&party(C.table, 0)->first, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
        }
        registered = first_lane(registered);
        scans = first_lane(scans);
        auto started = [&]() { return lane < kParties ? peek(&party(C.table, lane)->started) : 0u; };
        auto give_out = [&](uint32_t number, uint32_t start, uint32_t here) {
            const uint32_t upto = wave_inclusive_scan(here);
            const Span span{number, start, lane_of(upto, 63), upto - here, here};
            if (lane < kParties) publish(&party(C.table, lane)->span[number % kSpanSlots], endor_compress_plan::span_word(span));
            return span;  // before and here: of the lane's party
        };
        uint32_t given = 0, given_start = 0, given_end = 0;  // the last span given out
        if (scans) {
            uint32_t here;
            for (uint32_t polls = 0;; ++polls) {
                here = started();
                if (endor_compress_plan::has_waited(polls, wave_sum(here), groups)) break;
            }
            given_end = span_end(give_out(0, 0, here), groups, nblocks);
        }
        Span span;
        auto uniform_span = [&](uint64_t w, uint32_t from) {
            return span_of(uint64_t(lane_of(static_cast<uint32_t>(w >> 32), from)) << 32 | lane_of(static_cast<uint32_t>(w), from));
        };
        for (bool found = false; !found;) {  // the first span this workgroup has blocks in
            const uint64_t w = lane < kSpanSlots ? peek(&own_party->span[lane]) : 0;
#pragma unroll
            for (uint32_t i = 0; i < kSpanSlots; ++i) {
                span = uniform_span(w, i);
                const uint64_t before = uint64_t(lane_of(static_cast<uint32_t>(w >> 32), (i + kSpanSlots - 1) % kSpanSlots)) << 32 |
                                        lane_of(static_cast<uint32_t>(w), (i + kSpanSlots - 1) % kSpanSlots);
                found = (lane_of(static_cast<uint32_t>(w >> 32), i) >> 31) != 0 &&
                        endor_compress_plan::begins_with(span, before, registered, nblocks);
                if (found) break;
            }
        }
        Part part = part_of(span, blockIdx.x, registered, groups, nblocks);
        const bool whole = is_whole(span, groups);
        if (whole) scans = blockIdx.x == 0;
        auto next = [&](uint32_t b) -> uint32_t {
            if (b + part.stride < part.end || part.end >= nblocks) return b + part.stride;
            const uint32_t number = span.number + 1;
            uint64_t w;
            do {
                w = peek(&own_party->span[number % kSpanSlots]);
                span = uniform_span(w, 0);
            } while ((first_lane(static_cast<uint32_t>(w >> 32)) >> 31) == 0 || span.number != number);
            part = part_of(span, blockIdx.x, registered, groups, nblocks);
            return part.first;
        };
        uint32_t b0 = part.first, b1 = next(b0), b2 = next(b1);
        if (lane == 0) {
            s_block[0] = b0;
            s_block[1] = b1;
            s_block[2] = b2;
        }
        tell(1);

        uint32_t n = 0;
        auto place = [&](uint64_t w) {  // of the workgroup's n-th block, b0, whose word is w
            take_in_lds();
            const uint32_t b = b0, b3 = next(b2);
            if (lane == 0) {
                s_block[(n + kHeld) % kRing] = b3;
                s_first[n % kRing] = word_upto(w) - word_own(w);
                if (b + 1 == nblocks) {
                    *C.nnz_out = static_cast<int64_t>(word_upto(w));
                    if (C.row_offsets) C.row_offsets[C.rows] = static_cast<int64_t>(word_upto(w));
                }
            }
            tell(n + 2);
            ++n;
            b0 = b1;
            b1 = b2;
            b2 = b3;
        };
        if (!scans) {
            while (b0 < nblocks) {
                uint64_t w;
                while (!((w = peek(block_word<E>(C.table, b0))) & kPlaced)) __builtin_amdgcn_s_sleep(1);
                place(w);
            }
            return;
        }
        __builtin_amdgcn_s_setprio(3);
        uint64_t before = 0;
        uint32_t pos = 0;
        // The spans that are due, and when all blocks have places the one that says that there are no more, which a workgroup
        // that starts late waits for.  (Where all are running there is nothing more to give out.)
        auto give_out_due = [&]() {
            while (!whole && pos >= given_start && given_start < nblocks) {
                given_start = given_end;
                given_end = span_end(give_out(++given, given_start, started()), groups, nblocks);
            }
        };
        give_out_due();
        while (b0 < nblocks || pos < nblocks) {
            const uint32_t j = pos + lane;  // (two or four words a lane: no faster where counts arrive steadily, by 3 and 8 us slower)
            const uint64_t w = peek(block_word<E>(C.table, j < nblocks ? j : nblocks - 1));
            const uint64_t mine = peek(block_word<E>(C.table, b0 < nblocks ? b0 : nblocks - 1));
            const uint64_t missing = ~__builtin_amdgcn_ballot_w64(j < nblocks && (w & kCounted) != 0);
            const uint32_t run = missing ? __builtin_ctzll(missing) : 64u;  // blocks from `pos` on that have been counted
            const uint32_t cnt = lane < run ? word_own(w) : 0u;
            const uint32_t incl = wave_inclusive_scan(cnt);
            take_in_lds();
            give_out_lds();
            if (lane < run) publish(block_word<E>(C.table, j), placed_word(before + incl, cnt));
            before += lane_of(incl, 63);
            pos += run;
            give_out_due();
            if (b0 < nblocks && (mine & kPlaced)) place(mine);
        }
        return;
    }

    PackScratch<E> &S = s_scratch[wave];
    auto until = [&](uint32_t placed) {
        while (__hip_atomic_load(&s_placed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < placed) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    auto valid = [&](uint32_t block) -> uint32_t {
        const int64_t left = C.n - (int64_t(block) * kTiles + wave) * kTileElems;
        return block >= nblocks || left <= 0 ? 0u : left < kTileElems ? static_cast<uint32_t>(left) : uint32_t(kTileElems);
    };
    auto load = [&](uint32_t block, TileData<E> &T) {
        const uint32_t nvalid = valid(block);
        const uint8_t *at = static_cast<const uint8_t *>(C.dense) + (int64_t(nvalid ? block : 0) * kTiles + wave) * kTileElems * E;
        const __amdgpu_buffer_rsrc_t r = buffer_range(const_cast<uint8_t *>(at), (nvalid * E) & ~15u);
#pragma unroll
        for (int k = 0; k < Sh::kSteps; ++k)
            T.d[k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + k * 1024, 0, 2));
    };
    auto count = [&](uint32_t n, uint32_t block, TileData<E> &T) {
        const uint32_t buf = n & 1, slot = n % kRing;
        const int64_t tile = int64_t(block) * kTiles + wave;
        const uint32_t nvalid = valid(block);
        if ((nvalid * E) & 15u) {  // the last tile: the elements that do not fill a 16-byte unit
            const uint32_t unit = nvalid / Sh::kLaneElems;
            const uint8_t *in = static_cast<const uint8_t *>(C.dense) + tile * kTileElems * E;
            const u32x4 v = load_dense16<E, false>(in, unit * Sh::kLaneElems, nvalid);
#pragma unroll
            for (uint32_t k = 0; k < Sh::kSteps; ++k) T.d[k] = unit == k * 64 + lane ? v : T.d[k];
        }
#pragma unroll
        for (int k = 0; k < Sh::kSteps; ++k) {
            const uint32_t bits = nonzero_bits<E>(T.d[k]);
            if (E == 2)
                reinterpret_cast<uint8_t *>(S.words[buf])[k * 64 + lane] = static_cast<uint8_t>(bits);
            else
                reinterpret_cast<uint16_t *>(S.words[buf])[k * 64 + lane] = static_cast<uint16_t>(bits);
        }
        lds_sync();
        const uint64_t word = S.words[buf][lane];
        const uint32_t pc = __popcll(word), incl = wave_inclusive_scan(pc);
        T.before = incl - pc;
        T.cnt = lane_of(incl, 63);
        if (lane == 0) {
            struct Mem {
                uint32_t *mine, *arrived;
                const MatParams &table;
                uint32_t block, nblocks;
                __device__ __forceinline__ void count(uint32_t own) { *mine = own; }
                __device__ __forceinline__ uint32_t arrive(uint32_t v) {
                    give_out_lds();
                    const uint32_t had = __hip_atomic_fetch_add(arrived, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    take_in_lds();
                    return had;
                }
                __device__ __forceinline__ void clear_arrived() { __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
                __device__ __forceinline__ void publish(uint64_t w) {
                    give_out_lds();
                    if (block < nblocks) ::publish(block_word<E>(table, block), w);
                }
            };
            const Mem mem{&s_count[slot][wave], &s_arrived[slot], C.table, block, nblocks};
            endor_compress_plan::tile_counted(mem, kTiles, T.cnt);
        }
        {
            const uint32_t nw = (nvalid + 63) / 64;
            const __amdgpu_buffer_rsrc_t r = buffer_range(C.bitmap + (nw ? tile * kTileWords : 0), nw * 8);
            const u32x2 v = {static_cast<uint32_t>(word), static_cast<uint32_t>(word >> 32)};
            __builtin_amdgcn_raw_buffer_store_b64(v, r, lane * 8, 0, 2);
        }
        if (lane == 0 && nvalid)  // (past this partition's L2, like everything in these lines)
            __hip_atomic_store(reinterpret_cast<uint16_t *>(C.table.tile_off + size_t(tile / kTilesPerChunk) * kChunkStride + kCountsAt) + tile % kTilesPerChunk,
                               static_cast<uint16_t>(T.cnt), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto pack = [&](uint32_t n, uint32_t block, const TileData<E> &T) {
        const uint32_t buf = n & 1, slot = n % kRing;
        const int64_t e0 = (int64_t(block) * kTiles + wave) * kTileElems;
        uint64_t first = s_first[slot];
        for (uint32_t v = 0; v < wave; ++v) first += s_count[slot][v];
        first = (uint64_t(__builtin_amdgcn_readfirstlane(int(first >> 32))) << 32) | uint32_t(__builtin_amdgcn_readfirstlane(int(first)));
        const uint32_t cnt = T.cnt;
        const uintptr_t vaddr = reinterpret_cast<uintptr_t>(C.values) + E * first, a16 = vaddr & ~uintptr_t(15);
        const uint32_t shift = static_cast<uint32_t>(vaddr - a16) / E;
        S.start[lane] = T.before + shift;
        lds_sync();
        // the rows that start in this tile begin with the non-zeros before it plus those of its earlier words
        if (C.row_offsets) {  // wave-uniform
            int64_t i = (e0 + C.cols - 1) / C.cols + lane;  // lane 0: the first such row
            for (; i < C.rows; i += 64) {
                const int64_t le = i * C.cols - e0;
                if (le >= kTileElems) break;
                const uint32_t wi = static_cast<uint32_t>(le) >> 6;
                const uint32_t in_tile = S.start[wi] - shift + __popcll(S.words[buf][wi] & ((uint64_t(1) << (le & 63)) - 1));
                C.row_offsets[i] = static_cast<int64_t>(first + in_tile);
            }
        }
        // scatter the non-zero elements into LDS in rank order
#pragma unroll
        for (int k = 0; k < Sh::kSteps; ++k) {
            const uint32_t wi = k * Sh::kLaneElems + lane / Sh::kLanesPerWord;
            const uint64_t w = S.words[buf][wi];
            const uint32_t sh = (lane % Sh::kLanesPerWord) * Sh::kLaneElems;
            uint32_t at = E * (S.start[wi] + __popcll(w & ((uint64_t(1) << sh) - 1)));
            const uint32_t bits = static_cast<uint32_t>(w >> sh) & ((1u << Sh::kLaneElems) - 1);
            const uint32_t dd[4] = {T.d[k].x, T.d[k].y, T.d[k].z, T.d[k].w};
#pragma unroll
            for (int j = 0; j < Sh::kLaneElems; ++j) {
                const uint32_t nz = (bits >> j) & 1u;
                if (nz) {
                    const uint32_t v = dd[(E * j) >> 2] >> (8 * ((E * j) & 3));
                    if (E == 2)
                        *reinterpret_cast<uint16_t *>(reinterpret_cast<uint8_t *>(S.stage) + at) = static_cast<uint16_t>(v);
                    else
                        *(reinterpret_cast<uint8_t *>(S.stage) + at) = static_cast<uint8_t>(v);
                }
                at += E * nz;
            }
        }
        lds_sync();
        // write the slice out: elements [shift, end) of the staging area go to values[first, ..), never past `capacity`
        const int64_t room = C.capacity > static_cast<int64_t>(first) ? C.capacity - static_cast<int64_t>(first) : 0;
        const uint32_t len = room < cnt ? static_cast<uint32_t>(room) : cnt;
        const uint32_t end = shift + len;
        const uint32_t u0 = shift ? 1u : 0u, u1 = end / Sh::kLaneElems;  // whole units [u0, u1)
        {
            const __amdgpu_buffer_rsrc_t r = buffer_range(reinterpret_cast<void *>(a16), len ? u1 * 16 : 0u);
            constexpr int kRounds = (PackScratch<E>::kUnits + 63) / 64;
            const uint32_t rounds = (u1 + 63) / 64;
            // unit 0, if it is shared, goes with the ends below: its lane is sent out of range
            const uint32_t off0 = lane < u0 ? 0x40000000u : lane * 16;
#pragma unroll
            for (int i = 0; i < kRounds; ++i) {
                if (i >= 4 && i >= int(rounds)) break;
                const uint32_t ch = i * 64 + lane;
                const u32x4 v = S.stage[ch < uint32_t(PackScratch<E>::kUnits) ? ch : 0];
                __builtin_amdgcn_raw_buffer_store_b128(v, r, (i == 0 ? off0 : lane * 16) + i * 1024, 0, 2);
            }
            // the units shared with the neighbours, element by element: lanes 0.. the first, lanes 32.. the last
            const uint32_t el = lane < 32 ? lane : u1 * Sh::kLaneElems + (lane - 32);
            const bool head = lane < Sh::kLaneElems && u0 && el >= shift && el < end;
            const bool tail = lane >= 32 && lane < 32 + Sh::kLaneElems && el < end && (u1 >= u0);
            if (head || tail) {
                if (E == 2)
                    global_ptr_mut<uint16_t>(a16)[el] = reinterpret_cast<const uint16_t *>(S.stage)[el];
                else
                    global_ptr_mut<uint8_t>(a16)[el] = reinterpret_cast<const uint8_t *>(S.stage)[el];
            }
        }
        lds_sync();
    };

    // (the first block is asked for before it is known whether all of the grid is running, as it nearly always is)
    TileData<E> T0, T1, T2;
    uint32_t b0 = blockIdx.x ? blockIdx.x - 1 : nblocks, n = 0;
    load(b0, T0);
    load(b0 + gridDim.x - 1, T1);
    until(1);
    const uint32_t first = first_lane(s_block[0]);
    uint32_t b1 = first_lane(s_block[1]), b2 = first_lane(s_block[2]);
    if (first >= nblocks) return;
    if (first != b0 || b1 != b0 + gridDim.x - 1) {
        b0 = first;
        load(b0, T0);
        load(b1, T1);
    }
    load(b2, T2);
    count(0, b0, T0);
    wait_loads_to_lds();
    // block n is counted, n + 1 and n + 2 are asked for
    auto step = [&](uint32_t &ba, uint32_t bb, TileData<E> &A, TileData<E> &B) __attribute__((always_inline)) {
        count(n + 1, bb, B);
        until(n + 2);
        const uint32_t further = s_block[(n + kHeld) % kRing];
        pack(n, ba, A);
        ba = first_lane(further);
        load(ba, A);
        ++n;
    };
    while (true) {
        if (b0 >= nblocks) break;
        step(b0, b1, T0, T1);
        if (b1 >= nblocks) break;
        step(b1, b2, T1, T2);
        if (b2 >= nblocks) break;
        step(b2, b0, T2, T0);
    }
}

// The tile counts endor_compress_kernel left in a chunk's slice, turned into its table: one workgroup per chunk.
__global__ __launch_bounds__(kTilesPerChunk) void endor_finish_table_kernel(MatParams M) {
    __shared__ uint32_t s_wave[kTilesPerChunk / 64];
    const uint32_t c = blockIdx.x, t = threadIdx.x, wave = t >> 6;
    uint32_t *to = M.tile_off + size_t(c) * kChunkStride;
    const int64_t ntiles = (M.n + kTileElems - 1) / kTileElems;
    const uint32_t cnt = int64_t(c) * kTilesPerChunk + t < ntiles ? reinterpret_cast<const uint16_t *>(to + kCountsAt)[t] : 0u;  // tiles past the end count as empty
    const uint32_t incl = wave_inclusive_scan(cnt);
    if ((t & 63) == 63) s_wave[wave] = incl;
    __syncthreads();  // every count has been read
    uint32_t before = 0;
    for (uint32_t v = 0; v < wave; ++v) before += s_wave[v];
    to[t] = before + incl - cnt;
    if (t == kTilesPerChunk - 1) {
        to[kTilesPerChunk] = before + incl;
        M.chunk_total[c] = before + incl;
    }
}

}  // namespace

#endif  // ENDOR_COMPRESS_PASS_H_
