// Device side of the Endor library for gfx950 (MI355X): the parallel form of
// Algorithm 2 (Section 4.1, "Decompression") and the offset table it needs.
//
// Algorithm 2 is a sequential walk with one running counter k: position e of the
// flat bit vector receives values[k] when bit e is 1 (then k advances) and the
// all-zero pattern otherwise.  Hence out[e] = bit(e) ? values[rank(e)] : 0 with
// rank(e) = number of 1 bits before e, and the work splits into
//
//   1. endor_tile_offsets_kernel: rank at every tile start (a tile is 4096
//      consecutive flat positions = 64 bitmap words = one 64-lane wave's worth of
//      words).  One workgroup covers a chunk of 256 tiles: it popcounts the chunk's
//      128 KiB of bitmap, scans the 256 tile counts and stores the tile offsets
//      relative to the chunk start plus the chunk's total.
//   2. endor_expand_kernel: one single-wave workgroup per tile, waves fully
//      independent (no workgroup barrier; measured faster on MI355X than wider
//      workgroups or several tiles per wave).  The wave adds up the totals of the
//      chunks before its own (a few loads per lane) to get the chunk's absolute
//      start, brings the tile's contiguous slice of `values` straight from memory
//      into LDS (16 bytes per lane and load), scans the 64 word popcounts across
//      lanes (DPP), and then, in 8 steps
//      of 512 elements, every lane turns one bitmap byte into 8 output elements
//      (8 LDS reads at rank-within-byte offsets, masked by the bits) and issues one
//      16-byte store, so a wave writes 1 KiB of contiguous dense output per store
//      instruction.
//
// The same tile expander, fed differently, gives the row-subset kernel (Section 4.2's
// selective load) and - run backwards, as a scatter - the pack step of the device-side
// compressor (Algorithm 1).  The element width (2 bytes, or 1 for the 8-bit variant of
// Section 4.2) is a template parameter throughout.  The products on the compressed form
// have files of their own; the compressor that reads a large matrix once and the column
// subset by workgroups that stay are in endor_compress_pass.h and endor_cols_stream.h.
//
// One rule shaped all of these kernels: a load under a per-lane test whose result is used
// after the test is waited for on the spot, so several of them in a row are as many trips
// to memory.  Loads are therefore either unconditional (behind one wave-uniform test, or
// from a clamped index, with the exceptional tiles in a loop of their own) or go straight
// to LDS.
//
// The path is bound by memory traffic (2 bytes written, 1/8 + 2p bytes read per
// element), so there is no matrix-core work here; all arithmetic on the format is
// integer and the values are only ever moved, never interpreted.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

#include "endor.h"
#include "endor_cols_plan.h"
#include "endor_compress_plan.h"
#include "endor_device.h"
#include "endor_layout.h"
#include "endor_value_units.h"

namespace {

using endor_device::chunk_base;
using endor_device::dpp_or_zero;
using endor_device::global_ptr;
using endor_device::global_ptr_mut;
using endor_device::load_to_lds16;
using endor_device::row_inclusive_scan;
using endor_device::u32x4;
using endor_device::wave_inclusive_scan;
using endor_device::wait_loads_to_lds;
using endor_device::wave_sum;

using endor_layout::kTileElems;      // flat positions per tile
using endor_layout::kTileWords;      // 64-bit bitmap words per tile (= lanes per wave)
using endor_layout::kTilesPerChunk;  // tiles one count workgroup covers
using endor_layout::kChunkStride;
using endor_layout::kMaxElems;
using endor_layout::align256;
using endor_layout::chunks_of;
using endor_layout::dims_ok;
using endor_layout::workspace_bytes_n;

using endor_cols_plan::kBlock;  // threads per workgroup of the row-offset and column kernels
using endor_cols_plan::kLineBytes;
using endor_cols_plan::Store;
constexpr int kWaves = kBlock / 64;
// Launch shapes.  Both were settled by measurement on MI355X (Llama2-70B layer, half the
// elements kept): the tile-offset kernel with 16 waves per 256-tile chunk, the expand kernel
// with one single-wave workgroup per tile (wider workgroups, several tiles per wave and half
// tiles per wave were all slower), non-temporal value loads and stores, cacheable bitmap loads.
constexpr int kCountWaves = 16;               // waves per workgroup of the tile-offset kernel
constexpr int kCountBlock = 64 * kCountWaves;
constexpr int kCountTilesPerWave = kTilesPerChunk / kCountWaves;
constexpr int kCountSteps = kCountTilesPerWave / 2;  // two tiles per step

static_assert(kTileWords == 64, "one bitmap word per lane");
static_assert(kTilesPerChunk == 256 && kCountBlock >= kTilesPerChunk && kCountTilesPerWave % 2 == 0 &&
                  kCountSteps >= 1,
              "the tile-offset workgroup scans one tile count per thread");

struct MatParams {
    const uint64_t *bitmap;
    const void *values;     // nnz elements of 1 or 2 bytes
    void *dense;            // rows*cols elements of the same width
    uint32_t *chunk_total;  // [nchunks] 1 bits per chunk
    uint32_t *tile_off;     // [nchunks][257] 1 bits before each tile, relative to the chunk start
    int64_t n;              // rows*cols
    int64_t nnz;
    uint32_t chunk_begin;   // first workgroup-chunk of this matrix inside the batch
    uint32_t nchunks;
};

struct BatchParams {
    MatParams m[ENDOR_MAX_BATCH];
    // the matrices' chunk_begin again, side by side: a wave finds its matrix from one scalar load
    // of these instead of walking the descriptors (entries past `count` hold 0xffffffff)
    uint32_t first_chunk[ENDOR_MAX_BATCH];
    int count;
};

// Bitmap word `w` of a matrix with `full_words` complete words and `tail_bits`
// valid bits in the word after them; pad bits and words past the end read as 0.
__device__ __forceinline__ uint64_t load_word_guarded(const uint64_t *bitmap, int64_t w,
                                                      int64_t full_words, uint32_t tail_bits) {
    if (w < full_words) return bitmap[w];
    if (w == full_words && tail_bits != 0) return bitmap[w] & ((uint64_t(1) << tail_bits) - 1);
    return 0;
}

// The chunk's number inside its matrix, in a way that has all of the descriptor in registers by then: otherwise the
// compiler loads each field before its first use, and a wave waits for the scalar cache four times before it knows where
// its values are.
__device__ __forceinline__ uint32_t chunk_in(const MatParams &M, uint32_t chunk) {
    uint32_t c;
    asm("s_sub_u32 %0, %1, %2"
        : "=s"(c)
        : "s"(chunk), "s"(M.chunk_begin), "s"(M.bitmap), "s"(M.values), "s"(M.dense), "s"(M.chunk_total), "s"(M.tile_off), "s"(M.n), "s"(M.nnz)
        : "scc");
    return c;
}

// The matrix that a chunk belongs to, and the chunk's number in it.  The first one's descriptor comes with the number that
// says whether it is the one; the others are counted off the vector unit, two scalar instructions a matrix.  (The
// compiler's own form was a vector addition, or a trip through a vector register, for each of the sixteen, 100 instructions in a row
// at the start of every wave.  Expanding 5003 x 3171, 0.7 kept, 12.2 us, now 11.4; the matrices of a Llama2-70B layer in one
// batch 450.8, now 448.5; 9216 x 36864, 8-bit, 92.8, now 92.3.)
__device__ __forceinline__ MatParams matrix_of(const BatchParams &P, uint32_t chunk, uint32_t &c) {
    MatParams M = P.m[0];
    c = chunk_in(M, chunk);
    if (chunk >= P.first_chunk[1]) {
        uint32_t mi = 1;
#pragma unroll
        for (int i = 2; i < ENDOR_MAX_BATCH; ++i)  // ascending, so a count
            asm("s_cmp_ge_u32 %1, %2\n\ts_addc_u32 %0, %0, 0" : "+s"(mi) : "s"(chunk), "s"(P.first_chunk[i]) : "scc");
        M = P.m[mi];
        c = chunk_in(M, chunk);
    }
    return M;
}

// ---------------------------------------------------------------- kernel 1: tile offsets

struct alignas(16) WordPair {
    uint64_t a, b;
};

// Workgroup of kCountWaves waves per chunk; wave w popcounts tiles
// [w*kCountTilesPerWave, (w+1)*kCountTilesPerWave) of the chunk in steps of two tiles
// (128 words: lanes 0..31 hold tile 2i, lanes 32..63 tile 2i+1, two words per lane),
// with all of its loads issued before the first popcount.
__global__ __launch_bounds__(kCountBlock) void endor_tile_offsets_kernel(BatchParams P) {
    __shared__ uint32_t s_cnt[kTilesPerChunk];
    __shared__ uint32_t s_wave[kTilesPerChunk / 64];

    const uint32_t gc = blockIdx.x;
    uint32_t c;
    const MatParams M = matrix_of(P, gc, c);
    const uint64_t *bitmap = M.bitmap;
    const int64_t full_words = M.n >> 6;
    const uint32_t tail_bits = static_cast<uint32_t>(M.n & 63);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;

    const uint32_t t0 = wave * kCountTilesPerWave;  // first tile of this wave inside the chunk
    const int64_t wbase = (int64_t(c) * kTilesPerChunk + t0) * kTileWords;
    const bool all_fast = (reinterpret_cast<uintptr_t>(bitmap) & 15) == 0 &&
                          wbase + kCountSteps * 128 <= full_words;  // wave-uniform

    uint32_t p[kCountSteps];
    if (all_fast) {
        WordPair wp[kCountSteps];
#pragma unroll
        for (int i = 0; i < kCountSteps; ++i)
            wp[i] = *reinterpret_cast<const WordPair *>(bitmap + wbase + i * 128 + lane * 2);
#pragma unroll
        for (int i = 0; i < kCountSteps; ++i) p[i] = __popcll(wp[i].a) + __popcll(wp[i].b);
    } else {
#pragma unroll
        for (int i = 0; i < kCountSteps; ++i) {
            const int64_t w = wbase + i * 128 + lane * 2;
            p[i] = __popcll(load_word_guarded(bitmap, w, full_words, tail_bits)) +
                   __popcll(load_word_guarded(bitmap, w + 1, full_words, tail_bits));
        }
    }
#pragma unroll
    for (int i = 0; i < kCountSteps; ++i) {
        uint32_t q = row_inclusive_scan(p[i]);
        q += dpp_or_zero<0x142, 0xa>(q);  // lanes 31 and 63 now hold the two tile counts
        if ((lane & 31) == 31) s_cnt[t0 + 2 * i + (lane >> 5)] = q;
    }
    __syncthreads();

    if (threadIdx.x < kTilesPerChunk) {  // the first four waves scan the 256 tile counts
        const uint32_t cnt = s_cnt[threadIdx.x];
        const uint32_t incl = wave_inclusive_scan(cnt);
        if (lane == 63) s_wave[wave] = incl;
        s_cnt[threadIdx.x] = incl - cnt;
    }
    __syncthreads();
    if (threadIdx.x < kTilesPerChunk) {
        uint32_t before = 0;
        for (uint32_t v = 0; v < wave; ++v) before += s_wave[v];
        const uint32_t excl = before + s_cnt[threadIdx.x];
        uint32_t *to = M.tile_off + size_t(c) * kChunkStride;
        to[threadIdx.x] = excl;
        if (threadIdx.x == kTilesPerChunk - 1) {
            const uint32_t total = before + s_wave[wave];
            to[kTilesPerChunk] = total;
            M.chunk_total[c] = total;
        }
    }
}

// ---------------------------------------------------------------- kernel 2: expand

// Element width E in bytes: 2 (fp16, the paper's main case) or 1 (the 8-bit variant of
// Section 4.2).  A lane produces 16 bytes of output per step, i.e. kLaneElems elements
// covering kLaneElems bitmap bits; a tile of 4096 elements takes kSteps steps.
template <int E>
struct Shape {
    static constexpr int kLaneElems = 16 / E;                  // 8 or 16
    static constexpr int kSteps = kTileElems / (64 * kLaneElems);  // 8 or 4
    static constexpr int kLanesPerWord = 64 / kLaneElems;      // 8 or 4
};

// LDS a wave needs to expand a tile.  kCap = values the staging area holds at once: 4096 (a
// whole tile, whatever its density) or, for matrices known to be sparse, 1024 - a tile with more
// 1 bits than that is then expanded step by step (slower, but such tiles are rare there) and
// the smaller footprint lets more waves share a compute unit, which is what a store-dominated
// matrix wants (measured at one element in ten kept: 103 -> 97 us on 8192 x 28672).
template <int E, int kCap = kTileElems>
struct alignas(16) WaveScratch {
    static_assert(kCap >= 1024 && kCap <= kTileElems, "a step covers up to 1024 values");
    static constexpr int kLaneElems = Shape<E>::kLaneElems;
    // staging in 16-byte units: up to kLaneElems-1 elements of alignment slack in front, kCap
    // values, and kLaneElems-1 elements a lane may read past its last value (those reads are
    // masked off by the bits)
    // (8-bit values are read as dword pairs around a lane's values, up to 4 bytes further: one unit more)
    static constexpr int kStageChunks = (E * (2 * (kLaneElems - 1) + kCap) + 15) / 16 + (E == 1 ? 1 : 0);
    static constexpr int kStageRounds = (kStageChunks + 63) / 64;
    // last index a lane's values may start at
    static constexpr uint32_t kMaxIndex = (kStageChunks - (E == 1 ? 1 : 0)) * (16 / E) - kLaneElems;
    u32x4 stage[kStageChunks];   // the tile's slice of `values`, from the 16-byte boundary below it
    uint64_t words[kTileWords];  // the tile's bitmap words
    uint32_t start[kTileWords];  // per word: index into `stage` (in elements) of its first value
    // 8-bit values only: per 4-bit pattern the v_perm_b32 selector that moves the pattern's
    // consecutive values to the positions of its 1 bits and zeroes the others
    uint32_t nibble_sel[E == 1 ? 16 : 1];
};

// Selector for pattern n (bits 0..3): output byte k takes source byte popcount(n below k) when
// bit k is set, and the constant zero (selector 0x0c) otherwise.
__device__ __forceinline__ uint32_t nibble_selector(uint32_t n) {
    uint32_t sel = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        sel |= (((n >> k) & 1u) ? uint32_t(__popc(n & ((1u << k) - 1))) : 0x0cu) << (8 * k);
    return sel;
}

// 16 bytes of `values`, which are not empty, at byte address p, with elements outside [vbeg, vend) read as 0.  For
// the units over an end of the array, element by element: all loads unconditional, from a place that exists, so
// that they are one trip to memory (under a test each is waited for, 8 or 16 trips one after the other, 4 to 9 us
// at the end of every call whose last value does not end a unit).
template <int E>
__device__ __forceinline__ u32x4 load_values16(uintptr_t p, uintptr_t vbeg, uintptr_t vend) {
    uint32_t v[16 / E];
#pragma unroll
    for (int j = 0; j < 16 / E; ++j) {
        const uintptr_t q = p + E * j;
        const bool in = q >= vbeg && q + E <= vend;
        const uintptr_t at = in ? q : vbeg;
        v[j] = (E == 2) ? uint32_t(*global_ptr<uint16_t>(at)) : uint32_t(*global_ptr<uint8_t>(at));
        v[j] = in ? v[j] : 0u;
    }
    uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 16 / E; ++j) d[(E * j) >> 2] |= v[j] << (8 * ((E * j) & 3));
    u32x4 r;
    r.x = d[0];
    r.y = d[1];
    r.z = d[2];
    r.w = d[3];
    return r;
}

// A tile's slice of `values`, as 16-byte units from the boundary a16 at or below its first value, goes to the staging
// area: units that lie inside the array as a whole straight from memory (global_load_lds_dwordx4: lane l of an
// instruction deposits its 16 bytes at the LDS address in M0 plus 16*l), no registers in between, streamed past the
// caches as values are read once (the bitmap, read by both kernels, stays cacheable); the units over an end of the
// array, usually one, element by element.  ask() puts the loads out, finish() is what remains to be done when the
// bitmap has been worked on, with a wait.
// Only the unit itself goes that way: with all units of the array's first and last tiles put together from their
// elements, trip after trip, 2048 x 2048, four in five kept, took 8.6 us (now 5.0), 4096 x 4096 14.4 (11.7).
template <int E, int kRounds>
struct ValueSlice {
    uintptr_t a16, vbeg, vend;
    uint32_t units;
    bool inside;  // wave-uniform: all of them lie inside `values`

    __device__ __forceinline__ ValueSlice(uintptr_t a16_, uint32_t units_, uintptr_t vbeg_, uintptr_t vend_)
        : a16(a16_), vbeg(vbeg_), vend(vend_), units(units_), inside(endor_value_units::all_inside(a16_, units_, vbeg_, vend_)) {}
    // those that do: [first, last)
    __device__ __forceinline__ uint32_t first() const { return endor_value_units::first_whole(a16, units, vbeg); }
    __device__ __forceinline__ uint32_t last() const { return endor_value_units::end_of_whole(a16, units, vbeg, vend); }
    __device__ __forceinline__ void ask(u32x4 *stage, uint32_t lane) const {
        if (__builtin_expect(inside, 1)) {
#pragma unroll
            for (int q = 0; q < kRounds; ++q) {
                const uint32_t ch = q * 64 + lane;
                if (ch < units) load_to_lds16(reinterpret_cast<const u32x4 *>(a16) + ch, &stage[q * 64]);
            }
        } else {
            const uint32_t f = first(), l = last();
#pragma unroll 1
            for (int q = 0; q < kRounds; ++q) {
                const uint32_t ch = q * 64 + lane;
                if (ch >= f && ch < l) load_to_lds16(reinterpret_cast<const u32x4 *>(a16) + ch, &stage[q * 64]);
            }
        }
    }
    __device__ __forceinline__ void finish(u32x4 *stage, uint32_t lane) const {
        if (__builtin_expect(!inside, 0)) {
            const uint32_t f = first(), whole = last() - f;
#pragma unroll 1
            for (uint32_t i = lane; i < units - whole; i += 64) {  // (more than two behind a table that is not the bitmap's)
                const uint32_t ch = i < f ? i : i + whole;
                stage[ch] = vbeg < vend ? load_values16<E>(a16 + 16 * uintptr_t(ch), vbeg, vend) : u32x4{0u, 0u, 0u, 0u};
            }
        }
        wait_loads_to_lds();
    }
};

// 0xffff in the halves whose bit is set: bits 0,1 of `b` -> low, high half
__device__ __forceinline__ uint32_t half_mask(uint32_t b) {
    return ((b & 1u) ? 0xffffu : 0u) | ((b & 2u) ? 0xffff0000u : 0u);
}

// Sink that writes the expanded tile to memory: a 16-byte non-temporal store per lane
// and step when the tile is complete and the output 16-byte aligned, else element by
// element with a bounds check.  kBurst holds the steps' results back and releases all of
// them after the last step: measured 11 % faster when almost everything is stores (one
// element in ten kept), 6 % slower at three in ten, so the host picks it by density.
template <int E, bool kAlignedOut, bool kBurst, uint32_t kElems = kTileElems>
struct StoreSink {
    uint8_t *out;     // byte address of the tile's first output element (of kElems)
    uint32_t nvalid;  // elements of the tile that exist
    u32x4 held[kBurst ? Shape<E>::kSteps : 1];
    // how far a loop over the steps must be unrolled for `held` to stay in registers
    static constexpr int kStepUnroll = kBurst ? Shape<E>::kSteps : 1;
    __device__ __forceinline__ void put(uint32_t le, u32x4 d) const {
        __builtin_nontemporal_store(d, reinterpret_cast<u32x4 *>(out + size_t(le) * E));
    }
    __device__ __forceinline__ void operator()(int k, uint32_t le, u32x4 d) {
        if (kAlignedOut && nvalid == kElems) {
            if (kBurst) {
                held[k] = d;
                if (k == Shape<E>::kSteps - 1) {
#pragma unroll
                    for (int g = 0; g < Shape<E>::kSteps; ++g)
                        put(le - (Shape<E>::kSteps - 1 - g) * 64 * Shape<E>::kLaneElems, held[g]);
                }
            } else {
                put(le, d);
            }
        } else {
            const uint32_t dd[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int j = 0; j < Shape<E>::kLaneElems; ++j) {
                if (le + j < nvalid) {
                    const uint32_t v = dd[(E * j) >> 2] >> (8 * ((E * j) & 3));
                    if (E == 2)
                        reinterpret_cast<uint16_t *>(out)[le + j] = static_cast<uint16_t>(v);
                    else
                        out[le + j] = static_cast<uint8_t>(v);
                }
            }
        }
    }
};

// One step of the expansion: every lane turns kLaneElems bitmap bits into 16 bytes of output.
// S.words and S.start (per word: index into S.stage of its first value) are in place.
template <int E, int kCap, class Sink>
__device__ __forceinline__ void expand_step(const WaveScratch<E, kCap> &S, int k, uint32_t lane, Sink &sink) {
    using Sh = Shape<E>;
    const uint32_t wi = k * Sh::kLaneElems + lane / Sh::kLanesPerWord;
    const uint64_t w = S.words[wi];
    const uint32_t sh = (lane % Sh::kLanesPerWord) * Sh::kLaneElems;
    const uint32_t bits = static_cast<uint32_t>(w >> sh) & ((1u << Sh::kLaneElems) - 1);
    uint32_t s = S.start[wi] + __popcll(w & ((uint64_t(1) << sh) - 1));
    // with a whole tile staged the index cannot leave the staging area; with a smaller area a
    // table that does not belong to the bitmap could make it, so it is clamped
    if (kCap < kTileElems) s = s > WaveScratch<E, kCap>::kMaxIndex ? WaveScratch<E, kCap>::kMaxIndex : s;
    // every element is read from the staging area at its rank; the ones whose bit is 0
    // pick up a neighbour's value and are masked to the all-zero pattern.
    u32x4 d;
    if (E == 2) {
        const uint16_t *sp = reinterpret_cast<const uint16_t *>(S.stage) + s;
        uint32_t h[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) h[j] = sp[__popc(bits & ((1u << j) - 1))];
        d.x = (h[0] | (h[1] << 16)) & half_mask(bits);
        d.y = (h[2] | (h[3] << 16)) & half_mask(bits >> 2);
        d.z = (h[4] | (h[5] << 16)) & half_mask(bits >> 4);
        d.w = (h[6] | (h[7] << 16)) & half_mask(bits >> 6);
    } else {
        // 8-bit values: an output dword's four elements take consecutive values, so one read of the
        // two dwords around them, a funnel shift and a byte permute replace four single-byte
        // gathers (the 8-bit kernel was bound by vector ALU and LDS instructions, not by memory)
        const uint32_t *sw = reinterpret_cast<const uint32_t *>(S.stage);
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t at = s + __popc(bits & ((1u << (4 * q)) - 1));  // byte index of the dword's first value
            const uint32_t lo = sw[at >> 2], hi = sw[(at >> 2) + 1];
            const uint32_t x = __builtin_amdgcn_alignbyte(hi, lo, at & 3u);
            o[q] = __builtin_amdgcn_perm(x, x, S.nibble_sel[(bits >> (4 * q)) & 15u]);
        }
        d.x = o[0];
        d.y = o[1];
        d.z = o[2];
        d.w = o[3];
    }
    sink(k, (k * 64 + lane) * Sh::kLaneElems, d);
}

// LDS operations of one wave execute in issue order, so reads after this point see the writes
// before it; the fences only keep the compiler from moving them.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Expand one tile with one wave.
//   word     this lane's 64 bitmap bits of the tile (bits past the end already cleared)
//   vaddr    byte address of the tile's first value; cnt = number of 1 bits in the tile
//   [vbeg, vend)  the byte range of the whole `values` array (nothing outside is read)
//   sink     receives, per step k, the 16 expanded bytes of this lane: sink(k, le, d) with le
//            the index inside the tile of the lane's first element
// The caller has not touched S since the wave's previous call returned.
// (Measured alternatives to the per-element gather that lost for the store-bound kernels: one
// 32-bit read per output dword plus a byte permutation, with misaligned reads 1.8x slower,
// with aligned pairs and a funnel shift 1.0-1.4x.)
template <int E, int kCap, class Sink>
__device__ __forceinline__ void expand_tile(WaveScratch<E, kCap> &S, uint32_t lane, uint64_t word, uintptr_t vaddr,
                                            uint32_t cnt, uintptr_t vbeg, uintptr_t vend, Sink &sink) {
    using Sh = Shape<E>;
    using WS = WaveScratch<E, kCap>;
    // --- the loads of the tile's value slice (16-byte units from the 16-byte boundary at or
    //     below its first value) go out first: they depend on the table only, and the wave's
    //     bitmap word, loaded by the caller, may still be on its way
    const uintptr_t a16 = vaddr & ~uintptr_t(15);
    const uint32_t shift = static_cast<uint32_t>(vaddr - a16) / E;  // elements of slack in front
    if (E == 1 && lane < 16) S.nibble_sel[lane] = nibble_selector(lane);
    cnt = cnt > kCap ? kCap : cnt;  // a stale or foreign table must not overrun the staging area
    const uint32_t nch = cnt ? (((shift + cnt) * E + 15) >> 4) : 0;  // < kStageChunks
    const ValueSlice<E, WS::kStageRounds> slice(a16, nch, vbeg, vend);
    slice.ask(S.stage, lane);
    const uint32_t pc = __popcll(word);
    const uint32_t incl = wave_inclusive_scan(pc);
    const uint32_t excl = incl - pc;
    if (kCap < kTileElems) {
        // more 1 bits than the staging area holds (decided on the bitmap itself, not on the
        // table): stage and expand the tile one step at a time; a step has at most 1024 values
        const uint32_t ones = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
        if (ones > kCap) {  // wave-uniform
            wait_loads_to_lds();  // what is on its way into the staging area lands before it is reused
            S.words[lane] = word;
#pragma unroll Sink::kStepUnroll
            for (int k = 0; k < Sh::kSteps; ++k) {
                // values before the step's first word; the step's own count
                const uint32_t w0 = k * Sh::kLaneElems;
                const uint32_t first = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(4 * w0, static_cast<int>(excl)));
                const uint32_t last = static_cast<uint32_t>(
                    __builtin_amdgcn_ds_bpermute(4 * (w0 + Sh::kLaneElems - 1), static_cast<int>(incl)));
                const uintptr_t va = vaddr + uintptr_t(E) * first;
                const uintptr_t b16 = va & ~uintptr_t(15);
                const uint32_t sh = static_cast<uint32_t>(va - b16) / E;
                const uint32_t n = last - first;  // <= 1024 <= kCap
                const uint32_t nc = n ? (((sh + n) * E + 15) >> 4) : 0;
                S.start[lane] = excl - first + sh;  // meaningful for the step's words only
                const ValueSlice<E, WS::kStageRounds> of_step(b16, nc, vbeg, vend);
                of_step.ask(S.stage, lane);
                of_step.finish(S.stage, lane);
                wave_lds_sync();
                expand_step<E, kCap>(S, k, lane, sink);
                wave_lds_sync();
            }
            return;
        }
    }
    S.words[lane] = word;
    S.start[lane] = excl + shift;
    slice.finish(S.stage, lane);
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < Sh::kSteps; ++k) expand_step<E, kCap>(S, k, lane, sink);
    // the next tile's LDS writes must stay behind this tile's LDS reads
    wave_lds_sync();
}

// kCap: values the staging area holds (the host picks it from the batch's density); kBurst: all
// stores of a tile released together (for store-dominated matrices).
template <int E, bool kAlignedOut, int kCap, bool kBurst>
__global__ __launch_bounds__(64) void endor_expand_kernel(BatchParams P) {
    __shared__ WaveScratch<E, kCap> s_scratch;
    const uint32_t gc = blockIdx.x / kTilesPerChunk;
    const uint32_t tl = blockIdx.x % kTilesPerChunk;  // tile, relative to the chunk
    uint32_t c;
    const MatParams M = matrix_of(P, gc, c);
    const uint32_t lane = threadIdx.x;

    const int64_t n = M.n;
    const int64_t ntiles = (n + kTileElems - 1) / kTileElems;
    const int64_t tile = int64_t(c) * kTilesPerChunk + tl;
    if (tile >= ntiles) return;

    const uintptr_t vbeg = reinterpret_cast<uintptr_t>(M.values);
    const uintptr_t vend = vbeg + E * static_cast<uintptr_t>(M.nnz);
    const int64_t e0 = tile * kTileElems;
    const int64_t left = n - e0;
    // the bitmap word first: its load is in flight while the table is looked up
    uint64_t word = M.bitmap[tile * kTileWords + (64 * int64_t(lane) < left ? lane : 0u)];
    if (left < kTileElems) {  // wave-uniform
        const int64_t bits = left - 64 * int64_t(lane);
        if (bits < 64) word = bits > 0 ? word & ((uint64_t(1) << bits) - 1) : 0;
    }
    const uint32_t *tile_off = M.tile_off + size_t(c) * kChunkStride + tl;
    const uint32_t o0 = tile_off[0];
    const uint32_t o1 = tile_off[1];
    const uint64_t base = chunk_base(M.chunk_total, c, lane);
    const uint32_t cnt = o1 - o0;  // 1 bits in this tile
    StoreSink<E, kAlignedOut, kBurst> sink;
    sink.out = reinterpret_cast<uint8_t *>(M.dense) + e0 * E;
    sink.nvalid = left < kTileElems ? static_cast<uint32_t>(left) : uint32_t(kTileElems);
    expand_tile<E>(s_scratch, lane, word, vbeg + E * (base + o0), cnt, vbeg, vend, sink);
}

// Both kernels in one for a small matrix: a workgroup of kSmallTiles tiles counts the bitmap before them
// itself, all of it, instead of reading a table another kernel has to build first, and writes its part of
// the table on the way.  Two dependent launches were most of the time of a small call.  What bounds it is
// a chain: the launch, the bitmap (read n/2^15 times in all, from the second-level cache), the values, the
// stores.  So the counting is one trip to memory where a thread has no more than kBatch pieces of it, and four
// waves share a tile, a quarter each, which shortens what follows.
constexpr int kSmallTiles = 4;
constexpr int kParts = 4;  // waves per tile
constexpr int kSmallWaves = kSmallTiles * kParts;
constexpr int kPartWords = kTileWords / kParts, kPartElems = kTileElems / kParts;
static_assert(kSmallWaves == 16 && kPartWords == 16, "a value per wave, and a word, in each of 16 lanes");

__device__ __forceinline__ uint32_t row_sum(uint32_t x) {  // over the first 16 lanes
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(row_inclusive_scan(x)), 15));
}

template <int E, bool kAlignedOut>
__global__ __launch_bounds__(64 * kSmallWaves) void endor_decompress_small_kernel(MatParams M) {
    typedef WaveScratch<E, kPartElems> WS;
    __shared__ WS s_scratch[kSmallWaves];
    __shared__ uint32_t s_before[2][kSmallWaves];  // 1 bits before the workgroup's chunk, and from there to its first tile
    __shared__ uint32_t s_cnt[kSmallWaves];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t tile0 = blockIdx.x * kSmallTiles;  // a chunk's tiles are a multiple of a workgroup's
    const uint32_t tile = tile0 + wave / kParts;
    const uint32_t c = tile0 / kTilesPerChunk;
    const uint32_t n = static_cast<uint32_t>(M.n);
    const uint32_t ntiles = (n + kTileElems - 1) / kTileElems, last_word = (n - 1) >> 6;
    // this wave's words, one in each of 16 lanes (and again in the others)
    const uint32_t w_own = tile0 * kTileWords + wave * kPartWords + (lane & 15);
    uint64_t word = M.bitmap[w_own < last_word ? w_own : last_word];

    // the words before the workgroup's tiles (all of them complete), two a load
    struct alignas(8) Words2 {
        uint64_t a, b;
    };
    constexpr uint32_t kBatch = 8;
    uint32_t before[2] = {0, 0};
    const uint32_t npairs = tile0 * (kTileWords / 2), chunk_pair = c * kTilesPerChunk * (kTileWords / 2);
    for (uint32_t w0 = 0; w0 < npairs; w0 += kBatch * 64 * kSmallWaves) {
        Words2 x[kBatch];
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            const uint32_t w = w0 + k * 64 * kSmallWaves + threadIdx.x;
            x[k] = reinterpret_cast<const Words2 *>(M.bitmap)[w < npairs ? w : npairs - 1];
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            const uint32_t w = w0 + k * 64 * kSmallWaves + threadIdx.x;
            const uint32_t pc = w < npairs ? __popcll(x[k].a) + __popcll(x[k].b) : 0;
            before[0] += w < chunk_pair ? pc : 0u;
            before[1] += w < chunk_pair ? 0u : pc;
        }
    }
    if (w_own == last_word && (n & 63)) word &= (uint64_t(1) << (n & 63)) - 1;
    if (w_own > last_word) word = 0;
    const uint32_t pc = __popcll(word), incl = row_inclusive_scan(pc);
    const uint32_t cnt = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 15));
    const uint32_t b0 = wave_sum(before[0]), b1 = wave_sum(before[1]);
    if (lane == 0) {
        s_before[0][wave] = b0;
        s_before[1][wave] = b1;
        s_cnt[wave] = cnt;
    }
    __syncthreads();
    // before the chunk; from there to the workgroup's tiles; to this tile, to this part; and to the end of the workgroup's tiles
    const uint32_t v = lane & 15, of_v = s_cnt[v];
    const uint32_t base = row_sum(s_before[0][v]), first = row_sum(s_before[1][v]);
    const uint32_t off_tile = first + row_sum(v < (wave & ~(kParts - 1u)) ? of_v : 0u), off = first + row_sum(v < wave ? of_v : 0u);
    const uint32_t total = first + row_sum(of_v);
    uint32_t *to = M.tile_off + size_t(c) * kChunkStride;
    if (wave % kParts == 0 && lane == 0) to[tile % kTilesPerChunk] = off_tile;
    // the chunk's last workgroup with a tile completes its table: tiles past the end count as empty
    if (tile0 + kSmallTiles >= ntiles || tile0 % kTilesPerChunk + kSmallTiles == kTilesPerChunk) {
        for (uint32_t t = (tile0 % kTilesPerChunk) + kSmallTiles + threadIdx.x; t <= kTilesPerChunk; t += 64 * kSmallWaves) to[t] = total;
        if (threadIdx.x == 0) M.chunk_total[c] = total;
    }
    const uint32_t e0 = (tile0 * kParts + wave) * kPartElems;
    if (e0 >= n) return;
    WS &S = s_scratch[wave];
    const uintptr_t vbeg = reinterpret_cast<uintptr_t>(M.values), vend = vbeg + E * static_cast<uintptr_t>(M.nnz);
    const uintptr_t vaddr = vbeg + E * (uintptr_t(base) + off), a16 = vaddr & ~uintptr_t(15);
    const uint32_t shift = static_cast<uint32_t>(vaddr - a16) / E, nch = cnt ? ((shift + cnt) * E + 15) >> 4 : 0;
    const ValueSlice<E, WS::kStageRounds> slice(a16, nch, vbeg, vend);
    slice.ask(S.stage, lane);
    if (E == 1 && lane < 16) S.nibble_sel[lane] = nibble_selector(lane);
    if (lane < kPartWords) {
        S.words[lane] = word;
        S.start[lane] = incl - pc + shift;
    }
    slice.finish(S.stage, lane);
    wave_lds_sync();
    StoreSink<E, kAlignedOut, false, kPartElems> sink;
    sink.out = reinterpret_cast<uint8_t *>(M.dense) + size_t(e0) * E;
    sink.nvalid = n - e0 < kPartElems ? n - e0 : uint32_t(kPartElems);
#pragma unroll
    for (int k = 0; k < Shape<E>::kSteps / kParts; ++k) expand_step<E, kPartElems>(S, k, lane, sink);
}

// This lane's 64 bits of a segment of `nbits` (<= 4096) bits that starts at an arbitrary
// bit position e of the bitmap: bits e + 64*lane .. +63, funnelled out of two neighbouring
// words, with everything past the segment (or past the bitmap) cleared.
__device__ __forceinline__ uint64_t segment_word(const uint64_t *bitmap, int64_t nwords, int64_t e,
                                                 uint32_t nbits, uint32_t lane) {
    // Both loads are unconditional, from indices clamped into the bitmap, and the cases are
    // sorted out with selects afterwards: under a test each load would be waited for on the
    // spot, and a caller that fetches the next segment's word ahead would gain nothing.
    const int64_t w0 = (e >> 6) + lane;
    const uint32_t bs = static_cast<uint32_t>(e & 63);
    const int64_t last = nwords - 1;  // nwords >= 1: the callers have at least one element
    const uint64_t lo = bitmap[w0 < last ? w0 : last];
    const uint64_t hi = bitmap[w0 + 1 < last ? w0 + 1 : last];
    uint64_t word = (w0 < nwords ? lo : 0) >> bs;
    word |= ((w0 + 1 < nwords ? hi : 0) << 1) << (63 - bs);  // hi << (64 - bs), and nothing when bs is 0
    const uint32_t have = lane * 64 < nbits ? nbits - lane * 64 : 0u;  // bits of this lane that belong to the segment
    if (have < 64) word &= (uint64_t(1) << have) - 1;
    return word;
}

// ---------------------------------------------------------------- kernel 2b: selected rows

struct RowsParams {
    const uint64_t *bitmap;
    const void *values;
    void *out;                   // nsel x cols
    const int64_t *row_offsets;  // rows + 1
    const int64_t *sel;          // nsel row indices
    int64_t rows, cols, nnz, nsel;
    uint32_t segs;               // ceil(cols / 4096) tiles per row
};

// Row-subset decompression (the selective load of Section 4.2): output row r is row
// sel[r] of the matrix.  One wave per (selected row, 4096-column segment).  The segment
// starts at an arbitrary bit position, so a lane's 64 bits are funnelled out of two
// neighbouring bitmap words; its first value is row_offsets[row] plus the 1 bits of the
// row's earlier segments, counted here from the bitmap.
template <int E, bool kAlignedOut, int kCap = kTileElems>
__global__ __launch_bounds__(64) void endor_expand_rows_kernel(RowsParams R) {
    __shared__ WaveScratch<E, kCap> s_scratch;
    const uint32_t lane = threadIdx.x;
    // (the block's number, once all parameters are in registers: a wait for them less when the row is known)
    uint32_t block;
    asm("s_mov_b32 %0, %1"
        : "=s"(block)
        : "s"(blockIdx.x), "s"(R.bitmap), "s"(R.values), "s"(R.out), "s"(R.row_offsets), "s"(R.sel), "s"(R.rows), "s"(R.cols), "s"(R.nnz), "s"(R.segs));
    const int64_t r = block / R.segs;
    const uint32_t g = block % R.segs;
    const int64_t i = R.sel[r];
    if (i < 0 || i >= R.rows) return;  // an index outside the matrix leaves its output row untouched

    const int64_t n = R.rows * R.cols;
    const int64_t nwords = (n + 63) >> 6;
    const int64_t row_bit = i * R.cols;                  // first bit of the row
    const int64_t e = row_bit + int64_t(g) * kTileElems;  // first bit of the segment
    const int64_t left = R.cols - int64_t(g) * kTileElems;
    const uint32_t nbits = left < kTileElems ? static_cast<uint32_t>(left) : uint32_t(kTileElems);

    // everything that depends on the row index only goes out together: the segment's own bits,
    // the row's first value, and the bitmap words before the segment
    const uint64_t word = segment_word(R.bitmap, nwords, e, nbits, lane);
    const uint64_t row_first = static_cast<uint64_t>(R.row_offsets[i]);

    // 1 bits of the row before this segment: words [row_bit>>6, e>>6], first and last partial.
    // A lane's share stays below 2^28; the total may not fit 32 bits for very wide rows, so
    // the two 16-bit halves are summed across the wave separately.  Two words per lane and
    // pass, loaded unconditionally (an index past the last word reads the last again and is
    // dropped), so that a pass is one trip to memory.
    uint64_t before = 0;
    {
        uint32_t part = 0;
        const int64_t wa = row_bit >> 6, wb = e >> 6;  // wb < nwords: e is a position of the matrix
        for (int64_t w0 = wa; w0 <= wb; w0 += 128) {
            uint64_t x[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t w = w0 + 64 * k + lane;
                x[k] = R.bitmap[w <= wb ? w : wb];
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t w = w0 + 64 * k + lane;
                uint64_t y = w <= wb ? x[k] : 0;
                if (w == wa) y &= ~uint64_t(0) << (row_bit & 63);
                if (w == wb) y &= (uint64_t(1) << (e & 63)) - 1;
                part += __popcll(y);
            }
        }
        before = uint64_t(wave_sum(part & 0xffffu)) + (uint64_t(wave_sum(part >> 16)) << 16);
    }
    const uint32_t cnt = wave_sum(__popcll(word));

    const uintptr_t vbeg = reinterpret_cast<uintptr_t>(R.values);
    const uintptr_t vend = vbeg + E * static_cast<uintptr_t>(R.nnz);
    const uint64_t first = row_first + before;
    StoreSink<E, kAlignedOut, false> sink;
    sink.out = reinterpret_cast<uint8_t *>(R.out) + (r * R.cols + int64_t(g) * kTileElems) * E;
    sink.nvalid = nbits;
    expand_tile<E, kCap>(s_scratch, lane, word, vbeg + E * first, cnt, vbeg, vend, sink);
}

// ---------------------------------------------------------------- kernel 2c: selected columns

struct ColsParams {
    const uint64_t *bitmap;
    const void *values;
    void *out;                   // rows x nsel
    const int64_t *row_offsets;  // rows + 1
    const int64_t *sel;          // nsel column indices
    int64_t rows, cols, nnz, nsel;
    uint32_t stage_units;        // 16-byte units the staging area holds, one of them spare (kStaged)
};

// 64 bits of row-aligned "virtual word" k of a row that starts at bit row_bit: bits
// row_bit + 64k .. +63, clipped to the row's `cols` bits and to the bitmap.
__device__ __forceinline__ uint64_t row_word(const uint64_t *bitmap, int64_t nwords, int64_t row_bit,
                                             int64_t cols, int64_t k) {
    const int64_t e = row_bit + 64 * k;
    const int64_t w0 = e >> 6;
    const uint32_t bs = static_cast<uint32_t>(e & 63);
    uint64_t word = (w0 < nwords ? bitmap[w0] : 0) >> bs;
    if (bs != 0) word |= (w0 + 1 < nwords ? bitmap[w0 + 1] : 0) << (64 - bs);
    const int64_t rem = cols - 64 * k;
    if (rem < 64) word &= (uint64_t(1) << rem) - 1;
    return word;
}

// Column-subset decompression (the other half of Section 4.2's selective load: the columns
// of a down projection that belong to active neurons).  out[i][q] = W[i][sel[q]].  One
// workgroup per row.  It first lays the row's bitmap out in LDS as 32-bit pieces, each with
// the number of the row's 1 bits before it; a query is then one coalesced load of its
// column index, one LDS read of such a pair and a handful of 32-bit operations for
//     rank = row_offsets[i] + before[piece] + popcount(bits of the piece below the column),
// and one 2-byte load of values[rank] (or a zero).  Queries are taken several at a time so that
// their loads are in flight together.
//
// kStaged: the row's whole value slice goes straight to LDS (no registers) while the bitmap is
// worked on, and the queries read it there; the host says when that pays.
//
// kStore: how the output is stored (Store).  kQ: queries per thread and round.
template <int E, bool kStaged, Store kStore, int kQ>
__global__ __launch_bounds__(kBlock) void endor_gather_cols_kernel(ColsParams C) {
    typedef std::conditional_t<E == 2, uint16_t, uint8_t> Elem;
    // [np] pairs (32 bits of the row's bitmap, 1 bits of the row before them) | staged values
    extern __shared__ __attribute__((aligned(16))) uint32_t s_dyn[];
    __shared__ uint32_t s_wave[2][kWaves];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const int64_t i = blockIdx.x;
    const int64_t nwords = (C.rows * C.cols + 63) >> 6;
    const int64_t row_bit = i * C.cols;
    const uint32_t nvw = static_cast<uint32_t>((C.cols + 63) >> 6);

    // The row's values, on their way to LDS while the bitmap is worked on: 16-byte units from the
    // boundary at or below the first one.  A row that does not fit, or whose units reach over an end of
    // the array, is gathered from memory.
    // Staged: the row's entry and the next one in one trip; for the last row, which has no next one, the one
    // before (a single row is never staged).
    const bool last_row = i + 1 == C.rows;
    const int64_t *entry = C.row_offsets + (kStaged && last_row ? i - 1 : i);
    const int64_t entry0 = entry[0], entry1 = kStaged ? entry[1] : 0;
    const int64_t row_first = kStaged && last_row ? entry1 : entry0;
    const uintptr_t vaddr = reinterpret_cast<uintptr_t>(C.values) + E * static_cast<uintptr_t>(row_first);
    const uint8_t *stage = reinterpret_cast<const uint8_t *>(s_dyn + 4 * nvw);
    uint32_t staged = 0;  // of the row's values, those in LDS
    if (kStaged) {
        // how much is staged; a row that turns out to have more values is gathered after all
        const int64_t row_next = last_row ? C.nnz : entry1;
        const uintptr_t vbeg = reinterpret_cast<uintptr_t>(C.values), vend = vbeg + E * static_cast<uintptr_t>(C.nnz);
        const uintptr_t a16 = vaddr & ~uintptr_t(15);
        const uint64_t count = row_first >= 0 && row_next > row_first && row_next <= C.nnz ? static_cast<uint64_t>(row_next - row_first) : 0;
        const uint64_t units = ((vaddr - a16) + E * count + 15) >> 4;
        if (count != 0 && units < C.stage_units && a16 >= vbeg && a16 + 16 * units <= vend) {  // workgroup-uniform
            staged = static_cast<uint32_t>(count);
            u32x4 *to = reinterpret_cast<u32x4 *>(s_dyn + 4 * nvw);
            for (uint32_t u0 = 64 * wave; u0 < units; u0 += kBlock)
                if (u0 + lane < units) load_to_lds16(reinterpret_cast<const u32x4 *>(a16) + u0 + lane, to + u0);
        }
        stage += vaddr - a16;
    }

    // kLines: a row's queries are counted from the start of the line that its output begins in; the `early` numbers
    // before its first are no queries.
    uint8_t *row_out = static_cast<uint8_t *>(C.out) + E * i * C.nsel;
    const uint32_t early = kStore == Store::kLines ? static_cast<uint32_t>(reinterpret_cast<uintptr_t>(row_out) % kLineBytes / E) : 0;
    const int64_t nsel = C.nsel + early;
    const int64_t *sel = C.sel - early;
    row_out -= E * early;

    // first round of column indices: in flight during the bitmap work
    int64_t c[kQ];
#pragma unroll
    for (int u = 0; u < kQ; ++u) {
        const int64_t q = u * kBlock + threadIdx.x;
        c[u] = q < nsel && (kStore != Store::kLines || u || threadIdx.x >= early) ? sel[q] : -1;
    }

    // scan of the word popcounts, kBlock words per round: wave scan, then the waves' totals
    // through LDS (two alternating slots, so one barrier per round is enough)
    uint32_t carry = 0;
    for (uint32_t k0 = 0, round = 0; k0 < nvw; k0 += kBlock, ++round) {
        const uint32_t k = k0 + threadIdx.x;
        const uint64_t w = k < nvw ? row_word(C.bitmap, nwords, row_bit, C.cols, k) : 0;
        const uint32_t lo = static_cast<uint32_t>(w), hi = static_cast<uint32_t>(w >> 32);
        const uint32_t pc = __popc(lo) + __popc(hi);
        const uint32_t incl = wave_inclusive_scan(pc);
        if (lane == 63) s_wave[round & 1][wave] = incl;
        __syncthreads();
        uint32_t before = carry;
#pragma unroll
        for (uint32_t v = 0; v < kWaves; ++v) {
            const uint32_t t = s_wave[round & 1][v];
            before += v < wave ? t : 0;
            carry += t;
        }
        if (k < nvw) {
            const uint32_t excl = before + incl - pc;
            u32x4 pairs;
            pairs.x = lo;
            pairs.y = excl;
            pairs.z = hi;
            pairs.w = excl + __popc(lo);
            reinterpret_cast<u32x4 *>(s_dyn)[k] = pairs;
        }
    }
    if (kStaged) {
        wait_loads_to_lds();
        // carry: the row's 1 bits.  More than are staged: the next entry of row_offsets is not this row's end.
        // (Costs 0.5 of 63 us on a tenth of 8192 x 28672; to find it out query by query cost 1 us.)
        if (static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(carry))) > staged) staged = 0;
    }
    __syncthreads();

    // values from the row's first to the end of the array; none if the offset is not inside it
    const uint64_t room = (row_first >= 0 && row_first <= C.nnz) ? static_cast<uint64_t>(C.nnz - row_first) : 0;
    const uint8_t *row_values = static_cast<const uint8_t *>(C.values) + E * row_first;
    const uint64_t ucols = static_cast<uint64_t>(C.cols);
    // The queries.  kFromLds: the row's values are staged.  (Two loops, not one with a test: the test cost the
    // staged form 15 % and the gather up to 5 %.)
    auto answer = [&](auto from_lds) {
        constexpr bool kFromLds = decltype(from_lds)::value;
        for (int64_t q0 = 0; q0 < nsel; q0 += kQ * kBlock) {
            int64_t cn[kQ];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {  // the next round's indices
                const int64_t q = q0 + (kQ + u) * kBlock + threadIdx.x;
                cn[u] = q < nsel ? sel[q] : -1;
            }
            uint32_t v[kQ];
            bool live[kQ], hit[kQ];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                // an index outside the matrix (or past nsel) leaves its output column untouched
                live[u] = static_cast<uint64_t>(c[u]) < ucols;
                const uint32_t cc = live[u] ? static_cast<uint32_t>(c[u]) : 0u;
                const uint64_t pair = reinterpret_cast<const uint64_t *>(s_dyn)[cc >> 5];
                const uint32_t piece = static_cast<uint32_t>(pair);
                const uint32_t b = cc & 31;
                const uint32_t r = static_cast<uint32_t>(pair >> 32) + __popc(piece & ((1u << b) - 1));  // rank inside the row
                hit[u] = live[u] && ((piece >> b) & 1) != 0 && r < room;
                if (kFromLds) {
                    // r is at most the row's 1 bits: one value past the staged ones, in the area's spare unit
                    v[u] = (E == 2) ? uint32_t(reinterpret_cast<const uint16_t *>(stage)[r]) : uint32_t(stage[r]);
                    continue;
                }
                // The load itself is unconditional (a query without a value reads the first selected
                // index instead and drops it): with the load under the test, the compiler waits for
                // memory after every query and every store, one at a time.
                const uint8_t *at = hit[u] ? row_values + size_t(E) * r : reinterpret_cast<const uint8_t *>(C.sel);
                v[u] = (E == 2) ? uint32_t(*reinterpret_cast<const uint16_t *>(at)) : uint32_t(*at);
            }
#pragma unroll
            for (int u = 0; u < kQ; ++u) v[u] = hit[u] ? v[u] : 0u;
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                const int64_t q = q0 + u * kBlock + threadIdx.x;
                if (live[u]) {
                    Elem *at = reinterpret_cast<Elem *>(row_out) + q;
                    if (kStore != Store::kPlain)
                        __builtin_nontemporal_store(static_cast<Elem>(v[u]), at);
                    else
                        *at = static_cast<Elem>(v[u]);
                }
                c[u] = cn[u];
            }
        }
    };
    if (kStaged && staged)  // workgroup-uniform
        answer(std::true_type{});
    else
        answer(std::false_type{});
}

// ---------------------------------------------------------------- device-side compression

// 16 bytes of the dense matrix: elements [le, le + kLaneElems) of a tile that has
// `nvalid` elements; elements past the end read as zero.
template <int E, bool kAlignedIn>
__device__ __forceinline__ u32x4 load_dense16(const uint8_t *tile_in, uint32_t le, uint32_t nvalid) {
    if (kAlignedIn && le + Shape<E>::kLaneElems <= nvalid)
        return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(tile_in + size_t(le) * E));
    // unconditional loads, from an element that exists, sorted out afterwards: one trip, not one for every element
    uint32_t v[Shape<E>::kLaneElems];
#pragma unroll
    for (int j = 0; j < Shape<E>::kLaneElems; ++j) {
        const uint32_t at = le + j < nvalid ? le + j : 0u;
        v[j] = (E == 2) ? uint32_t(reinterpret_cast<const uint16_t *>(tile_in)[at]) : uint32_t(tile_in[at]);
        v[j] = le + j < nvalid ? v[j] : 0u;
    }
    uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < Shape<E>::kLaneElems; ++j) d[(E * j) >> 2] |= v[j] << (8 * ((E * j) & 3));
    u32x4 r;
    r.x = d[0];
    r.y = d[1];
    r.z = d[2];
    r.w = d[3];
    return r;
}

// A lane's kSteps 16-byte pieces of a tile of the dense matrix.  A whole, aligned tile is one
// wave-uniform case with unconditional loads, all issued before the first is used (under a
// per-piece bounds test the compiler waits after every load); only the ragged last tile and
// unaligned inputs go piece by piece.
template <int E, bool kAlignedIn>
__device__ __forceinline__ void load_dense_tile(const uint8_t *tile_in, uint32_t lane, uint32_t nvalid,
                                                u32x4 (&d)[Shape<E>::kSteps]) {
    using Sh = Shape<E>;
    if (kAlignedIn && nvalid == kTileElems) {
#pragma unroll
        for (int k = 0; k < Sh::kSteps; ++k)
            d[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(tile_in) + k * 64 + lane);
    } else {
#pragma unroll
        for (int k = 0; k < Sh::kSteps; ++k) d[k] = load_dense16<E, kAlignedIn>(tile_in, (k * 64 + lane) * Sh::kLaneElems, nvalid);
    }
}

// bit j = (element j of the 16 bytes is not the all-zero pattern)
template <int E>
__device__ __forceinline__ uint32_t nonzero_bits(u32x4 d) {
    const uint32_t dd[4] = {d.x, d.y, d.z, d.w};
    uint32_t bits = 0;
    if constexpr (E == 2) {  // both halves of a dword at once; a compare and a select each where the compiler sees the minimum
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t ones;
            asm("v_pk_min_u16 %0, %1, %2" : "=v"(ones) : "v"(dd[i]), "s"(0x00010001u));
            bits |= ones << (2 * i);
        }
        return (bits | bits >> 15) & 0xffu;
    }
#pragma unroll
    for (int j = 0; j < Shape<E>::kLaneElems; ++j) {
        const uint32_t v = (dd[(E * j) >> 2] >> (8 * ((E * j) & 3))) & ((E == 2) ? 0xffffu : 0xffu);
        bits |= (v != 0 ? 1u : 0u) << j;
    }
    return bits;
}

struct CompressParams {
    const void *dense;
    uint64_t *bitmap;
    void *values;
    int64_t n;
    int64_t capacity;  // elements `values` has room for
    int64_t *nnz_out;  // where the number of non-zeros goes
    int64_t *row_offsets;  // rows + 1 entries, or null
    int64_t rows, cols;
    MatParams table;   // chunk_total / tile_off of this matrix (bitmap, n filled in as well)
};

// Algorithm 1, step 1 on the device: the position bitmap, and each tile's count in its slot of the
// offset table (the table then comes from a scan of the counts, 5 us, instead of a second pass over
// the bitmap, 6.5 us on 28672 x 8192).  One wave per tile; the lane
// bit groups of the 4096 elements are assembled into 64-bit words through LDS.
template <int E, bool kAlignedIn>
__global__ __launch_bounds__(64) void endor_mask_kernel(CompressParams C) {
    using Sh = Shape<E>;
    __shared__ uint64_t s_words[kTileWords];
    const uint32_t lane = threadIdx.x;
    const int64_t tile = blockIdx.x;
    const int64_t e0 = tile * kTileElems;
    const int64_t left = C.n - e0;
    const uint32_t nvalid = left < kTileElems ? static_cast<uint32_t>(left) : uint32_t(kTileElems);
    const uint8_t *tile_in = reinterpret_cast<const uint8_t *>(C.dense) + e0 * E;
    u32x4 d[Sh::kSteps];
    load_dense_tile<E, kAlignedIn>(tile_in, lane, nvalid, d);
#pragma unroll
    for (int k = 0; k < Sh::kSteps; ++k) {
        const uint32_t bits = nonzero_bits<E>(d[k]);
        if (E == 2)
            reinterpret_cast<uint8_t *>(s_words)[k * 64 + lane] = static_cast<uint8_t>(bits);
        else
            reinterpret_cast<uint16_t *>(s_words)[k * 64 + lane] = static_cast<uint16_t>(bits);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int64_t w = tile * kTileWords + lane;
    const uint64_t word = s_words[lane];
    // streamed, like the values (endor_pack_kernel); pad bits are zero: elements past n read as zero
    if (w < ((C.n + 63) >> 6)) __builtin_nontemporal_store(word, &C.bitmap[w]);
    const uint32_t count = wave_sum(__popcll(word));
    if (lane == 0) C.table.tile_off[size_t(tile / kTilesPerChunk) * kChunkStride + tile % kTilesPerChunk] = count;
}

// The tile counts endor_mask_kernel left in the table, turned into the table: one workgroup per chunk.
__global__ __launch_bounds__(kTilesPerChunk) void endor_scan_counts_kernel(MatParams M) {
    __shared__ uint32_t s_wave[kTilesPerChunk / 64];
    const uint32_t c = blockIdx.x, t = threadIdx.x, wave = t >> 6;
    uint32_t *to = M.tile_off + size_t(c) * kChunkStride;
    const int64_t ntiles = (M.n + kTileElems - 1) / kTileElems;
    const uint32_t cnt = int64_t(c) * kTilesPerChunk + t < ntiles ? to[t] : 0u;  // tiles past the end count as empty
    const uint32_t incl = wave_inclusive_scan(cnt);
    if ((t & 63) == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t v = 0; v < wave; ++v) before += s_wave[v];
    to[t] = before + incl - cnt;
    if (t == kTilesPerChunk - 1) {
        to[kTilesPerChunk] = before + incl;
        M.chunk_total[c] = before + incl;
    }
}

// Algorithm 1, step 2 on the device: pack the non-zero elements of one tile at the
// tile's offset.  The values are scattered into LDS at rank order and written out in
// 16-byte units; the units a tile shares with its neighbours (first and last) are
// written element by element so that each element of `values` has exactly one writer.
template <int E, bool kAlignedIn>
__global__ __launch_bounds__(64) void endor_pack_kernel(CompressParams C) {
    using Sh = Shape<E>;
    __shared__ WaveScratch<E> S;
    const uint32_t lane = threadIdx.x;
    const int64_t tile = blockIdx.x;
    // the tile's elements first: their loads are in flight while the table is looked up
    const int64_t e0 = tile * kTileElems;
    const int64_t left = C.n - e0;
    const uint32_t nvalid = left < kTileElems ? static_cast<uint32_t>(left) : uint32_t(kTileElems);
    const uint8_t *tile_in = reinterpret_cast<const uint8_t *>(C.dense) + e0 * E;
    u32x4 d[Sh::kSteps];
    load_dense_tile<E, kAlignedIn>(tile_in, lane, nvalid, d);

    const MatParams &M = C.table;
    const uint32_t c = static_cast<uint32_t>(tile / kTilesPerChunk);
    const uint32_t tl = static_cast<uint32_t>(tile % kTilesPerChunk);
    const uint32_t *tile_off = M.tile_off + size_t(c) * kChunkStride + tl;
    const uint32_t o0 = tile_off[0];
    uint32_t cnt = tile_off[1] - o0;
    cnt = cnt > kTileElems ? kTileElems : cnt;
    const uint64_t first = chunk_base(M.chunk_total, c, lane) + o0;  // index of the tile's first value
    if (e0 + kTileElems >= C.n && lane == 0) {  // the last tile knows the total
        *C.nnz_out = static_cast<int64_t>(first + cnt);
        if (C.row_offsets) C.row_offsets[C.rows] = static_cast<int64_t>(first + cnt);
    }

    const uintptr_t vbase = reinterpret_cast<uintptr_t>(C.values);
    const uintptr_t vaddr = vbase + E * first;
    const uintptr_t a16 = vaddr & ~uintptr_t(15);
    const uint32_t shift = static_cast<uint32_t>(vaddr - a16) / E;

    // word popcounts from the data itself (the same bits endor_mask_kernel wrote)
    uint32_t bits[Sh::kSteps];
#pragma unroll
    for (int k = 0; k < Sh::kSteps; ++k) {
        bits[k] = nonzero_bits<E>(d[k]);
        if (E == 2)
            reinterpret_cast<uint8_t *>(S.words)[k * 64 + lane] = static_cast<uint8_t>(bits[k]);
        else
            reinterpret_cast<uint16_t *>(S.words)[k * 64 + lane] = static_cast<uint16_t>(bits[k]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint64_t word = S.words[lane];
    const uint32_t pc = __popcll(word);
    const uint32_t incl = wave_inclusive_scan(pc);
    S.start[lane] = incl - pc + shift;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // the rows that start in this tile begin with the non-zeros before it plus those of its earlier
    // words (a separate kernel that looked every row start up took 7 us on 28672 rows)
    if (C.row_offsets) {  // wave-uniform
        int64_t i = (e0 + C.cols - 1) / C.cols + lane;  // lane 0: the first such row
        for (; i < C.rows; i += 64) {
            const int64_t le = i * C.cols - e0;
            if (le >= kTileElems) break;
            const uint32_t wi = static_cast<uint32_t>(le) >> 6;
            const uint32_t in_tile = S.start[wi] - shift + __popcll(S.words[wi] & ((uint64_t(1) << (le & 63)) - 1));
            C.row_offsets[i] = static_cast<int64_t>(first + in_tile);
        }
    }

    // scatter the non-zero elements into LDS in rank order
#pragma unroll
    for (int k = 0; k < Sh::kSteps; ++k) {
        const uint32_t wi = k * Sh::kLaneElems + lane / Sh::kLanesPerWord;
        const uint64_t w = S.words[wi];
        const uint32_t sh = (lane % Sh::kLanesPerWord) * Sh::kLaneElems;
        const uint32_t s = S.start[wi] + __popcll(w & ((uint64_t(1) << sh) - 1));
        const uint32_t dd[4] = {d[k].x, d[k].y, d[k].z, d[k].w};
#pragma unroll
        for (int j = 0; j < Sh::kLaneElems; ++j) {
            if ((bits[k] >> j) & 1u) {
                const uint32_t idx = s + __popc(bits[k] & ((1u << j) - 1));
                const uint32_t v = dd[(E * j) >> 2] >> (8 * ((E * j) & 3));
                if (E == 2)
                    reinterpret_cast<uint16_t *>(S.stage)[idx] = static_cast<uint16_t>(v);
                else
                    reinterpret_cast<uint8_t *>(S.stage)[idx] = static_cast<uint8_t>(v);
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // write the slice out: elements [shift, shift + cnt) of the staging area go to
    // values[first, first + cnt), never past `capacity`.  Streamed stores: what goes through the memory-side
    // cache pushes earlier writes out of it between this call's reads.  28672 x 8192, a call whose outputs are
    // new buffers, a tenth / three tenths / half / nine tenths kept: 201 / 232 / 239 / 276 us without, 199 / 209 /
    // 219 / 257 with (into the buffer of the call before, which that cache still holds, half kept: 215 / 220).
    const uint32_t nch = cnt ? (((shift + cnt) * E + 15) >> 4) : 0;
    const int64_t room = C.capacity - static_cast<int64_t>(first);  // elements this tile may write
    for (uint32_t ch = lane; ch < nch; ch += 64) {
        const uint32_t el0 = ch * Sh::kLaneElems;  // staging index of the unit's first element
        const bool inside = el0 >= shift && el0 + Sh::kLaneElems <= shift + cnt &&
                            static_cast<int64_t>(el0 + Sh::kLaneElems - shift) <= room;
        if (inside) {
            __builtin_nontemporal_store(S.stage[ch], global_ptr_mut<u32x4>(a16 + 16 * uintptr_t(ch)));
        } else {
#pragma unroll
            for (int j = 0; j < Sh::kLaneElems; ++j) {
                const uint32_t el = el0 + j;
                if (el >= shift && el < shift + cnt && static_cast<int64_t>(el - shift) < room) {
                    if (E == 2)
                        global_ptr_mut<uint16_t>(a16)[el] = reinterpret_cast<const uint16_t *>(S.stage)[el];
                    else
                        global_ptr_mut<uint8_t>(a16)[el] = reinterpret_cast<const uint8_t *>(S.stage)[el];
                }
            }
        }
    }
}

}  // namespace

#include "endor_compress_pass.h"
#include "endor_cols_stream.h"

namespace {

// total number of 1 bits of a matrix whose table has been built: one wave
__global__ __launch_bounds__(64) void endor_total_kernel(MatParams M, int64_t *__restrict__ nnz_out) {
    const uint64_t total = chunk_base(M.chunk_total, M.nchunks, threadIdx.x);
    if (threadIdx.x == 0) *nnz_out = static_cast<int64_t>(total);
}

// Check mode: one wave per matrix compares nnz with the number of 1 bits the table records.
__global__ __launch_bounds__(64) void endor_check_kernel(BatchParams P, int32_t *__restrict__ status) {
    const MatParams &M = P.m[blockIdx.x];
    const uint64_t total = chunk_base(M.chunk_total, M.nchunks, threadIdx.x);
    if (threadIdx.x == 0)
        status[M.chunk_begin] = total == static_cast<uint64_t>(M.nnz) ? ENDOR_OK : ENDOR_ERR_NNZ_MISMATCH;
}

// ---------------------------------------------------------------- kernel 3: row offsets

// One wave per row start: rank(i*cols) = chunk start + tile offset + 1 bits of the
// tile's words below the position.  Entry `rows` is the total number of 1 bits.
__global__ __launch_bounds__(kBlock) void endor_row_offsets_kernel(MatParams M, int64_t rows, int64_t cols,
                                                                   int64_t *__restrict__ row_offsets) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const int64_t i = int64_t(blockIdx.x) * kWaves + wave;
    if (i > rows) return;
    const int64_t e = i * cols;  // == n for i == rows
    const int64_t ntiles = (M.n + kTileElems - 1) / kTileElems;
    int64_t tile = e >> 12;
    uint64_t rank;
    if (tile >= ntiles) {
        // position n when n is a multiple of the tile size: everything counts
        rank = chunk_base(M.chunk_total, M.nchunks, lane);
    } else {
        const uint32_t c = static_cast<uint32_t>(tile / kTilesPerChunk);
        const uint32_t tl = static_cast<uint32_t>(tile % kTilesPerChunk);
        rank = chunk_base(M.chunk_total, c, lane) + M.tile_off[size_t(c) * kChunkStride + tl];
        const int64_t w = tile * kTileWords + lane;
        const int64_t we = e >> 6;  // word holding position e
        uint64_t word = 0;
        if (w <= we) word = load_word_guarded(M.bitmap, w, M.n >> 6, static_cast<uint32_t>(M.n & 63));
        if (w == we) word &= (uint64_t(1) << (e & 63)) - 1;
        rank += wave_sum(__popcll(word));
    }
    if (lane == 0) row_offsets[i] = static_cast<int64_t>(rank);
}

// ---------------------------------------------------------------- host side

struct Group {
    BatchParams P;
    uint32_t chunks = 0;
    bool aligned_out = true;
    int64_t elems = 0, nnz = 0;  // totals over the group (launch heuristics only)
};

enum Need { kNeedBitmap = 1, kNeedValuesDense = 2 };

// Validate `count` matrices starting at the workspace offset *ws_off and fill one
// launch group.  Advances *ws_off past the slices it used.
endor_status fill_group(const endor_matrix *mats, int count, int need, int elem_bytes, char *ws,
                        size_t ws_bytes, size_t *ws_off, Group *g) {
    const uintptr_t elem_mask = static_cast<uintptr_t>(elem_bytes - 1);
    g->P.count = 0;
    for (int i = 0; i < ENDOR_MAX_BATCH; ++i) g->P.first_chunk[i] = 0xffffffffu;
    g->chunks = 0;
    g->aligned_out = true;
    g->elems = 0;
    g->nnz = 0;
    for (int i = 0; i < count; ++i) {
        const endor_matrix &m = mats[i];
        if (m.rows < 0 || m.cols < 0) return ENDOR_ERR_INVALID_ARG;
        if (!dims_ok(m.rows, m.cols)) return ENDOR_ERR_UNSUPPORTED;
        const int64_t n = m.rows * m.cols;
        if (n == 0) continue;
        if (!m.d_bitmap || (reinterpret_cast<uintptr_t>(m.d_bitmap) & 7)) return ENDOR_ERR_INVALID_ARG;
        if (need & kNeedValuesDense) {
            if (m.nnz < 0 || m.nnz > n) return ENDOR_ERR_INVALID_ARG;
            if (!m.d_dense || (reinterpret_cast<uintptr_t>(m.d_dense) & elem_mask)) return ENDOR_ERR_INVALID_ARG;
            if (m.nnz > 0 && (!m.d_values || (reinterpret_cast<uintptr_t>(m.d_values) & elem_mask)))
                return ENDOR_ERR_INVALID_ARG;
            if (reinterpret_cast<uintptr_t>(m.d_dense) & 15) g->aligned_out = false;
        }
        const uint32_t nc = chunks_of(n);
        const size_t need_bytes = workspace_bytes_n(n);
        if (*ws_off + need_bytes > ws_bytes) return ENDOR_ERR_BUFFER_TOO_SMALL;
        MatParams &M = g->P.m[g->P.count++];
        M.bitmap = reinterpret_cast<const uint64_t *>(m.d_bitmap);
        M.values = m.d_values;
        M.dense = m.d_dense;
        M.chunk_total = reinterpret_cast<uint32_t *>(ws + *ws_off);
        M.tile_off = reinterpret_cast<uint32_t *>(ws + *ws_off + align256(nc * sizeof(uint32_t)));
        M.n = n;
        M.nnz = m.nnz;
        M.chunk_begin = g->chunks;
        g->P.first_chunk[g->P.count - 1] = g->chunks;
        M.nchunks = nc;
        g->chunks += nc;
        g->elems += n;
        g->nnz += m.nnz;
        *ws_off += need_bytes;
    }
    return ENDOR_OK;
}

template <int E>
void launch_expand(const Group &g, hipStream_t s) {
    const dim3 grid(g.chunks * kTilesPerChunk);
    if (!g.aligned_out)
        hipLaunchKernelGGL((endor_expand_kernel<E, false, kTileElems, false>), grid, dim3(64), 0, s, g.P);
    else if (g.nnz * 5 < g.elems)  // fewer than one element in five kept: store-dominated
        hipLaunchKernelGGL((endor_expand_kernel<E, true, 1024, true>), grid, dim3(64), 0, s, g.P);
    else
        hipLaunchKernelGGL((endor_expand_kernel<E, true, kTileElems, false>), grid, dim3(64), 0, s, g.P);
}

// Largest matrix (in elements) that the one-kernel form takes: four chunks.  Measured back to back, half
// kept, fp16, two kernels / one: 1024 x 1024 10 / 5.9 us (as long as the host takes to enqueue it), 1448 x
// 1448 10.0 / 6.5, 2048 x 1500 11.3 / 7.5, 2048 x 2048 11.0 / 8.9, 2048 x 3000 11.2 / 13.9: every workgroup counts all of
// the bitmap before its tiles.  (With one wave per tile, 256 threads and 8-byte pieces: 1024 x 1024 6.7,
// 1024 x 2048 8.9.)
constexpr int64_t kSmallElems = int64_t(1) << 22;

template <int E>
void launch_small(const Group &g, hipStream_t s) {
    const MatParams &M = g.P.m[0];
    const dim3 grid(static_cast<unsigned>((M.n + kTileElems * kSmallTiles - 1) / (kTileElems * kSmallTiles)));
    if (g.aligned_out)
        hipLaunchKernelGGL((endor_decompress_small_kernel<E, true>), grid, dim3(64 * kSmallWaves), 0, s, M);
    else
        hipLaunchKernelGGL((endor_decompress_small_kernel<E, false>), grid, dim3(64 * kSmallWaves), 0, s, M);
}

// A bitmap that the kernels fetch from pinned host memory would cross the link once per workgroup of
// the one-kernel form, so that form is for device memory only.
bool in_device_memory(const void *p) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();  // not the launch's error
        return false;
    }
    return a.type == hipMemoryTypeDevice;
}

// The shared driver of every device entry point.  `mats` holds 16-bit typed pointers;
// with elem_bytes == 1 they are really 8-bit (endor_matrix_u8 has the same layout).
endor_status run_batch(const endor_matrix *mats, int count, void *d_workspace, size_t workspace_bytes,
                       void *stream, bool build, bool expand, int elem_bytes = 2) {
    if (count < 0 || (count > 0 && !mats)) return ENDOR_ERR_INVALID_ARG;
    if (count == 0) return ENDOR_OK;
    for (int i = 0; i < count; ++i) {
        if (mats[i].rows < 0 || mats[i].cols < 0) return ENDOR_ERR_INVALID_ARG;
        if (!dims_ok(mats[i].rows, mats[i].cols)) return ENDOR_ERR_UNSUPPORTED;
    }
    // a batch of empty matrices needs no workspace; anything else needs an aligned one
    if (endor_batch_workspace_bytes(mats, count) != 0 &&
        (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 255)))
        return ENDOR_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(d_workspace);
    const int need = kNeedBitmap | (expand ? kNeedValuesDense : 0);

    // validate everything before the first launch
    {
        size_t off = 0;
        Group g;
        for (int b = 0; b < count; b += ENDOR_MAX_BATCH) {
            const int nb = count - b < ENDOR_MAX_BATCH ? count - b : ENDOR_MAX_BATCH;
            endor_status st = fill_group(mats + b, nb, need, elem_bytes, ws, workspace_bytes, &off, &g);
            if (st != ENDOR_OK) return st;
        }
    }
    size_t off = 0;
    Group g;
    for (int b = 0; b < count; b += ENDOR_MAX_BATCH) {
        const int nb = count - b < ENDOR_MAX_BATCH ? count - b : ENDOR_MAX_BATCH;
        fill_group(mats + b, nb, need, elem_bytes, ws, workspace_bytes, &off, &g);
        if (g.chunks == 0) continue;
        if (build && expand && g.P.count == 1 && g.P.m[0].n <= kSmallElems && in_device_memory(g.P.m[0].bitmap)) {
            if (elem_bytes == 2)
                launch_small<2>(g, s);
            else
                launch_small<1>(g, s);
            if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
            continue;
        }
        if (build) {
            hipLaunchKernelGGL(endor_tile_offsets_kernel, dim3(g.chunks), dim3(kCountBlock), 0, s, g.P);
            if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
        }
        if (expand) {
            if (elem_bytes == 2)
                launch_expand<2>(g, s);
            else
                launch_expand<1>(g, s);
            if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
        }
    }
    return ENDOR_OK;
}

endor_matrix one_matrix(int64_t rows, int64_t cols, const uint8_t *d_bitmap, const uint16_t *d_values,
                        int64_t nnz, uint16_t *d_dense) {
    endor_matrix m;
    m.rows = rows;
    m.cols = cols;
    m.d_bitmap = d_bitmap;
    m.d_values = d_values;
    m.nnz = nnz;
    m.d_dense = d_dense;
    return m;
}

// Per-row offsets from a finished table.  A matrix without elements has no chunks and no tiles: all
// entries are 0 then.
int64_t row_offsets_blocks(int64_t rows) { return (rows + 1 + kWaves - 1) / kWaves; }
bool row_offsets_ok(int64_t rows) { return row_offsets_blocks(rows) <= 0x7fffffff; }

endor_status launch_row_offsets(const MatParams &M, int64_t rows, int64_t cols, int64_t *d_row_offsets, hipStream_t s) {
    if (!row_offsets_ok(rows)) return ENDOR_ERR_UNSUPPORTED;
    const unsigned blocks = static_cast<unsigned>(row_offsets_blocks(rows));
    hipLaunchKernelGGL(endor_row_offsets_kernel, dim3(blocks), dim3(kBlock), 0, s, M, rows, cols, d_row_offsets);
    return hipGetLastError() == hipSuccess ? ENDOR_OK : ENDOR_ERR_HIP;
}

}  // namespace

extern "C" size_t endor_workspace_bytes(int64_t rows, int64_t cols) {
    if (!dims_ok(rows, cols)) return 0;
    return workspace_bytes_n(rows * cols);
}

extern "C" size_t endor_batch_workspace_bytes(const endor_matrix *mats, int count) {
    if (count < 0 || (count > 0 && !mats)) return 0;
    size_t total = 0;
    for (int i = 0; i < count; ++i) {
        if (!dims_ok(mats[i].rows, mats[i].cols)) return 0;
        total += workspace_bytes_n(mats[i].rows * mats[i].cols);
    }
    return total;
}

extern "C" endor_status endor_build_offsets_batch(const endor_matrix *mats, int count, void *d_workspace,
                                                  size_t workspace_bytes, void *stream) {
    return run_batch(mats, count, d_workspace, workspace_bytes, stream, true, false);
}

extern "C" endor_status endor_decompress_batch(const endor_matrix *mats, int count, void *d_workspace,
                                               size_t workspace_bytes, void *stream) {
    return run_batch(mats, count, d_workspace, workspace_bytes, stream, true, true);
}

extern "C" endor_status endor_decompress_batch_with_offsets(const endor_matrix *mats, int count,
                                                            const void *d_workspace, size_t workspace_bytes,
                                                            void *stream) {
    return run_batch(mats, count, const_cast<void *>(d_workspace), workspace_bytes, stream, false, true);
}

extern "C" endor_status endor_check_batch(const endor_matrix *mats, int count, const void *d_workspace,
                                          size_t workspace_bytes, int32_t *d_status, void *stream) {
    if (count < 0 || (count > 0 && (!mats || !d_status))) return ENDOR_ERR_INVALID_ARG;
    if (count == 0) return ENDOR_OK;
    if (reinterpret_cast<uintptr_t>(d_status) & 3) return ENDOR_ERR_INVALID_ARG;
    for (int i = 0; i < count; ++i) {
        if (mats[i].rows < 0 || mats[i].cols < 0 || mats[i].nnz < 0) return ENDOR_ERR_INVALID_ARG;
        if (!dims_ok(mats[i].rows, mats[i].cols)) return ENDOR_ERR_UNSUPPORTED;
    }
    if (endor_batch_workspace_bytes(mats, count) != 0 &&
        (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 255)))
        return ENDOR_ERR_INVALID_ARG;
    if (endor_batch_workspace_bytes(mats, count) > workspace_bytes) return ENDOR_ERR_BUFFER_TOO_SMALL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *ws = const_cast<char *>(static_cast<const char *>(d_workspace));
    size_t off = 0;
    for (int b = 0; b < count; b += ENDOR_MAX_BATCH) {
        const int nb = count - b < ENDOR_MAX_BATCH ? count - b : ENDOR_MAX_BATCH;
        // one descriptor per matrix, empty ones included (they have no chunks and no 1 bits);
        // chunk_begin carries the matrix's index inside the batch for the kernel
        BatchParams P;
        P.count = nb;
        for (int i = 0; i < ENDOR_MAX_BATCH; ++i) P.first_chunk[i] = 0xffffffffu;  // not used by the check kernel
        for (int i = 0; i < nb; ++i) {
            const endor_matrix &m = mats[b + i];
            const int64_t n = m.rows * m.cols;
            MatParams &M = P.m[i];
            M = MatParams{};
            M.n = n;
            M.nnz = m.nnz;
            M.nchunks = n > 0 ? chunks_of(n) : 0;
            M.chunk_total = reinterpret_cast<uint32_t *>(ws + off);
            M.chunk_begin = static_cast<uint32_t>(b + i);
            off += n > 0 ? workspace_bytes_n(n) : 0;
        }
        hipLaunchKernelGGL(endor_check_kernel, dim3(nb), dim3(64), 0, s, P, d_status);
        if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    }
    return ENDOR_OK;
}

extern "C" endor_status endor_decompress(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                         const uint16_t *d_values, int64_t nnz, void *d_workspace,
                                         size_t workspace_bytes, uint16_t *d_dense, void *stream) {
    const endor_matrix m = one_matrix(rows, cols, d_bitmap, d_values, nnz, d_dense);
    return run_batch(&m, 1, d_workspace, workspace_bytes, stream, true, true);
}

extern "C" endor_status endor_decompress_with_offsets(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                                      const uint16_t *d_values, int64_t nnz,
                                                      const void *d_workspace, size_t workspace_bytes,
                                                      uint16_t *d_dense, void *stream) {
    const endor_matrix m = one_matrix(rows, cols, d_bitmap, d_values, nnz, d_dense);
    return run_batch(&m, 1, const_cast<void *>(d_workspace), workspace_bytes, stream, false, true);
}

extern "C" endor_status endor_build_offsets(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                            void *d_workspace, size_t workspace_bytes,
                                            int64_t *d_row_offsets, void *stream) {
    const endor_matrix m = one_matrix(rows, cols, d_bitmap, nullptr, 0, nullptr);
    if (d_row_offsets && (reinterpret_cast<uintptr_t>(d_row_offsets) & 7)) return ENDOR_ERR_INVALID_ARG;
    endor_status st = run_batch(&m, 1, d_workspace, workspace_bytes, stream, true, false);
    if (st != ENDOR_OK || !d_row_offsets) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t n = rows * cols;
    MatParams M{};
    if (n > 0) {
        size_t off = 0;
        Group g;
        fill_group(&m, 1, kNeedBitmap, 2, static_cast<char *>(d_workspace), workspace_bytes, &off, &g);
        M = g.P.m[0];
    }
    return launch_row_offsets(M, rows, cols, d_row_offsets, s);
}

// ---------------------------------------------------------------- no-allocation variant

namespace {

// The offset tables of endor_decompress_batch_static live here instead of in a caller's
// workspace.  Every device the library runs on holds its own copy of the array at its own
// address; in host code the array's name is only a handle for hipGetSymbolAddress, never
// a device address.
static __device__ __align__(256) unsigned char scratch[ENDOR_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, once known

// Device address of `scratch` on the current device, resolved on the first call per device.
endor_status static_scratch(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return ENDOR_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return ENDOR_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ENDOR_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return ENDOR_OK;
}

}  // namespace

extern "C" endor_status endor_decompress_batch_static(const endor_matrix *mats, int count, void *stream) {
    if (count < 0 || (count > 0 && !mats)) return ENDOR_ERR_INVALID_ARG;
    if (count == 0) return ENDOR_OK;
    for (int i = 0; i < count; ++i) {
        if (mats[i].rows < 0 || mats[i].cols < 0) return ENDOR_ERR_INVALID_ARG;
        if (!dims_ok(mats[i].rows, mats[i].cols)) return ENDOR_ERR_UNSUPPORTED;
    }
    const size_t need = endor_batch_workspace_bytes(mats, count);
    if (need > size_t(ENDOR_STATIC_SCRATCH_BYTES)) return ENDOR_ERR_BUFFER_TOO_SMALL;
    void *ws = nullptr;
    const endor_status st = static_scratch(&ws);
    if (st != ENDOR_OK) return st;
    // Nothing in the table has to start at zero: the tile-offset kernel writes every entry
    // of every chunk of this batch before the expand kernel reads it.
    return run_batch(mats, count, ws, size_t(ENDOR_STATIC_SCRATCH_BYTES), stream, true, true);
}

// ---------------------------------------------------------------- 8-bit elements (Section 4.2)

static_assert(sizeof(endor_matrix_u8) == sizeof(endor_matrix), "same descriptor layout for both widths");

extern "C" endor_status endor_decompress_u8(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                            const uint8_t *d_values, int64_t nnz, void *d_workspace,
                                            size_t workspace_bytes, uint8_t *d_dense, void *stream) {
    const endor_matrix m = one_matrix(rows, cols, d_bitmap, reinterpret_cast<const uint16_t *>(d_values), nnz,
                                      reinterpret_cast<uint16_t *>(d_dense));
    return run_batch(&m, 1, d_workspace, workspace_bytes, stream, true, true, 1);
}

extern "C" endor_status endor_decompress_u8_with_offsets(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                                         const uint8_t *d_values, int64_t nnz,
                                                         const void *d_workspace, size_t workspace_bytes,
                                                         uint8_t *d_dense, void *stream) {
    const endor_matrix m = one_matrix(rows, cols, d_bitmap, reinterpret_cast<const uint16_t *>(d_values), nnz,
                                      reinterpret_cast<uint16_t *>(d_dense));
    return run_batch(&m, 1, const_cast<void *>(d_workspace), workspace_bytes, stream, false, true, 1);
}

extern "C" endor_status endor_decompress_batch_u8(const endor_matrix_u8 *mats, int count, void *d_workspace,
                                                  size_t workspace_bytes, void *stream) {
    return run_batch(reinterpret_cast<const endor_matrix *>(mats), count, d_workspace, workspace_bytes, stream,
                     true, true, 1);
}

extern "C" endor_status endor_decompress_batch_u8_with_offsets(const endor_matrix_u8 *mats, int count,
                                                               const void *d_workspace, size_t workspace_bytes,
                                                               void *stream) {
    return run_batch(reinterpret_cast<const endor_matrix *>(mats), count, const_cast<void *>(d_workspace),
                     workspace_bytes, stream, false, true, 1);
}

// ---------------------------------------------------------------- selected rows (Section 4.2)

namespace {

endor_status run_rows(int elem_bytes, int64_t rows, int64_t cols, const uint8_t *d_bitmap, const void *d_values,
                      int64_t nnz, const int64_t *d_row_offsets, const int64_t *d_sel, int64_t nsel, void *d_out,
                      void *stream) {
    if (rows < 0 || cols < 0 || nsel < 0 || nnz < 0) return ENDOR_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return ENDOR_ERR_UNSUPPORTED;
    if (nsel == 0 || cols == 0) return ENDOR_OK;
    if (nsel > kMaxElems / cols) return ENDOR_ERR_UNSUPPORTED;
    const uintptr_t em = static_cast<uintptr_t>(elem_bytes - 1);
    if (nnz > rows * cols) return ENDOR_ERR_INVALID_ARG;
    if (!d_bitmap || (reinterpret_cast<uintptr_t>(d_bitmap) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (nnz > 0 && (!d_values || (reinterpret_cast<uintptr_t>(d_values) & em))) return ENDOR_ERR_INVALID_ARG;
    if (!d_row_offsets || (reinterpret_cast<uintptr_t>(d_row_offsets) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (!d_sel || (reinterpret_cast<uintptr_t>(d_sel) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (!d_out || (reinterpret_cast<uintptr_t>(d_out) & em)) return ENDOR_ERR_INVALID_ARG;
    RowsParams R;
    R.bitmap = reinterpret_cast<const uint64_t *>(d_bitmap);
    R.values = d_values;
    R.out = d_out;
    R.row_offsets = d_row_offsets;
    R.sel = d_sel;
    R.rows = rows;
    R.cols = cols;
    R.nnz = nnz;
    R.nsel = nsel;
    R.segs = static_cast<uint32_t>((cols + kTileElems - 1) / kTileElems);
    const int64_t blocks = nsel * R.segs;
    if (blocks > 0x7fffffff) return ENDOR_ERR_UNSUPPORTED;
    // every segment start (r*cols + g*4096 elements) is 16-byte aligned iff the row pitch is
    const bool aligned = (reinterpret_cast<uintptr_t>(d_out) & 15) == 0 && (cols * elem_bytes) % 16 == 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const dim3 grid(static_cast<unsigned>(blocks));
    // A selection is usually small (Section 4.2: the rows of the active neurons), so the kernel
    // lives on how many waves a compute unit holds at once: when no more than 9 elements in 16 are
    // kept overall, a staging area of 2304 values (a tile with more takes the step-by-step path)
    // lets 29 waves share a unit instead of 17.
    const bool small_stage = nnz <= (rows * cols / 16) * 9;
    if (elem_bytes == 2) {
        if (aligned && small_stage)
            hipLaunchKernelGGL((endor_expand_rows_kernel<2, true, 2304>), grid, dim3(64), 0, s, R);
        else if (aligned)
            hipLaunchKernelGGL((endor_expand_rows_kernel<2, true>), grid, dim3(64), 0, s, R);
        else
            hipLaunchKernelGGL((endor_expand_rows_kernel<2, false>), grid, dim3(64), 0, s, R);
    } else {
        if (aligned)
            hipLaunchKernelGGL((endor_expand_rows_kernel<1, true>), grid, dim3(64), 0, s, R);
        else
            hipLaunchKernelGGL((endor_expand_rows_kernel<1, false>), grid, dim3(64), 0, s, R);
    }
    if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    return ENDOR_OK;
}

}  // namespace

extern "C" endor_status endor_decompress_rows(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                              const uint16_t *d_values, int64_t nnz,
                                              const int64_t *d_row_offsets, const int64_t *d_sel, int64_t nsel,
                                              uint16_t *d_out, void *stream) {
    return run_rows(2, rows, cols, d_bitmap, d_values, nnz, d_row_offsets, d_sel, nsel, d_out, stream);
}

extern "C" endor_status endor_decompress_rows_u8(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                                 const uint8_t *d_values, int64_t nnz,
                                                 const int64_t *d_row_offsets, const int64_t *d_sel,
                                                 int64_t nsel, uint8_t *d_out, void *stream) {
    return run_rows(1, rows, cols, d_bitmap, d_values, nnz, d_row_offsets, d_sel, nsel, d_out, stream);
}

// ---------------------------------------------------------------- device-side compression

namespace {

// From how many elements on one pass over the dense matrix is faster than two, whose second finds a small matrix
// in the memory-side cache and which have nothing to wait for at the start.  Us a call, two passes / one, a tenth,
// half and nine tenths kept: fp16 8192 x 4096 55 / 56, 58.4 / 57.8, 62.5 / 57.7, 8192 x 8192 78 / 71, 85 / 77, 93 / 86;
// 8-bit 16384 x 8192 92 / 93, 99 / 94, 102 / 96, 36864 x 9216 with a tenth 186 / 173.
template <int E>
constexpr int64_t kPassMinElems = int64_t(E == 2 ? 40 : 160) << 20;
static_assert(kPassMinElems<2> / kTileElems >= kPackGroups * Blocks<2>::kTiles && kPassMinElems<1> / kTileElems >= kPackGroups * Blocks<1>::kTiles,
              "a block for every workgroup");
static_assert(kPassMinElems<2> >> 20 >= kPassMinChunks, "a party for every slice");

template <int E>
endor_status run_compress_device(int64_t rows, int64_t cols, const void *d_dense, uint8_t *d_bitmap,
                                 void *d_values, int64_t values_capacity, void *d_workspace,
                                 size_t workspace_bytes, int64_t *d_row_offsets, int64_t *d_nnz_out,
                                 void *stream) {
    if (rows < 0 || cols < 0 || values_capacity < 0) return ENDOR_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return ENDOR_ERR_UNSUPPORTED;
    if (!d_nnz_out || (reinterpret_cast<uintptr_t>(d_nnz_out) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (d_row_offsets && (reinterpret_cast<uintptr_t>(d_row_offsets) & 7)) return ENDOR_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t n = rows * cols;
    const uintptr_t em = E - 1;
    if (n > 0) {
        if (!d_dense || (reinterpret_cast<uintptr_t>(d_dense) & em)) return ENDOR_ERR_INVALID_ARG;
        if (!d_bitmap || (reinterpret_cast<uintptr_t>(d_bitmap) & 7)) return ENDOR_ERR_INVALID_ARG;
        if (values_capacity > 0 && (!d_values || (reinterpret_cast<uintptr_t>(d_values) & em)))
            return ENDOR_ERR_INVALID_ARG;
        if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 255)) return ENDOR_ERR_INVALID_ARG;
        if (workspace_bytes < workspace_bytes_n(n)) return ENDOR_ERR_BUFFER_TOO_SMALL;
    }
    if (d_row_offsets && !row_offsets_ok(rows)) return ENDOR_ERR_UNSUPPORTED;
    // one kernel between two small ones, or:
    // mask kernel: the bitmap, and each tile's count in its slot of the table; scan kernel: the table;
    // pack kernel: the values, the row offsets and the total
    CompressParams C{};
    C.dense = d_dense;
    C.bitmap = reinterpret_cast<uint64_t *>(d_bitmap);
    C.values = d_values;
    C.n = n;
    C.capacity = values_capacity;
    C.nnz_out = d_nnz_out;
    if (n == 0) {
        hipLaunchKernelGGL(endor_total_kernel, dim3(1), dim3(64), 0, s, C.table, d_nnz_out);
        if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
        return d_row_offsets ? launch_row_offsets(C.table, rows, cols, d_row_offsets, s) : ENDOR_OK;
    }
    const endor_matrix m = one_matrix(rows, cols, d_bitmap, nullptr, 0, nullptr);
    size_t off = 0;
    Group g;
    const endor_status st = fill_group(&m, 1, kNeedBitmap, E, static_cast<char *>(d_workspace), workspace_bytes, &off, &g);
    if (st != ENDOR_OK) return st;
    C.table = g.P.m[0];
    const bool aligned_in = (reinterpret_cast<uintptr_t>(d_dense) & 15) == 0;
    const uint32_t ntiles = static_cast<uint32_t>((n + kTileElems - 1) / kTileElems);
    C.row_offsets = d_row_offsets;
    C.rows = rows;
    C.cols = cols;
    if (aligned_in && n >= kPassMinElems<E>) {  // 16-byte loads; others go piece by piece in two passes
        const uint32_t nblocks = (ntiles + Blocks<E>::kTiles - 1) / Blocks<E>::kTiles;
        hipLaunchKernelGGL(endor_clear_blocks_kernel, dim3(C.table.nchunks), dim3(64), 0, s, C.table);
        if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
        hipLaunchKernelGGL(endor_compress_kernel<E>, dim3(kPackGroups), dim3(Blocks<E>::kThreads), 0, s, C, nblocks);
        if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
        hipLaunchKernelGGL(endor_finish_table_kernel, dim3(C.table.nchunks), dim3(kTilesPerChunk), 0, s, C.table);
        if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
        return ENDOR_OK;
    }
    const dim3 grid(ntiles);
    if (aligned_in)
        hipLaunchKernelGGL((endor_mask_kernel<E, true>), grid, dim3(64), 0, s, C);
    else
        hipLaunchKernelGGL((endor_mask_kernel<E, false>), grid, dim3(64), 0, s, C);
    if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    hipLaunchKernelGGL(endor_scan_counts_kernel, dim3(C.table.nchunks), dim3(kTilesPerChunk), 0, s, C.table);
    if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    if (aligned_in)
        hipLaunchKernelGGL((endor_pack_kernel<E, true>), grid, dim3(64), 0, s, C);
    else
        hipLaunchKernelGGL((endor_pack_kernel<E, false>), grid, dim3(64), 0, s, C);
    if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    return ENDOR_OK;
}

}  // namespace

extern "C" endor_status endor_compress_device(int64_t rows, int64_t cols, const uint16_t *d_dense,
                                              uint8_t *d_bitmap, uint16_t *d_values, int64_t values_capacity,
                                              void *d_workspace, size_t workspace_bytes,
                                              int64_t *d_row_offsets, int64_t *d_nnz_out, void *stream) {
    return run_compress_device<2>(rows, cols, d_dense, d_bitmap, d_values, values_capacity, d_workspace,
                                  workspace_bytes, d_row_offsets, d_nnz_out, stream);
}

extern "C" endor_status endor_compress_device_u8(int64_t rows, int64_t cols, const uint8_t *d_dense,
                                                 uint8_t *d_bitmap, uint8_t *d_values, int64_t values_capacity,
                                                 void *d_workspace, size_t workspace_bytes,
                                                 int64_t *d_row_offsets, int64_t *d_nnz_out, void *stream) {
    return run_compress_device<1>(rows, cols, d_dense, d_bitmap, d_values, values_capacity, d_workspace,
                                  workspace_bytes, d_row_offsets, d_nnz_out, stream);
}

// ---------------------------------------------------------------- selected columns (Section 4.2)

namespace {

constexpr int64_t kMaxGatherCols = int64_t(1) << 18;  // the row's bitmap and its prefixes live in LDS (16 bytes per 64 columns)

template <int E, bool kStaged, Store kStore>
void launch_cols(const ColsParams &C, int round, dim3 grid, size_t lds, hipStream_t s) {
    if (round == 3)
        hipLaunchKernelGGL((endor_gather_cols_kernel<E, kStaged, kStore, 3>), grid, dim3(kBlock), lds, s, C);
    else if (round == 4)
        hipLaunchKernelGGL((endor_gather_cols_kernel<E, kStaged, kStore, 4>), grid, dim3(kBlock), lds, s, C);
    else if constexpr (!kStaged)
        hipLaunchKernelGGL((endor_gather_cols_kernel<E, kStaged, kStore, 6>), grid, dim3(kBlock), lds, s, C);
}

template <int E, bool kStaged>
void launch_cols(const ColsParams &C, Store store, int round, dim3 grid, size_t lds, hipStream_t s) {
    if constexpr (E == 2) {
        if (store == Store::kLines) return launch_cols<E, kStaged, Store::kLines>(C, round, grid, lds, s);
        if (store == Store::kStreamed) return launch_cols<E, kStaged, Store::kStreamed>(C, round, grid, lds, s);
    }
    launch_cols<E, kStaged, Store::kPlain>(C, round, grid, lds, s);
}

template <int E, int kThreads>
void launch_cols_stream(const ColsParams &C, int queries, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(C.rows < StreamShape<kThreads>::kGroups ? C.rows : StreamShape<kThreads>::kGroups)), block(kThreads);
    if constexpr (kThreads == 512) {  // (256 threads have five queries and more)
        if (queries == 4) {
            hipLaunchKernelGGL((endor_stream_cols_kernel<E, kThreads, 4>), grid, block, 0, s, C);
            return;
        }
    }
    if (queries == 6)
        hipLaunchKernelGGL((endor_stream_cols_kernel<E, kThreads, 6>), grid, block, 0, s, C);
    else if (queries == 8)
        hipLaunchKernelGGL((endor_stream_cols_kernel<E, kThreads, 8>), grid, block, 0, s, C);
    else
        hipLaunchKernelGGL((endor_stream_cols_kernel<E, kThreads, kMaxStreamQueries>), grid, block, 0, s, C);
}

endor_status run_cols(int elem_bytes, int64_t rows, int64_t cols, const uint8_t *d_bitmap, const void *d_values,
                      int64_t nnz, const int64_t *d_row_offsets, const int64_t *d_sel, int64_t nsel, void *d_out,
                      void *stream) {
    if (rows < 0 || cols < 0 || nsel < 0 || nnz < 0) return ENDOR_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return ENDOR_ERR_UNSUPPORTED;
    if (nsel == 0 || rows == 0 || cols == 0) return ENDOR_OK;
    if (cols > kMaxGatherCols || rows > 0x7fffffff || nsel > kMaxElems / rows) return ENDOR_ERR_UNSUPPORTED;
    const uintptr_t em = static_cast<uintptr_t>(elem_bytes - 1);
    if (nnz > rows * cols) return ENDOR_ERR_INVALID_ARG;
    if (!d_bitmap || (reinterpret_cast<uintptr_t>(d_bitmap) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (nnz > 0 && (!d_values || (reinterpret_cast<uintptr_t>(d_values) & em))) return ENDOR_ERR_INVALID_ARG;
    if (!d_row_offsets || (reinterpret_cast<uintptr_t>(d_row_offsets) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (!d_sel || (reinterpret_cast<uintptr_t>(d_sel) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (!d_out || (reinterpret_cast<uintptr_t>(d_out) & em)) return ENDOR_ERR_INVALID_ARG;
    ColsParams C;
    C.bitmap = reinterpret_cast<const uint64_t *>(d_bitmap);
    C.values = d_values;
    C.out = d_out;
    C.row_offsets = d_row_offsets;
    C.sel = d_sel;
    C.rows = rows;
    C.cols = cols;
    C.nnz = nnz;
    C.nsel = nsel;
    const endor_cols_plan::Plan p = endor_cols_plan::make_plan(elem_bytes, rows, cols, nnz, nsel, reinterpret_cast<uintptr_t>(d_out));
    C.stage_units = p.stage_units;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (p.threads != 0) {
        if (p.threads == 512)
            elem_bytes == 2 ? launch_cols_stream<2, 512>(C, p.round, s) : launch_cols_stream<1, 512>(C, p.round, s);
        else
            elem_bytes == 2 ? launch_cols_stream<2, 256>(C, p.round, s) : launch_cols_stream<1, 256>(C, p.round, s);
        return hipGetLastError() == hipSuccess ? ENDOR_OK : ENDOR_ERR_HIP;
    }
    const dim3 grid(static_cast<unsigned>(rows));
    if (elem_bytes == 2)
        p.staged ? launch_cols<2, true>(C, p.store, p.round, grid, p.lds, s) : launch_cols<2, false>(C, p.store, p.round, grid, p.lds, s);
    else
        p.staged ? launch_cols<1, true>(C, p.store, p.round, grid, p.lds, s) : launch_cols<1, false>(C, p.store, p.round, grid, p.lds, s);
    if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    return ENDOR_OK;
}

}  // namespace

extern "C" endor_status endor_decompress_cols(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                              const uint16_t *d_values, int64_t nnz,
                                              const int64_t *d_row_offsets, const int64_t *d_sel, int64_t nsel,
                                              uint16_t *d_out, void *stream) {
    return run_cols(2, rows, cols, d_bitmap, d_values, nnz, d_row_offsets, d_sel, nsel, d_out, stream);
}

extern "C" endor_status endor_decompress_cols_u8(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                                 const uint8_t *d_values, int64_t nnz,
                                                 const int64_t *d_row_offsets, const int64_t *d_sel,
                                                 int64_t nsel, uint8_t *d_out, void *stream) {
    return run_cols(1, rows, cols, d_bitmap, d_values, nnz, d_row_offsets, d_sel, nsel, d_out, stream);
}
