// Fused products on the compressed form for one to endor_gemv_plan::kMaxRhs right-hand sides:
//     y_b[i] = sum_j W[i][j] * x_b[j],
// with W in the Endor bitmap format (Section 4.1) and never written out densely: the linear operation
// the decompressed weight is used for (Section 3.1), computed on the sparse form as Section 7
// ("Efficient Compute Unit") suggests.
//
// A wave walks rows (or parts of them) a segment of up to 4096 columns at a time.  Per segment:
// popcount and scan the lane's bitmap word, leave one entry per bitmap byte in LDS ((values of the
// segment before the byte) << 9 | the byte); then a lane takes the bytes lane, 64 + lane, ... in turn,
// reads each byte's window of values straight from memory, places the values by the byte's bit
// pattern and multiplies them with the matching 8 entries of each x.  Elements whose bit is 0 enter as
// +0.0, as they would from the dense matrix.
//
// What bounds it, at half density: reading.  8192 x 28672 takes 48 us (5.5 TB/s; the form before, a wave
// per row and a barrier per segment, 59); a kernel that only reads as many bytes the same way 42, this
// one without its loads of values 37.  At a tenth kept the work per bitmap byte bounds it: 40 us (the form
// before 44).  What made the difference, in turn (8192 x 28672): no barrier and no start per row 58 us;
// streamed loads of the windows 53 (plain reads of this size reach 5.9 TB/s, streamed ones 6.6);
// 12 waves of up to 168 registers instead of 16 of 128 for the longest segments 50 (with 128 the
// compiler reads a segment's entries one after the other, 51 to 58 us from one build to the next).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "endor.h"
#include "endor_device.h"
#include "endor_gemv.h"
#include "endor_gemv_plan.h"
#include "endor_gemv_windows.h"
#include "endor_layout.h"

namespace {

using endor_device::chunk_base;
using endor_device::global_ptr;
using endor_device::place_window;
using endor_device::row_inclusive_scan;
using endor_device::u32x4;
using endor_device::wave_inclusive_scan;
using endor_device::window_fifth;
using endor_device::window_finish;
using endor_device::window_guarded;
using endor_device::window_tables_init;
using endor_device::WindowTables;
using endor_gemv_windows::edge_entry;
using endor_gemv_windows::end_windows;
using endor_gemv_windows::entry_of;
using endor_gemv_windows::is_whole;
using endor_gemv_windows::kEdge;
using endor_gemv_windows::kElements;
using endor_gemv_windows::kWhole;
using endor_gemv_windows::whole_windows;
using endor_gemv_windows::Windows;
using endor_layout::dims_ok;
using endor_layout::kChunkStride;
using endor_layout::kTilesPerChunk;
using endor_layout::kTileWords;

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));

__device__ const u32x4 g_dummy = {0u, 0u, 0u, 0u};  // read where there is nothing to read

struct GemvParams {
    const uint64_t *bitmap;
    const uint16_t *values;
    const int64_t *row_offsets;   // rows + 1, or null: then
    const uint32_t *chunk_total;  // the offset table
    const uint32_t *tile_off;
    const uint16_t *x;  // right-hand sides of cols fp16 values, ldx elements apart
    float *y;           // one after the other, rows fp32 each
    int64_t rows, cols, nnz, ldx;
    uint32_t panel;      // columns of x in LDS at a time: whole segments
    uint32_t parts;      // items per row and panel
    uint32_t part_segs;  // segments per item
    // What a workgroup would begin with dividing, 64 bits by 32 twice and 32 by 32 five times, two hundred scalar
    // instructions before its first load: rows / workgroups, the share of them that has one more, waves / parts and
    // the remainder, and 65536 / parts rounded up or one more.
    uint32_t rows_each, more_share, row_step, part_step, part_inverse;
};

__device__ __forceinline__ float wave_sum_f32(float x) {
    // same lane order as wave_inclusive_scan, so the result does not depend on timing
#define ENDOR_DPP_ADD_F32(ctrl, rowmask)                                                                     \
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), ctrl, rowmask, \
                                                               0xf, true))
    ENDOR_DPP_ADD_F32(0x111, 0xf);
    ENDOR_DPP_ADD_F32(0x112, 0xf);
    ENDOR_DPP_ADD_F32(0x114, 0xf);
    ENDOR_DPP_ADD_F32(0x118, 0xf);
    ENDOR_DPP_ADD_F32(0x142, 0xa);
    ENDOR_DPP_ADD_F32(0x143, 0xc);
#undef ENDOR_DPP_ADD_F32
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}

// LDS operations of one wave execute in issue order; the fences only pin the compiler.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

__device__ __forceinline__ uint64_t uniform(uint64_t v) {  // wave-uniform, and the compiler has to know
    return (uint64_t(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)))) << 32) |
           static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}

// Sums of products of expanded fp16 elements with the matching entries of x, in fp32: products of fp16
// numbers are exact there, and fp16 subnormals count in full.  v_mfma_f32_4x4x4_16b_f16 multiplies 16
// separate 4 x 4 blocks; lane l holds four elements of row l%4 of block l/4 of W, and of column l%4 of X.
// Only the diagonals are wanted (row i of a block belongs to the same lane as column i): a quarter of the
// instruction's work, but two of them stand for eight multiply-adds.
struct Sums {
    f32x4 a;
    __device__ __forceinline__ void clear() { a = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }
    // 8 expanded elements against the matching 8 entries of x
    __device__ __forceinline__ void operator()(u32x4 d, u32x4 x) {
        a = __builtin_amdgcn_mfma_f32_4x4x4f16(half4(d.x, d.y), half4(x.x, x.y), a, 0, 0, 0);
        a = __builtin_amdgcn_mfma_f32_4x4x4f16(half4(d.z, d.w), half4(x.z, x.w), a, 0, 0, 0);
    }
    __device__ __forceinline__ float total(uint32_t lane) const {  // lane l's own sum is row l%4 of its column
        const float lo = (lane & 1) ? a.y : a.x, hi = (lane & 1) ? a.w : a.z;
        return wave_sum_f32((lane & 2) ? hi : lo);
    }
    __device__ __forceinline__ static f16x4 half4(uint32_t lo, uint32_t hi) {
        return __builtin_bit_cast(f16x4, uint64_t(lo) | (uint64_t(hi) << 32));
    }
};

// 8 halves without the first s (0 to 8) of them, zeros behind
__device__ __forceinline__ u32x4 drop_halves(u32x4 d, uint32_t s) {
    uint64_t lo = d.x | (uint64_t(d.y) << 32), hi = d.z | (uint64_t(d.w) << 32);
    const uint32_t b = 16 * (s & 3u);
    if (s >= 4) {
        lo = hi;
        hi = 0;
    }
    lo = (lo >> b) | ((hi << 1) << (63 - b));
    hi >>= b;
    if (s >= 8) lo = hi = 0;
    d.x = static_cast<uint32_t>(lo);
    d.y = static_cast<uint32_t>(lo >> 32);
    d.z = static_cast<uint32_t>(hi);
    d.w = static_cast<uint32_t>(hi >> 32);
    return d;
}

// Entries [c, c + 8) of a vector of `cols`, zeros past its end.  In two halves: the load alone
// (unconditional, from a place that exists), and what it means, once it is needed.
// kShort: vectors of fewer than 8 entries.
template <bool kShort>
__device__ __forceinline__ u32x4 x_load(const uint16_t *x, int64_t c, int64_t cols) {
    if (!kShort) return *global_ptr<u32x4_a2>(reinterpret_cast<uintptr_t>(x + (c < cols - 8 ? c : cols - 8)));
    uint32_t h[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = x[c + j < cols ? c + j : 0];
    u32x4 d;
    d.x = h[0] | (h[1] << 16);
    d.y = h[2] | (h[3] << 16);
    d.z = h[4] | (h[5] << 16);
    d.w = h[6] | (h[7] << 16);
    return d;
}
template <bool kShort>
__device__ __forceinline__ u32x4 x_take(u32x4 d, int64_t c, int64_t cols) {
    if (!kShort) {  // the piece that was read began `late` entries before c
        const int64_t late = c - (cols - 8);
        return late <= 0 ? d : drop_halves(d, late < 8 ? static_cast<uint32_t>(late) : 8u);
    }
    uint64_t lo = d.x | (uint64_t(d.y) << 32), hi = d.z | (uint64_t(d.w) << 32);
    const int64_t have = cols - c;  // entries that exist
    if (have < 8) {
        hi = have <= 4 ? 0 : hi & ((uint64_t(1) << (16 * (have - 4))) - 1);
        if (have < 4) lo = have <= 0 ? 0 : lo & ((uint64_t(1) << (16 * have)) - 1);
    }
    d.x = static_cast<uint32_t>(lo);
    d.y = static_cast<uint32_t>(lo >> 32);
    d.z = static_cast<uint32_t>(hi);
    d.w = static_cast<uint32_t>(hi >> 32);
    return d;
}

// This lane's 64 bits of a segment of `nbits` (<= 4096) bits that starts at an arbitrary bit
// position e of the bitmap.  In two halves again: the loads (unconditional, from indices clamped into
// the bitmap), and the funnel.
struct WordLoad {
    uint64_t lo, hi;
};
__device__ __forceinline__ WordLoad word_load(const uint64_t *bitmap, int64_t nwords, int64_t e, uint32_t lane) {
    // e is wave-uniform: a scalar base, and 32-bit offsets from it
    const int64_t w0 = (e >> 6) < nwords ? e >> 6 : nwords - 1, room = nwords - 1 - w0;
    const uint32_t lim = room < 64 ? static_cast<uint32_t>(room) : 64u;
    const uintptr_t base = reinterpret_cast<uintptr_t>(bitmap + w0);
    WordLoad L;
    L.lo = *global_ptr<uint64_t>(base + 8 * (lane < lim ? lane : lim));
    L.hi = *global_ptr<uint64_t>(base + 8 * (lane + 1 < lim ? lane + 1 : lim));
    return L;
}
__device__ __forceinline__ uint64_t word_take(WordLoad L, int64_t e, uint32_t nbits, uint32_t lane) {
    // bits past the bitmap's end lie past the segment's end: clamped loads need no test of their own
    const uint32_t bs = static_cast<uint32_t>(e & 63);
    uint64_t w = (L.lo >> bs) | ((L.hi << 1) << (63 - bs));  // hi << (64 - bs), and nothing when bs is 0
    const uint32_t have = lane * 64 < nbits ? nbits - lane * 64 : 0u;
    if (have < 64) w &= (uint64_t(1) << have) - 1;
    return w;
}

// A segment whose windows of values have been asked for.
template <int kSteps>
struct Segment {
    u32x4 win[kSteps];
    uint32_t end;  // the first dword after the segment's last window, for lane 63's last byte
    // wave-uniform
    uint32_t how;    // its windows are read: kWhole, kEdge, kElements
    uintptr_t base;  // that positions count from
};

// Entries to LDS, loads of the windows: streamed, although neighbouring windows overlap (the overlaps meet in
// the vector cache; 58 us without, 53 with, on 8192 x 28672, half kept).  There is no branch around the loads
// (the compiler would wait for them where it ends): a segment that is put together element by element when it is used reads a dummy.
template <int kSteps>
__device__ __forceinline__ void segment_issue(Segment<kSteps> &S, uint32_t *entry, uint64_t word, uint64_t &next_value,
                                              uintptr_t vbeg, uintptr_t vend, uint32_t lane) {
    const uint32_t pc = __popcll(word);
    const uint32_t incl = wave_inclusive_scan(pc);
    const uint32_t cnt = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
    const uintptr_t vseg = vbeg + 2 * next_value;  // the segment's first value
    next_value += cnt;
    const Windows whole = whole_windows(vseg);
    uintptr_t base = static_cast<uintptr_t>(whole.base), end = (vseg + 2 * uintptr_t(cnt)) & ~uintptr_t(3);
    uint32_t mask = whole.offset_mask;
    S.how = kWhole;
    S.base = base;
    {
        uint32_t at = whole.first + incl - pc;  // position of the first value of this lane's word
        uint32_t e8[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t byte = static_cast<uint32_t>(word >> (8 * b)) & 0xffu;
            e8[b] = entry_of(at, byte);
            at += __popc(byte);
        }
        if (__builtin_expect(!is_whole(vbeg, vend, vseg, cnt), 0)) {  // wave-uniform
            const Windows ends = end_windows(vbeg, vend, vseg);
            const uintptr_t dummy = reinterpret_cast<uintptr_t>(&g_dummy);
            S.how = ends.how;
            S.base = static_cast<uintptr_t>(ends.base);
            base = ends.how == kElements ? dummy : S.base;
            mask = ends.offset_mask;
            end = dummy;
#pragma unroll
            for (int b = 0; b < 8; ++b) e8[b] = edge_entry(e8[b] + ((ends.first - whole.first) << 9), ends.limit);
        }
        u32x4 lo, hi;
        lo.x = e8[0];
        lo.y = e8[1];
        lo.z = e8[2];
        lo.w = e8[3];
        hi.x = e8[4];
        hi.y = e8[5];
        hi.z = e8[6];
        hi.w = e8[7];
        if (kSteps == 8 || lane < 8 * kSteps) {
            reinterpret_cast<u32x4 *>(entry)[2 * lane] = lo;
            reinterpret_cast<u32x4 *>(entry)[2 * lane + 1] = hi;
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < kSteps; ++k)
        S.win[k] = __builtin_nontemporal_load(global_ptr<u32x4_a2>(base + ((entry[k * 64 + lane] >> 8) & mask)));
    S.end = *global_ptr<uint32_t>(end);
}

// The segment's products.  x(k, b): the 8 entries of right-hand side b that step k of this lane takes.
template <int kSteps, int kRhs, class X>
__device__ __forceinline__ void segment_multiply(const Segment<kSteps> &S, const uint32_t *entry, const WindowTables &T,
                                                 uintptr_t vbeg, uintptr_t vend, uint32_t lane, X x, Sums (&acc)[kRhs]) {
    if (__builtin_expect(S.how == kWhole, 1)) {  // wave-uniform
#pragma unroll
        for (int k = 0; k < kSteps; ++k) {
            const uint32_t e = entry[k * 64 + lane];
            const uint32_t after = k + 1 < kSteps ? static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(
                                                        static_cast<int>(S.win[(k + 1) % kSteps].x)))
                                                  : S.end;
            const u32x4 w = window_finish(S.win[k], window_fifth(S.win[k], after), e >> 8);
            const u32x4 d = place_window(T, e & 0xffu, w);
#pragma unroll
            for (int b = 0; b < kRhs; ++b) acc[b](d, x(k, b));
        }
    } else if (S.how == kEdge) {
#pragma unroll
        for (int k = 0; k < kSteps; ++k) {
            const uint32_t e = entry[k * 64 + lane];
            const u32x4 d = place_window(T, e & 0xffu, drop_halves(S.win[k], e >> 28));
#pragma unroll
            for (int b = 0; b < kRhs; ++b) acc[b](d, x(k, b));
        }
    } else {
        wait_loads();  // the dummies: or the compiler counts them as still on their way in what follows
#pragma unroll 1
        for (int k = 0; k < kSteps; ++k) {
            const uint32_t e = entry[k * 64 + lane];
            const u32x4 d = place_window(T, e & 0xffu, window_guarded(S.base + (e >> 8), vbeg, vend));
#pragma unroll
            for (int b = 0; b < kRhs; ++b) acc[b](d, x(k, b));
        }
    }
    wave_lds_sync();  // entries written later stay behind these reads
}

// 1 bits of flat positions [from, to), by 16 lanes; lane 15 has the result.
__device__ __forceinline__ uint32_t count_bits16(const uint64_t *bitmap, int64_t from, int64_t to, uint32_t lane) {
    const int64_t wa = from >> 6, wb = (to - 1) >> 6;
    uint32_t sum = 0;
    constexpr int kBatch = 8;  // words a lane has in flight
    for (int64_t w0 = wa; w0 <= wb; w0 += kBatch * 16) {
        uint64_t t[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {  // unconditional: an index past the last word reads the last again
            const int64_t w = w0 + 16 * k + lane;
            t[k] = bitmap[w <= wb ? w : wb];
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int64_t w = w0 + 16 * k + lane;
            uint64_t v = w <= wb ? t[k] : 0;
            if (w == wa) v &= ~uint64_t(0) << (from & 63);
            if (w == wb) v &= ~uint64_t(0) >> (63 - ((to - 1) & 63));
            sum += __popcll(v);
        }
    }
    return row_inclusive_scan(sum);
}

// Number of 1 bits before flat position e of the matrix, from the offset table: 16 lanes per position.
// `first`: those before chunk c_first, which holds e or comes before it.  Lane 15 of the 16 has the result.
__device__ __forceinline__ uint64_t rank_from_table(const GemvParams &G, int64_t e, uint32_t c_first, uint64_t first, uint32_t lane) {
    const int64_t we = e >> 6;
    const uint32_t c = static_cast<uint32_t>(e >> 20);  // chunk = 2^20 positions
    uint64_t t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // the tile's words before e
        const int64_t w = (e >> 12) * kTileWords + 16 * k + (lane & 15);
        t[k] = G.bitmap[w < we ? w : we];
    }
    uint64_t at = first + G.tile_off[size_t(c) * kChunkStride + (e >> 12) % kTilesPerChunk];
    for (uint32_t j = c_first; j < c; ++j) at += G.chunk_total[j];
    uint32_t below = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t w = (e >> 12) * kTileWords + 16 * k + (lane & 15);
        below += w < we ? __popcll(t[k]) : w == we ? __popcll(t[k] & ((uint64_t(1) << (e & 63)) - 1)) : 0;
    }
    return at + row_inclusive_scan(below);
}

// A workgroup per compute unit takes a block of consecutive rows.  x (or a panel of it) stays in LDS, where
// the items' starts in `values` are laid out as well (an item is a row, or a part of one); after that its
// waves run on their own, without a barrier, each through its items segment by segment.  A segment's
// windows are asked for before the segment before it is multiplied, its bitmap words one segment earlier,
// across the ends of items.
//
// kWaves: 12 for segments of 8 steps (see the top), else 16; the plan is endor_gemv_plan.h's; two workgroups of 8 waves per compute unit,
// or of 10 with 96 registers, were slower (53 -> 66 and 80 us for segments of 4 steps).
template <int kRhs, int kSteps, int kWaves, bool kShort>
__global__ __launch_bounds__(64 * kWaves, kWaves / 4) void endor_gemv_kernel(GemvParams G) {
    constexpr int kThreads = 64 * kWaves;
    constexpr int kMaxItems = endor_gemv_plan::max_items(kSteps, kRhs);
    constexpr int kSeg = 512 * kSteps;
    extern __shared__ u32x4 s_x[];  // kRhs panels
    __shared__ WindowTables s_tables;
    __shared__ alignas(16) uint32_t s_entry[kWaves][2][64 * kSteps];
    __shared__ uint64_t s_start[kMaxItems];    // index of an item's first value
    __shared__ uint64_t s_end[kMaxItems];      // of a row's first value in the next panel
    __shared__ float s_sum[kMaxItems * kRhs];  // an item's sums
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t group = blockIdx.x, more = endor_gemv_plan::more_before(group, G.more_share);
    const int64_t row_begin = static_cast<int64_t>(uint64_t(group) * G.rows_each) + more;
    const uint32_t parts = G.parts, nrows = G.rows_each + (endor_gemv_plan::more_before(group + 1, G.more_share) - more), items = nrows * parts;
    // x / parts, for numbers of items: x * part_inverse is off by at most x * parts, less than 65536
    auto by_parts = [&](uint32_t x) { return x * G.part_inverse >> 16; };
    const int64_t nwords = (G.rows * G.cols + 63) >> 6;
    const uintptr_t vbeg = reinterpret_cast<uintptr_t>(G.values);
    const uintptr_t vend = vbeg + 2 * static_cast<uintptr_t>(G.nnz);
    const uint32_t pieces = G.panel / 8;  // of x, per right-hand side
    const uint32_t row_step = G.row_step, part_step = G.part_step;  // from one of a wave's items to the next

    for (int64_t p_begin = 0; p_begin < G.cols; p_begin += G.panel) {
        const int64_t p_end = G.cols - p_begin < G.panel ? G.cols : p_begin + G.panel;
        // ---- the wave's items
        struct Place {
            uint32_t row, part, seg;  // of the block, of the row, of the part
            int64_t bit;              // the segment's first
            uint32_t nbits;
        };
        auto locate = [&](Place &P) {
            const int64_t c = p_begin + int64_t(P.part * G.part_segs + P.seg) * kSeg, left = p_end - c;
            P.bit = (row_begin + P.row) * G.cols + c;
            P.nbits = left <= 0 ? 0u : left < kSeg ? static_cast<uint32_t>(left) : uint32_t(kSeg);
        };
        auto after = [&](Place P) -> Place {
            if (++P.seg == G.part_segs) {
                P.seg = 0;
                P.row += row_step;
                P.part += part_step;
                if (P.part >= parts) {
                    P.part -= parts;
                    ++P.row;
                }
            }
            locate(P);
            return P;
        };
        Place next;  // the segment whose bitmap words have been asked for
        next.row = by_parts(wave);
        next.part = wave - next.row * parts;
        next.seg = 0;
        locate(next);
        WordLoad words = word_load(G.bitmap, nwords, next.bit, lane);
        // ---- x
        constexpr int kBatch = 4;  // pieces a thread has in flight
        for (int b = 0; b < kRhs; ++b) {
            const uint16_t *x = G.x + int64_t(b) * G.ldx;
            for (uint32_t p0 = threadIdx.x; p0 < pieces; p0 += kBatch * kThreads) {
                u32x4 d[kBatch];
#pragma unroll
                for (int q = 0; q < kBatch; ++q) d[q] = x_load<kShort>(x, p_begin + 8 * int64_t(p0 + q * kThreads), G.cols);
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const uint32_t p = p0 + q * kThreads;
                    if (p < pieces) s_x[b * pieces + p] = x_take<kShort>(d[q], p_begin + 8 * int64_t(p), G.cols);
                }
            }
        }
        if (p_begin == 0) window_tables_init(s_tables, threadIdx.x);
        // ---- where the items' values start
        if (G.row_offsets == nullptr) {
            const uint32_t c_first = static_cast<uint32_t>((row_begin * G.cols) >> 20);
            const uint64_t first = chunk_base(G.chunk_total, c_first, lane);
            for (uint32_t it0 = 4 * wave; it0 < items; it0 += 4 * kWaves) {
                const uint32_t it = it0 + lane / 16, r = by_parts(it);
                const int64_t c = p_begin + int64_t(it - r * parts) * G.part_segs * kSeg;
                if (it < items && c < p_end) {
                    const uint64_t rank = rank_from_table(G, (row_begin + r) * G.cols + c, c_first, first, lane);
                    if ((lane & 15) == 15) s_start[it] = rank;
                }
            }
        } else if (parts == 1) {
            for (uint32_t r = threadIdx.x; r < nrows; r += kThreads)
                s_start[r] = p_begin == 0 ? static_cast<uint64_t>(G.row_offsets[row_begin + r]) : s_end[r];
        } else {  // the row's first value and the 1 bits of its earlier parts, 16 lanes each
            for (uint32_t it0 = 4 * wave; it0 < items; it0 += 4 * kWaves) {
                const uint32_t it = it0 + lane / 16, r = by_parts(it);
                const int64_t c = p_begin + int64_t(it - r * parts) * G.part_segs * kSeg, bit = (row_begin + r) * G.cols;
                if (it < items && c < p_end) {
                    uint64_t at = p_begin == 0 ? static_cast<uint64_t>(G.row_offsets[row_begin + r]) : s_end[r];
                    if (c > p_begin) at += count_bits16(G.bitmap, bit + p_begin, bit + c, lane & 15);
                    if ((lane & 15) == 15) s_start[it] = at;
                }
            }
        }
        __syncthreads();
        uint32_t left = items > wave ? (items - wave + kWaves - 1) / kWaves * G.part_segs : 0;  // segments to go
        if (left) {
            Sums acc[kRhs];
#pragma unroll
            for (int b = 0; b < kRhs; ++b) acc[b].clear();
            Segment<kSteps> A, B;
            uint64_t value = 0;  // index of the next segment's first value
            auto issue = [&](uint32_t buf, Segment<kSteps> &S) {
                const uint64_t w = word_take(words, next.bit, next.nbits, lane);
                const Place here = next;
                next = after(here);
                words = word_load(G.bitmap, nwords, next.bit, lane);
                if (here.seg == 0) value = uniform(s_start[here.row * parts + here.part]);
                segment_issue(S, s_entry[wave][buf], w, value, vbeg, vend, lane);
                if (here.part + 1 == parts && here.seg + 1 == G.part_segs && lane == 0) s_end[here.row] = value;
                return here;
            };
            auto multiply = [&](uint32_t buf, const Segment<kSteps> &S, const Place &at) {
                const u32x4 *x = s_x + (at.part * G.part_segs + at.seg) * (kSeg / 8) + lane;
                segment_multiply(S, s_entry[wave][buf], s_tables, vbeg, vend, lane, [&](int k, int b) { return x[b * pieces + k * 64]; }, acc);
                if (at.seg + 1 == G.part_segs) {
                    float *sum = s_sum + (at.row * parts + at.part) * kRhs;
#pragma unroll
                    for (int b = 0; b < kRhs; ++b) {
                        const float t = acc[b].total(lane);
                        if (lane == 0) sum[b] = p_begin == 0 ? t : sum[b] + t;
                        acc[b].clear();
                    }
                }
            };
            // One way out of the loop, and no branch around a segment's loads: the compiler waits at the end
            // of a branch for what any way there may have left in flight.
            Place a = issue(0, A), b;
            for (; left > 2; left -= 2) {
                b = issue(1, B);
                multiply(0, A, a);
                a = issue(0, A);
                multiply(1, B, b);
            }
            if (left == 2) {
                b = issue(1, B);
                multiply(0, A, a);
                multiply(1, B, b);
            } else {
                multiply(0, A, a);
            }
        }
        __syncthreads();
    }
    for (uint32_t k = threadIdx.x; k < nrows * kRhs; k += kThreads) {
        const uint32_t b = kRhs == 1 ? 0 : k / nrows, r = k - b * nrows;
        float s = s_sum[r * parts * kRhs + b];
        for (uint32_t p = 1; p < parts; ++p) s += s_sum[(r * parts + p) * kRhs + b];
        G.y[int64_t(b) * G.rows + row_begin + r] = s;
    }
}

// a kernel, so that the call can be captured into a graph
__global__ __launch_bounds__(256) void endor_zero_kernel(float *__restrict__ y, int64_t count) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < count) y[i] = 0.0f;
}

// by_parts: items and the numbers a wave looks at past them, by parts
static_assert((512 + 4 * 16) * 16 < 65536, "exact");

template <int kRhs, int kSteps, bool kShort = false>
void launch_steps(GemvParams G, const endor_gemv_plan::Plan &p, hipStream_t s) {
    constexpr int kWaves = endor_gemv_plan::waves_of(kSteps);
    static_assert(sizeof(WindowTables) == endor_gemv_plan::kTableBytes, "LDS beside x");
    G.part_segs = static_cast<uint32_t>(p.part_segs);
    G.parts = static_cast<uint32_t>(p.parts);
    G.panel = static_cast<uint32_t>(p.parts * p.part_segs * endor_gemv_plan::seg_cols(kSteps));
    G.rows_each = static_cast<uint32_t>(G.rows / p.grid);
    G.more_share = endor_gemv_plan::more_share(static_cast<uint32_t>(G.rows % p.grid), static_cast<uint32_t>(p.grid));
    G.row_step = static_cast<uint32_t>(kWaves / p.parts);
    G.part_step = static_cast<uint32_t>(kWaves % p.parts);
    G.part_inverse = static_cast<uint32_t>(65536 / p.parts + 1);
    hipLaunchKernelGGL((endor_gemv_kernel<kRhs, kSteps, kWaves, kShort>), dim3(static_cast<unsigned>(p.grid)), dim3(64 * kWaves),
                       size_t(G.panel) * 2 * kRhs, s, G);
}

template <int kRhs>
void launch(const GemvParams &G, hipStream_t s) {
    const endor_gemv_plan::Plan p = endor_gemv_plan::make_plan(G.rows, G.cols, kRhs);
    if (G.cols < 8)  // one right-hand side
        launch_steps<1, 2, true>(G, p, s);
    else if (p.steps == 2)
        launch_steps<kRhs, 2>(G, p, s);
    else if (p.steps == 4)
        launch_steps<kRhs, 4>(G, p, s);
    else if constexpr (endor_gemv_plan::most_steps(kRhs) == 8)
        p.steps == 6 ? launch_steps<kRhs, 6>(G, p, s) : launch_steps<kRhs, 8>(G, p, s);
}

}  // namespace

namespace endor_gemv {

void zero(float *y, int64_t count, hipStream_t s) {
    hipLaunchKernelGGL(endor_zero_kernel, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s, y, count);
}

void small_product(const SmallProduct &p, hipStream_t s) {
    GemvParams G{};
    G.bitmap = p.bitmap;
    G.values = p.values;
    G.chunk_total = p.chunk_total;
    G.tile_off = p.tile_off;
    G.x = p.x;
    G.y = p.y;
    G.rows = p.rows;
    G.cols = p.cols;
    G.nnz = p.nnz;
    G.ldx = p.ldx;
    switch (p.nb) {
        case 1: launch<1>(G, s); break;
        case 2: launch<2>(G, s); break;
        case 3: launch<3>(G, s); break;
        default: launch<4>(G, s); break;
    }
}

}  // namespace endor_gemv

extern "C" endor_status endor_gemv_f16(int64_t rows, int64_t cols, const uint8_t *d_bitmap,
                                       const uint16_t *d_values, int64_t nnz, const int64_t *d_row_offsets,
                                       const uint16_t *d_x, float *d_y, void *stream) {
    if (rows < 0 || cols < 0 || nnz < 0) return ENDOR_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return ENDOR_ERR_UNSUPPORTED;
    if (rows == 0) return ENDOR_OK;
    if (rows > 0x7fffffff) return ENDOR_ERR_UNSUPPORTED;
    if (!d_y || (reinterpret_cast<uintptr_t>(d_y) & 3)) return ENDOR_ERR_INVALID_ARG;
    if (!d_row_offsets || (reinterpret_cast<uintptr_t>(d_row_offsets) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (cols > 0) {
        if (nnz > rows * cols) return ENDOR_ERR_INVALID_ARG;
        if (!d_bitmap || (reinterpret_cast<uintptr_t>(d_bitmap) & 7)) return ENDOR_ERR_INVALID_ARG;
        if (!d_x || (reinterpret_cast<uintptr_t>(d_x) & 1)) return ENDOR_ERR_INVALID_ARG;
        if (nnz > 0 && (!d_values || (reinterpret_cast<uintptr_t>(d_values) & 1))) return ENDOR_ERR_INVALID_ARG;
    }
    GemvParams G{};
    G.bitmap = reinterpret_cast<const uint64_t *>(d_bitmap);
    G.values = d_values;
    G.row_offsets = d_row_offsets;
    G.x = d_x;
    G.y = d_y;
    G.rows = rows;
    G.cols = cols;
    G.nnz = nnz;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (cols == 0)  // an empty sum
        endor_gemv::zero(d_y, rows, s);
    else
        launch<1>(G, s);
    if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    return ENDOR_OK;
}
