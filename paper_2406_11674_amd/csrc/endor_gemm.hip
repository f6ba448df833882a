// Fused small-batch product on the compressed form, on the matrix cores of gfx950:
//     Y[b][i] = sum_j W[i][j] * X[b][j],   b < nb <= 16,
// with W in the Endor bitmap format (Section 4.1) and never written out densely.  This is
// the linear operation the decompressed weight is used for (Section 3.1) for a few tokens
// at once, computed on the sparse form as Section 7 ("Efficient Compute Unit") suggests.
//
// Shape of the computation.  v_mfma_f32_16x16x32_f16 multiplies a 16 x 32 block of W (its A
// operand: lane l holds 8 columns of row l%16) with a 32 x 16 block of X^T (B operand: lane l
// holds the same 8 columns of right-hand side l%16) into a 16 x 16 fp32 tile.  A wave owns 16
// rows of W and walks them 256 columns (a round) at a time: 4096 elements, 64 bitmap words, 8
// matrix instructions.  Which 32 columns an instruction takes is free as long as both operands
// agree, so lane l simply owns the bitmap word l/16 of row l%16 and its step t is byte t of that
// word: the lane's place in its row's values is a register that grows by popcounts, and the
// expanded bytes need no exchange between lanes.
//
// A round:
//   1. the lane's bitmap word (loaded two rounds ahead) is counted, the row's four words are
//      summed with lane swaps, and the row's slice of `values` (consecutive) is asked for, 16
//      bytes per lane, neighbouring lanes taking neighbouring units of one row;
//   2. a round later the slices go to LDS, row by row;
//   3. eight steps: per bitmap nibble the window of four values it may consume (three dwords
//      from the dword below), shifted into place and moved to the positions of the 1 bits with
//      v_perm_b32, whose selectors come from a 16-entry table; then the matrix instruction.
// X goes to LDS once per workgroup and round (four row groups share it), in the order in which
// the steps read it, double buffered.
//
// Measured on 28672 x 8192, half kept, 16 right-hand sides: 76 us, 8192 x 28672 72 (the form before, which read
// every byte's 20-byte window from memory through the vector cache and handed the expanded bytes
// on with ds_bpermute: 112 and 104).  Few right-hand sides go to the vector form where that is faster
// (endor_gemv_plan.h).  No unit bounds it by itself: LDS serves 70 % of the clocks (64 lanes at random
// addresses cost 7 clocks per dword, six dwords per byte), the vector ALUs are busy 43 % of the
// time, memory alone would take 45 us; but without the LDS windows 69, with nothing multiplied 64,
// without the values 70 to 76: a round's phases follow one another in step, as all waves of a workgroup
// meet at every round's tile of X.  Measured alternatives: the windows as three aligned
// 8-byte reads and selects (48 clocks of LDS, 25 % more vector instructions) 84 us; two rounds of
// values in flight 84; three workgroups per compute unit 85; units of 64 aligned bytes 84.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "endor.h"
#include "endor_device.h"
#include "endor_gemm_plan.h"
#include "endor_gemm_units.h"
#include "endor_gemv.h"
#include "endor_gemv_plan.h"
#include "endor_layout.h"

namespace {

using endor_device::global_ptr;
using endor_device::u32x4;
using endor_device::wave_sum;
using endor_gemm_plan::kBlockRows;
using endor_gemm_plan::kGemmWaves;
using endor_gemm_plan::kSegCols;
using endor_gemm_plan::make_plan;
using endor_gemm_plan::Plan;
using endor_gemm_units::Fetch;
using endor_gemm_units::fetch_lane;
using endor_gemm_units::fetch_row;
using endor_gemm_units::is_far;
using endor_gemm_units::kFetchLoads;
using endor_gemm_units::kRows;
using endor_gemm_units::Limits;
using endor_gemm_units::limits_of;
using endor_gemm_units::Slice;
using endor_gemm_units::slice_of;
using endor_gemm_units::unit_offset;
using endor_layout::chunk_total_bytes;
using endor_layout::dims_ok;
using endor_layout::kChunkStride;
using endor_layout::kTileWords;
using endor_layout::kTilesPerChunk;
using endor_layout::workspace_bytes_n;

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSteps = kSegCols / 32;   // matrix instructions per round
constexpr int kAccs = 4;                // accumulators taken in turn
constexpr int kXStep = 64 * 16;         // bytes of the tile of X one matrix instruction reads: 16 per lane, in lane order

// Where the 8 columns 64*mq + 8*t of right-hand side n sit in the tile of X.  A step's 64 fragments
// fill kXStep bytes, so reading them is free of bank conflicts; the exclusive-or spreads the 32
// fragments of one right-hand side, which are stored together, over the banks.
__device__ __forceinline__ uint32_t x_slot(uint32_t n, uint32_t mq, uint32_t t) {
    return kXStep * t + 256 * mq + 16 * (n ^ t ^ (8 * (mq & 1)));
}

// Selectors of the value placement: entry n, for a nibble n of the bitmap, holds the two v_perm_b32
// selectors that move the nibble's consecutive values (a window of four halves in two dwords) to
// the positions of its 1 bits.  A selector byte of 0x0c yields zero, so 0 bits need no mask.
// 16 entries of 8 bytes: every lookup of a wave is free of bank conflicts.
struct alignas(16) NibbleTable {
    uint64_t sel[16];
};

__device__ __forceinline__ void nibble_table_init(NibbleTable &T, uint32_t t) {
    if (t < 16) {
        uint32_t s[2] = {0x0c0c0c0cu, 0x0c0c0c0cu};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if ((t >> e) & 1) {
                const uint32_t k = __popc(t & ((1u << e) - 1));  // half of the window this element takes: 0..3
                s[e >> 1] ^= ((((2 * k + 1) << 8) | (2 * k)) ^ 0x0c0cu) << (16 * (e & 1));
            }
        }
        T.sel[t] = uint64_t(s[0]) | (uint64_t(s[1]) << 32);
    }
}

// LDS operations of one wave execute in issue order; the fences only pin the compiler.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over a row's four lanes (lane l and those 16, 32, 48 lanes away), and the sum over the ones
// before this lane.
__device__ __forceinline__ uint32_t row_sum(uint32_t x, uint32_t mq, uint32_t *before) {
    const auto s16 = __builtin_amdgcn_permlane16_swap(x, x, false, false);   // the pair's even lane; its odd lane
    const uint32_t pair = s16[0] + s16[1];
    const auto s32 = __builtin_amdgcn_permlane32_swap(pair, pair, false, false);  // lanes 0..31's pair; lanes 32..63's
    *before = ((mq & 1) ? s16[0] : 0) + ((mq & 2) ? s32[0] : 0);
    return s32[0] + s32[1];
}

__device__ const u32x4 g_dummy = {0u, 0u, 0u, 0u};  // read where there is nothing to read

constexpr int kPitch = 560;  // bytes between the staged slices of two rows: 256 values and 14 bytes of slack make 33 units;
                             // 140 dwords put the 16 rows on 16 different groups of LDS banks
constexpr int kStageBytes = kRows * kPitch;  // a window's pieces reach at most 526 + 24 bytes into a slice

// What a lane needs to know of a round besides its values.
struct Round {
    uint64_t word;   // this lane's 64 bits
    uint32_t at;     // byte offset of the word's first value in the staging area
    uint32_t off;    // byte offset of the row's first value from the row's first value of the whole part
    uint32_t units;  // the row's units
    uint32_t whole;  // those that are read whole (they come first)
    // wave-uniform
    uint32_t late;  // the first unit that was not asked for ahead; kNoneLate if no row has one
    bool ragged;    // some row has a unit that reaches over an end of `values`
};

constexpr uint32_t kNoneLate = 64;

// One wave's 16 rows of W, walked 256 columns (a round) at a time.
//
// Lane = (row mr = lane%16, word mq = lane/16), which is the operand layout of the matrix
// instruction with the columns of a round renumbered: step t multiplies byte t of every lane's
// bitmap word, i.e. columns 64*mq + 8*t .. +7, and X is read in the same order.  A lane thus works
// through its own 64-bit word, its position inside the row's slice held in a register.
template <int kClass>
struct RowStreams {
    using F = Fetch<kClass>;
    static constexpr int kLoads = kFetchLoads<kClass>;
    struct Pieces {
        u32x4 d[kLoads + F::kTail];
    };

    uint32_t mr, mq;
    uint32_t fu, frow;  // fetching: this lane's unit, and its row inside a load's kRowsPer
    uintptr_t vbeg, vend;
    uintptr_t row_first;  // the range's first value of row mr
    uintptr_t wave_base;  // the unit that holds the range's first value of the wave's first row (wave-uniform)
    uint32_t delta;       // row_first - wave_base
    Limits limits;        // what may be read around wave_base
    bool far;             // wave-uniform: some value may lie too far from wave_base for 32-bit offsets
    bool ahead;           // wave-uniform, of a range that is not far: there is a unit to ask for ahead
    uint32_t off;         // bytes of the row's values before the next round

    __device__ __forceinline__ void init(uint32_t lane) {
        mr = lane & 15;
        mq = lane >> 4;
        const uint32_t l = fetch_lane<kClass>(lane);
        frow = l / F::kUnits;
        fu = l % F::kUnits;
    }

    // Start a range of `width` columns: at most 2^30 (a sixteenth of a matrix of one row), so an offset
    // inside a row's range stays below 2^31 whatever the matrix.
    __device__ __forceinline__ void begin(uintptr_t vbeg_, uintptr_t vend_, uintptr_t first, uint32_t width) {
        vbeg = vbeg_;
        vend = vend_;
        row_first = first;
        const uintptr_t b = first & ~uintptr_t(15);
        wave_base = (uintptr_t(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32)))) << 32) |
                    static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b)));
        far = __builtin_amdgcn_ballot_w64(is_far(first, wave_base, width)) != 0;
        delta = static_cast<uint32_t>(first - wave_base);
        limits = limits_of(vbeg, vend, wave_base);
        ahead = limits.ready;
        off = 0;
    }

    __device__ __forceinline__ uint32_t load_row(int i) const { return fetch_row<kClass>(i, frow); }

    // Start a round: its bitmap word is here, its values are asked for.  There is no branch around
    // the loads (the compiler would wait for them where it ends): a lane without a unit of its own
    // reads the row's last one again, and a range that cannot be read this way reads a dummy.
    __device__ __forceinline__ void fetch(uint64_t w, Round &R, Pieces &P) {
        R.word = w;
        uint32_t before;
        const uint32_t cnt = row_sum(__popcll(w), mq, &before);
        const uint32_t start = delta + off;
        R.at = mr * kPitch + (start & 15u) + 2 * before;
        R.off = off;
        off += 2 * cnt;
        if (far) {
            fetch_far(cnt, R, P);
        } else {
            const Slice slice = slice_of(limits, start, cnt);
            R.units = slice.units;
            R.whole = ahead ? slice.whole : 0u;
            const uint32_t info = ahead ? slice.info : 0u;
            const uintptr_t base = ahead ? wave_base : reinterpret_cast<uintptr_t>(&g_dummy);
            auto load = [&](uint32_t row_info, uint32_t unit) -> u32x4 {
                return *global_ptr<u32x4>(base + unit_offset(row_info, unit));
            };
#pragma unroll
            for (int i = 0; i < kLoads; ++i)
                P.d[i] = load(static_cast<uint32_t>(
                                  __builtin_amdgcn_ds_bpermute(static_cast<int>(4 * load_row(i)), static_cast<int>(info))), fu);
            if (F::kTail) P.d[kLoads] = load(info, F::kUnits);
        }
        R.ragged = __builtin_amdgcn_ballot_w64(R.whole < R.units) != 0;
        R.late = F::kTail != 0 || __builtin_amdgcn_ballot_w64(R.whole > F::kUnits) == 0 ? kNoneLate : uint32_t(F::kUnits);
    }

    // The same with each row's whole address handed to the lanes that load for it.
    __device__ __forceinline__ void fetch_far(uint32_t cnt, Round &R, Pieces &P) const {
        uintptr_t first = (row_first + R.off) & ~uintptr_t(15);
        const uintptr_t room = first >= vbeg && vend > first ? (vend - first) >> 4 : 0;
        R.units = cnt ? ((static_cast<uint32_t>(row_first + R.off) & 15u) + 2 * cnt + 15) >> 4 : 0u;
        R.whole = R.units < room ? R.units : static_cast<uint32_t>(room);
        if (R.whole == 0) first = reinterpret_cast<uintptr_t>(&g_dummy);
        const uint32_t last = R.whole ? R.whole - 1 : 0u;
        auto of_row = [](uint32_t row, uint32_t x) {
            return static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(static_cast<int>(4 * row), static_cast<int>(x)));
        };
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const uint32_t row = load_row(i), l = of_row(row, last);
            const uintptr_t p = (uintptr_t(of_row(row, static_cast<uint32_t>(first >> 32))) << 32) | of_row(row, static_cast<uint32_t>(first));
            P.d[i] = *global_ptr<u32x4>(p + 16 * (fu < l ? fu : l));
        }
        if (F::kTail) P.d[kLoads] = *global_ptr<u32x4>(first + 16 * (F::kUnits < last ? F::kUnits : last));
    }

    // The round's values into LDS.
    __device__ __forceinline__ void stage(uint8_t *lds, const Round &R, const Pieces &P) const {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) *reinterpret_cast<u32x4 *>(lds + load_row(i) * kPitch + 16 * fu) = P.d[i];
        if (F::kTail) *reinterpret_cast<u32x4 *>(lds + mr * kPitch + 16 * F::kUnits) = P.d[kLoads];
        if (R.late == kNoneLate && !R.ragged) return;  // wave-uniform
        const uintptr_t first = (row_first + R.off) & ~uintptr_t(15);
        for (uint32_t u = R.late + mq; u < R.whole; u += 4)
            *reinterpret_cast<u32x4 *>(lds + mr * kPitch + 16 * u) = *global_ptr<u32x4>(first + 16 * u);
        // the units over an end of `values` (usually one): element by element, zero outside
        for (uint32_t u = R.whole + mq; u < R.units; u += 4) {
            uint32_t h[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {  // unconditional loads from a safe address, sorted out afterwards
                const uintptr_t p = first + 16 * u + 2 * j;
                const bool in = p >= vbeg && p + 2 <= vend;
                const uint32_t v = *global_ptr<uint16_t>(in ? p : reinterpret_cast<uintptr_t>(&g_dummy));
                h[j] = in ? v : 0u;
            }
            u32x4 d;
            d.x = h[0] | (h[1] << 16);
            d.y = h[2] | (h[3] << 16);
            d.z = h[4] | (h[5] << 16);
            d.w = h[6] | (h[7] << 16);
            *reinterpret_cast<u32x4 *>(lds + mr * kPitch + 16 * u) = d;
        }
    }
};

struct alignas(4) Dwords3 {
    uint32_t a, b, c;
};

// Byte t of the lane's word expanded to the 16 bytes of an A operand.  `at`: byte offset in `lds`
// of the byte's first value; moved on to the next byte's.
__device__ __forceinline__ u32x4 expand_byte(const NibbleTable &T, const uint8_t *lds, uint64_t word, int t, uint32_t &at) {
    const uint32_t half = static_cast<uint32_t>(t < 4 ? word : word >> 32);
    const int sh = 8 * (t & 3);
    const uint32_t n0 = (sh == 0 ? half << 3 : half >> ((sh - 3) & 31)) & 0x78u;  // low nibble * 8
    const uint32_t n1 = (half >> (sh + 1)) & 0x78u;                               // high nibble * 8
    const uint32_t at1 = at + 2 * __popc(n0);
    const Dwords3 v0 = *reinterpret_cast<const Dwords3 *>(lds + (at & ~3u));
    const Dwords3 v1 = *reinterpret_cast<const Dwords3 *>(lds + (at1 & ~3u));
    const uint64_t s0 = *reinterpret_cast<const uint64_t *>(reinterpret_cast<const uint8_t *>(T.sel) + n0);
    const uint64_t s1 = *reinterpret_cast<const uint64_t *>(reinterpret_cast<const uint8_t *>(T.sel) + n1);
    const uint32_t x0 = __builtin_amdgcn_alignbyte(v0.b, v0.a, at), x1 = __builtin_amdgcn_alignbyte(v0.c, v0.b, at);
    const uint32_t y0 = __builtin_amdgcn_alignbyte(v1.b, v1.a, at1), y1 = __builtin_amdgcn_alignbyte(v1.c, v1.b, at1);
    u32x4 d;
    d.x = __builtin_amdgcn_perm(x0, x0, static_cast<uint32_t>(s0));
    d.y = __builtin_amdgcn_perm(x1, x0, static_cast<uint32_t>(s0 >> 32));
    d.z = __builtin_amdgcn_perm(y0, y0, static_cast<uint32_t>(s1));
    d.w = __builtin_amdgcn_perm(y1, y0, static_cast<uint32_t>(s1 >> 32));
    at = at1 + 2 * __popc(n1);
    return d;
}

// A round's eight matrix instructions.  kAccs accumulators in turn: shorter chains of sums, and
// neighbouring instructions are independent.
__device__ __forceinline__ void multiply_round(const NibbleTable &T, const uint8_t *lds, const uint8_t *xt, uint32_t x_lane,
                                               const Round &R, f32x4 (&acc)[kAccs]) {
    uint32_t at = R.at;
#pragma unroll
    for (int t = 0; t < kSteps; ++t) {
        const u32x4 a = expand_byte(T, lds, R.word, t, at);
        const u32x4 b = *reinterpret_cast<const u32x4 *>(xt + kXStep * t + (x_lane ^ (16 * t)));
        acc[t % kAccs] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b),
                                                                acc[t % kAccs], 0, 0, 0);
    }
}

struct GemmParams {
    const uint64_t *bitmap;
    const uint16_t *values;
    const uint32_t *chunk_total;
    const uint32_t *tile_off;
    const uint16_t *x;  // nb right-hand sides of cols fp16 values, ldx elements apart
    float *y;           // nb x rows
    float *partial;     // sums of the row blocks that several workgroups share: slot x nb x kBlockRows
    int64_t rows, cols, nnz, ldx;
    int32_t nb;
    uint32_t segs;    // rounds per row block (the last one may lie past the last column)
    uint32_t per_wg;  // rounds per workgroup
    uint32_t rounds;  // in all
};

struct alignas(16) GemmScratch {
    NibbleTable table;
    // the segment's 256 columns of the 16 right-hand sides in the order the steps read them, for
    // this round and the next
    alignas(16) uint8_t xt[2][kSteps * kXStep];
    alignas(16) uint8_t stage[kGemmWaves][kStageBytes];  // per wave: the round's values, row by row
};

// A workgroup takes per_wg consecutive rounds of the whole product, counted row block by row block
// (64 rows, a group of 16 per wave) and inside a block from left to right: every workgroup has the
// same amount of work whatever the shape, and a row block is shared by few of them.  A block that
// lies inside one workgroup's share is written to y, the parts of the others go to the slot
// (workgroup + block) of the scratch.
//
// kAligned: rows of W start on 64-bit bitmap words (cols a multiple of 64: every model shape) and
// X moves in whole aligned 16-byte pieces.  The general form funnels a lane's bitmap bits out of
// two words and loads X element by element.  kXUnits: 16-byte pieces of X per thread and round,
// 1 for up to eight right-hand sides, else 2.
template <int kClass, bool kAligned, int kXUnits>
__global__ __launch_bounds__(64 * kGemmWaves, 2) void endor_gemm_f16_kernel(GemmParams G) {
    __shared__ GemmScratch S;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n = G.rows * G.cols;
    const int64_t nwords = (n + 63) >> 6;
    const uintptr_t vbeg = reinterpret_cast<uintptr_t>(G.values);
    const uintptr_t vend = vbeg + 2 * static_cast<uintptr_t>(G.nnz);
    nibble_table_init(S.table, threadIdx.x);  // visible after the first round's barrier
    RowStreams<kClass> V;
    V.init(lane);
    const uint32_t mr = V.mr, mq = V.mq;
    const uint32_t x_lane = x_slot(mr, mq, 0);

    uint32_t r = blockIdx.x * G.per_wg;
    const uint32_t r_end = G.rounds - r < G.per_wg ? G.rounds : r + G.per_wg;
    while (r < r_end) {
        const uint32_t block = r / G.segs, seg_begin = r % G.segs;
        const uint32_t left_in_block = G.segs - seg_begin;
        const uint32_t count = r_end - r < left_in_block ? r_end - r : left_in_block;  // rounds of this part
        r += count;
        // a group past the last row still runs (with no valid row): its wave takes part in loading X
        const int64_t row0 = int64_t(block) * kBlockRows + wave * kRows;
        const int64_t c_begin = int64_t(seg_begin) * kSegCols;
        // columns of the part, counted from c_begin
        const uint32_t width = G.cols - c_begin <= 0 ? 0u : G.cols - c_begin < int64_t(count) * kSegCols ? static_cast<uint32_t>(G.cols - c_begin)
                                                                            : count * kSegCols;

        // This lane's 64 bitmap bits of a round: row mr, columns 64*mq .. of the round.  In two halves:
        // the loads alone (unconditional, from a position that exists), and what they mean, once they
        // are needed.
        const bool row_ok = row0 + mr < G.rows;
        const int64_t word_bit = (row_ok ? row0 + mr : 0) * G.cols + c_begin + 64 * mq;  // round 0's first bit
        const uint64_t *my_words = G.bitmap + (word_bit >> 6);
        struct WordLoad {
            uint64_t lo, hi;
        };
        auto word_there = [&](uint32_t k) { return row_ok && k * kSegCols + 64 * mq < width; };
        auto load_word = [&](uint32_t k) -> WordLoad {
            const bool there = word_there(k);
            const uint64_t *p = there ? my_words + k * (kSegCols / 64) : G.bitmap;
            WordLoad L;
            L.lo = *p;
            L.hi = 0;
            if (!kAligned) L.hi = p[there && (word_bit >> 6) + k * (kSegCols / 64) + 1 < nwords ? 1 : 0];
            return L;
        };
        auto take_word = [&](uint32_t k, WordLoad L) -> uint64_t {
            uint64_t w = L.lo;
            if (!kAligned) {
                const uint32_t bs = static_cast<uint32_t>(word_bit & 63);
                w = (w >> bs) | ((L.hi << 1) << (63 - bs));  // hi << (64 - bs), and nothing when bs is 0
                const uint32_t have = width - (k * kSegCols + 64 * mq);
                if (have < 64) w &= (uint64_t(1) << have) - 1;
            }
            return word_there(k) ? w : 0;
        };
        WordLoad w0 = load_word(0), w1 = load_word(1), w2 = load_word(2);

        // The round's 256 columns of X go to LDS once per workgroup, 32 pieces of 16 bytes per
        // right-hand side: thread t carries pieces t and 256 + t through registers (loaded while the
        // round before is multiplied, stored before the round's barrier).  Columns past the part's
        // end count as zero.
        struct XPieces {
            u32x4 d[kXUnits];
            uint16_t h[kXUnits][8];
        };
        const uint16_t *x_row[kXUnits];
#pragma unroll
        for (int i = 0; i < kXUnits; ++i) {
            const int b = static_cast<int>(i * 2 * kGemmWaves + (threadIdx.x >> 5));
            x_row[i] = G.x + int64_t(b < G.nb ? b : G.nb - 1) * G.ldx + c_begin;
        }
        const uint32_t x_col = 8 * (threadIdx.x & 31);
        auto x_fetch = [&](uint32_t k, XPieces &X) {
            const uint32_t c = k * kSegCols + x_col;
#pragma unroll
            for (int i = 0; i < kXUnits; ++i) {
                if (kAligned) {
                    X.d[i] = *reinterpret_cast<const u32x4 *>(x_row[i] + (c < width ? c : 0));
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) X.h[i][j] = x_row[i][c + j < width ? c + j : 0];
                }
            }
        };
        auto x_store = [&](uint32_t k, uint32_t buf, const XPieces &X) {
            const uint32_t c = k * kSegCols + x_col;
#pragma unroll
            for (int i = 0; i < kXUnits; ++i) {
                u32x4 f;
                if (kAligned) {
                    f = X.d[i];
                    if (c >= width) f = u32x4{0u, 0u, 0u, 0u};
                } else {
                    uint32_t h[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) h[j] = c + j < width ? uint32_t(X.h[i][j]) : 0u;
                    f.x = h[0] | (h[1] << 16);
                    f.y = h[2] | (h[3] << 16);
                    f.z = h[4] | (h[5] << 16);
                    f.w = h[6] | (h[7] << 16);
                }
                const uint32_t b = i * 2 * kGemmWaves + (threadIdx.x >> 5), u = threadIdx.x & 31;
                *reinterpret_cast<u32x4 *>(S.xt[buf] + x_slot(b, u >> 3, u & 7)) = f;
            }
        };
        XPieces X;
        x_fetch(0, X);

        // Cursor of every row at the first column of the range: the number of 1 bits before flat
        // position e_r = row*cols + c_begin is (start of its chunk) + (tile offset) + (1 bits of
        // the tile's words below e_r).  Lane r < 16 looks up the first two terms of row r, the
        // whole wave counts the third for each row in turn.  All loads go out, without a test, before the
        // first result is needed, so the lookups cost one trip to memory: under their tests they were three in a
        // row at the start of every block (16 right-hand sides of 131072 x 256 24.3 us, now 22.5,
        // of 28672 x 8192 1.5 us less).
        uintptr_t cursor = vbeg;
        if (c_begin < G.cols && row0 < G.rows) {  // wave-uniform
            // (opaque: what follows from the lane alone would be kept in registers over all blocks, and three workgroups
            // of the dense form with unaligned columns would no longer fit a compute unit: 169 registers;
            // 2999 x 9001, 0.7 kept, 7 right-hand sides 29.1 us, so 22.6)
            uint32_t l = lane;
            asm volatile("" : "+v"(l));
            const int64_t e_first = row0 * G.cols + c_begin;
            const uint32_t c_first = static_cast<uint32_t>(e_first >> 20);  // chunk = 2^20 positions
            int64_t last_row = row0 + kRows - 1;
            if (last_row >= G.rows) last_row = G.rows - 1;
            const uint32_t span = static_cast<uint32_t>((last_row * G.cols + c_begin) >> 20) - c_first;  // chunks after the first
            // lane r: where row r starts
            const int64_t e = (row0 + (l & 15) < G.rows ? row0 + (l & 15) : last_row) * G.cols + c_begin;
            const uint32_t c = static_cast<uint32_t>(e >> 20);
            const uint32_t k = c - c_first;  // <= span
            const endor_device::ChunkTotals before_first = endor_device::chunk_totals(G.chunk_total, c_first, 0, l);
            const uint32_t ct = G.chunk_total[c_first + (l < span ? l : 0u)];
            const uint32_t tile = G.tile_off[size_t(c) * kChunkStride + static_cast<uint32_t>((e >> 12) % kTilesPerChunk)];
            // the words of the tile that row r starts in, up to that position
            uint64_t words[kRows];
    #pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int64_t e_r = (row0 + r < G.rows ? row0 + r : last_row) * G.cols + c_begin;
                const uint32_t we = static_cast<uint32_t>(e_r >> 6) % kTileWords;  // of the tile
                words[r] = G.bitmap[(e_r >> 12) * kTileWords + (l < we ? l : we)];  // (a word of the bitmap: e_r is a position)
            }
            __builtin_amdgcn_sched_barrier(0);
            // totals of the chunks the 16 rows start in, scanned: lane k holds sum of chunks c_first .. c_first+k
            const uint32_t incl = endor_device::wave_inclusive_scan(l < span ? ct : 0u);  // < 2^26
            uint32_t before_chunk = static_cast<uint32_t>(
                __builtin_amdgcn_ds_bpermute(static_cast<int>(4 * (k ? k - 1 : 0)), static_cast<int>(incl)));
            if (k == 0) before_chunk = 0;
            uint64_t wide = 0;  // the same for rows so wide that the 16 starts span more than 64 chunks
            if (span > 64) {
                for (uint32_t j = c_first; j < c; ++j) wide += G.chunk_total[j];
                before_chunk = 0;
            }
            // chunk start + tile offset of row `lane`
            const uint64_t head = endor_device::chunk_base_of(G.chunk_total, c_first, l, before_first) + wide + before_chunk + tile;
            uint32_t below = 0;  // lane r: 1 bits of row r's tile below e_r
    #pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int64_t e_r = (row0 + r < G.rows ? row0 + r : last_row) * G.cols + c_begin;
                const uint32_t we = static_cast<uint32_t>(e_r >> 6) % kTileWords;
                const uint64_t keep = l < we ? ~uint64_t(0) : l == we ? (uint64_t(1) << (e_r & 63)) - 1 : 0;
                const uint32_t sum = wave_sum(__popcll(words[r] & keep));
                if (l == static_cast<uint32_t>(r)) below = sum;
            }
            const uint64_t rank = head + below;  // lane r < 16: row r
            const uint32_t lo = static_cast<uint32_t>(
                __builtin_amdgcn_ds_bpermute(static_cast<int>(4 * mr), static_cast<int>(static_cast<uint32_t>(rank))));
            const uint32_t hi = static_cast<uint32_t>(
                __builtin_amdgcn_ds_bpermute(static_cast<int>(4 * mr), static_cast<int>(static_cast<uint32_t>(rank >> 32))));
            cursor = vbeg + 2 * ((uint64_t(hi) << 32) | lo);
        }

        V.begin(vbeg, vend, cursor, width);

        // A round's values are in flight while the one before is multiplied, its bitmap words one
        // round longer.  The loop body handles two rounds: no register is copied from one buffer to
        // the other (a copy would wait for the load).
        f32x4 acc[kAccs] = {};
        typename RowStreams<kClass>::Pieces P;
        Round R;
        V.fetch(take_word(0, w0), R, P);
        auto round = [&](uint32_t k, int buf, WordLoad &wk) {
            // the round's values and tile of X have arrived; after the barrier the whole tile is in
            // LDS, and every wave is through the round before (whose tile is stored over next)
            x_store(k, buf, X);
            V.stage(S.stage[wave], R, P);
            __syncthreads();
            const Round now = R;
            if (k + 1 < count) {  // not behind the last round: that took 7 to 10 % of a product of one-round blocks
                x_fetch(k + 1, X);
                const uint64_t w = take_word(k + 1, wk);
                wk = load_word(k + 3);
                V.fetch(w, R, P);
            }
            multiply_round(S.table, S.stage[wave], S.xt[buf], x_lane, now, acc);
            wave_lds_sync();  // the next round's LDS writes must stay behind this round's LDS reads
        };
        for (uint32_t k = 0; k < count; k += 2) {
            round(k, 0, w1);
            if (k + 1 >= count) break;
            round(k + 1, 1, w2);
        }
        __syncthreads();  // every wave is through with the tiles of X before the next part's are stored

        // ---- lane l holds rows 4*(l/16) .. +3 of right-hand side l%16
        f32x4 sum = acc[0];
#pragma unroll
        for (int k = 1; k < kAccs; ++k) sum += acc[k];
        if (static_cast<int32_t>(mr) < G.nb) {
            if (count == G.segs) {
                float *dst = G.y + int64_t(mr) * G.rows + row0 + 4 * mq;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (row0 + 4 * mq + i < G.rows) dst[i] = sum[i];
            } else {
                const size_t slot = size_t(blockIdx.x) + block;
                *reinterpret_cast<f32x4 *>(G.partial + (slot * G.nb + mr) * kBlockRows + wave * kRows + 4 * mq) = sum;
            }
        }
    }
}

// y[b][i] = the parts of row i's block, added in ascending order.  An output a thread, so that it is one trip to memory, and
// 32-bit divisions (rounds are fewer than 2^32): with a workgroup for all of a block's outputs, four a thread in turn, and two
// divisions of 64 bits, 4096 x 4096 with 16 right-hand sides took 18.2 us, now 13.6; 1024 x 8192 (8 right-hand sides, many
// parts) 14.7, with four parts a trip 12.6, with three or eight and no test around a load 11.7.
__global__ __launch_bounds__(256) void endor_gemm_reduce_kernel(const float *__restrict__ partial, float *__restrict__ y,
                                                                int64_t rows, int32_t nb, uint32_t segs, uint32_t per_wg) {
    const uint32_t block = blockIdx.x;
    const uint32_t first = block * segs / per_wg, last = ((block + 1) * segs - 1) / per_wg;
    if (first == last) return;  // one workgroup's block: written already
    const uint32_t i = blockIdx.y * 256 + threadIdx.x;
    const int64_t row = int64_t(block) * kBlockRows + i % kBlockRows;
    if (i >= uint32_t(nb) * kBlockRows || row >= rows) return;
    const float *src = partial + size_t(first + block) * nb * kBlockRows + i;
    const size_t step = size_t(nb) * kBlockRows;
    // (parts that there are not read the last one again)
    float s = src[0];
    auto add = [&](auto many, uint32_t k) {
        constexpr uint32_t kMany = decltype(many)::value;
        float part[kMany];
#pragma unroll
        for (uint32_t j = 0; j < kMany; ++j) part[j] = src[(k + j < last ? k + j - first : last - first) * step];
#pragma unroll
        for (uint32_t j = 0; j < kMany; ++j)
            if (k + j <= last) s += part[j];
    };
    if (last - first <= 3)
        add(std::integral_constant<uint32_t, 3>(), first + 1);
    else
        for (uint32_t k = first + 1; k <= last; k += 8) add(std::integral_constant<uint32_t, 8>(), k);
    y[(i / kBlockRows) * rows + row] = s;
}

template <int kClass>
void launch_gemm(const GemmParams &G, bool aligned, dim3 grid, dim3 block, hipStream_t s) {
    if (G.nb <= 8) {
        if (aligned)
            hipLaunchKernelGGL((endor_gemm_f16_kernel<kClass, true, 1>), grid, block, 0, s, G);
        else
            hipLaunchKernelGGL((endor_gemm_f16_kernel<kClass, false, 1>), grid, block, 0, s, G);
    } else {
        if (aligned)
            hipLaunchKernelGGL((endor_gemm_f16_kernel<kClass, true, 2>), grid, block, 0, s, G);
        else
            hipLaunchKernelGGL((endor_gemm_f16_kernel<kClass, false, 2>), grid, block, 0, s, G);
    }
}

}  // namespace

extern "C" size_t endor_gemm_scratch_bytes(int64_t rows, int64_t cols, int nb) {
    if (!dims_ok(rows, cols) || nb < 1 || nb > ENDOR_GEMM_MAX_BATCH || rows == 0 || cols == 0) return 0;
    const Plan p = make_plan(rows, cols);
    if (!p.split) return 0;
    return ((size_t(p.wgs) + p.blocks) * nb * kBlockRows * sizeof(float) + 255) & ~size_t(255);
}

extern "C" endor_status endor_gemm_f16(int64_t rows, int64_t cols, const uint8_t *d_bitmap, const uint16_t *d_values,
                                       int64_t nnz, const void *d_workspace, size_t workspace_bytes,
                                       const uint16_t *d_x, int64_t ldx, int nb, float *d_y, void *d_scratch,
                                       size_t scratch_bytes, void *stream) {
    if (rows < 0 || cols < 0 || nnz < 0 || nb < 0 || nb > ENDOR_GEMM_MAX_BATCH) return ENDOR_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return ENDOR_ERR_UNSUPPORTED;
    if (rows == 0 || nb == 0) return ENDOR_OK;
    if (rows > (int64_t(1) << 31) - kRows) return ENDOR_ERR_UNSUPPORTED;
    if (!d_y || (reinterpret_cast<uintptr_t>(d_y) & 3)) return ENDOR_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t count = int64_t(nb) * rows;
    if (cols == 0) {
        endor_gemv::zero(d_y, count, s);  // an empty sum: every output is +0.0
        return hipGetLastError() == hipSuccess ? ENDOR_OK : ENDOR_ERR_HIP;
    }
    if (nnz > rows * cols || ldx < cols) return ENDOR_ERR_INVALID_ARG;
    if (!d_bitmap || (reinterpret_cast<uintptr_t>(d_bitmap) & 7)) return ENDOR_ERR_INVALID_ARG;
    if (!d_x || (reinterpret_cast<uintptr_t>(d_x) & 1)) return ENDOR_ERR_INVALID_ARG;
    if (nnz > 0 && (!d_values || (reinterpret_cast<uintptr_t>(d_values) & 1))) return ENDOR_ERR_INVALID_ARG;
    const int64_t n = rows * cols;
    if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 255)) return ENDOR_ERR_INVALID_ARG;
    if (workspace_bytes < workspace_bytes_n(n)) return ENDOR_ERR_BUFFER_TOO_SMALL;
    const Plan p = make_plan(rows, cols);
    const size_t need = endor_gemm_scratch_bytes(rows, cols, nb);
    if (p.split) {
        if (!d_scratch || (reinterpret_cast<uintptr_t>(d_scratch) & 255)) return ENDOR_ERR_INVALID_ARG;
        if (scratch_bytes < need) return ENDOR_ERR_BUFFER_TOO_SMALL;
    }
    if (endor_gemv_plan::takes(rows, cols, nb)) {  // a few right-hand sides: no scratch is used
        endor_gemv::SmallProduct q;
        q.bitmap = reinterpret_cast<const uint64_t *>(d_bitmap);
        q.values = d_values;
        q.chunk_total = static_cast<const uint32_t *>(d_workspace);
        q.tile_off = reinterpret_cast<const uint32_t *>(static_cast<const char *>(d_workspace) + chunk_total_bytes(n));
        q.x = d_x;
        q.y = d_y;
        q.rows = rows;
        q.cols = cols;
        q.nnz = nnz;
        q.ldx = ldx;
        q.nb = nb;
        endor_gemv::small_product(q, s);
        return hipGetLastError() == hipSuccess ? ENDOR_OK : ENDOR_ERR_HIP;
    }
    GemmParams G;
    G.bitmap = reinterpret_cast<const uint64_t *>(d_bitmap);
    G.values = d_values;
    G.chunk_total = static_cast<const uint32_t *>(d_workspace);
    G.tile_off = reinterpret_cast<const uint32_t *>(static_cast<const char *>(d_workspace) + chunk_total_bytes(n));
    G.x = d_x;
    G.y = d_y;
    G.partial = static_cast<float *>(d_scratch);
    G.rows = rows;
    G.cols = cols;
    G.nnz = nnz;
    G.ldx = ldx;
    G.nb = nb;
    G.segs = p.segs;
    G.per_wg = p.per_wg;
    G.rounds = p.rounds;
    const bool aligned = cols % 64 == 0 && (reinterpret_cast<uintptr_t>(d_x) & 15) == 0 && ldx % 8 == 0;
    const dim3 grid(p.wgs), block(64 * kGemmWaves);
    // How many units of a row are asked for ahead, by the average density: 3.5 standard deviations
    // of a row's count in a round (16 sqrt(p (1 - p)) values) above its mean still fit.
    if (nnz <= n / 50 * 13)
        launch_gemm<0>(G, aligned, grid, block, s);
    else if (nnz <= n / 50 * 26)
        launch_gemm<1>(G, aligned, grid, block, s);
    else
        launch_gemm<2>(G, aligned, grid, block, s);
    if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    if (p.split) {
        hipLaunchKernelGGL(endor_gemm_reduce_kernel, dim3(p.blocks, (nb * kBlockRows + 255) / 256), dim3(256), 0, s, G.partial, d_y, rows, nb,
                           p.segs, p.per_wg);
        if (hipGetLastError() != hipSuccess) return ENDOR_ERR_HIP;
    }
    return ENDOR_OK;
}
