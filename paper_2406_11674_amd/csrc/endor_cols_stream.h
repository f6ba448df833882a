// Column-subset decompression of matrices with long rows: workgroups that stay, a row after the other.  Included by
// endor_kernels.hip, whose types and loads it uses.
//
// endor_gather_cols_kernel takes a row through three phases in turn, bitmap, values, queries, and the four to six
// workgroups of a compute unit hardly overlap them.  Here two workgroups of eight waves (or four of four, for rows of
// up to 15 KB) stay on a compute unit and take every groups-th row, and in one step, which ends with the only barrier,
// answer the queries of a row from LDS while the values of the next one arrive there, its ranks are finished, the
// bitmap of the one after is counted and that of the next after that is on its way.  The columns asked for are read once
// and stay in registers, an output row is a buffer that drops what is outside it.
//
// Bound by the step's chain of LDS reads and waits, 0.9 us at least, and by memory: a tenth of 8192 x 28672, half kept,
// reads every line of the values, 46 us by themselves: 55 us, a workgroup per row 63 (one workgroup of 16 waves with
// three rows' values: 56, but 104 against 61 on 28672 x 8192, where steps are short).
#ifndef ENDOR_COLS_STREAM_H_
#define ENDOR_COLS_STREAM_H_

namespace {

constexpr uint32_t kOutside = 0x7fffffffu;  // an offset past every range
using endor_cols_plan::kMaxStreamQueries;
using endor_cols_plan::StreamShape;

// vmcnt(N) and lgkmcnt(0)
template <int N>
__device__ __forceinline__ void wait_all_but() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x70);
}

// kQ: queries of a thread.
template <int E, int kThreads, int kQ>
__global__ __launch_bounds__(kThreads, 4) void endor_stream_cols_kernel(ColsParams C) {
    typedef std::conditional_t<E == 2, uint16_t, uint8_t> Elem;
    typedef StreamShape<kThreads> Sh;
    constexpr uint32_t kUnits = Sh::kUnits;
    constexpr int kWaves = Sh::kWaves;
    // the values of two rows: variables of their own, so that what is read from one does not wait for the loads into the other
    __shared__ u32x4 s_v0[kUnits], s_v1[kUnits];
    __shared__ u32x4 s_pairs[2][kThreads];  // two pairs (32 bits of the row's bitmap, 1 bits of the row before them) a word
    __shared__ uint32_t s_count[2][kWaves];
    __shared__ uint32_t s_total[2];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    const int64_t nwords = (C.rows * C.cols + 63) >> 6;
    const uint32_t nvw = static_cast<uint32_t>((C.cols + 63) >> 6);
    const uint32_t scan_waves = (nvw + 63) / 64;
    const uint32_t groups = gridDim.x;
    const uint32_t nrows = static_cast<uint32_t>((C.rows - blockIdx.x + groups - 1) / groups);  // of this workgroup
    const uintptr_t vbeg = reinterpret_cast<uintptr_t>(C.values), vend = vbeg + E * static_cast<uintptr_t>(C.nnz);

    uint32_t col[kQ], to[kQ];  // the column (0 where there is none), and where its value goes in an output row
#pragma unroll
    for (int u = 0; u < kQ; ++u) {
        const int64_t q = u * kThreads + threadIdx.x;
        const int64_t c = q < C.nsel ? C.sel[q] : -1;
        const bool live = static_cast<uint64_t>(c) < static_cast<uint64_t>(C.cols);  // others leave their output column untouched
        col[u] = live ? static_cast<uint32_t>(c) : 0u;
        to[u] = live ? static_cast<uint32_t>(q) * E : kOutside;
    }

    struct Row {  // wave-uniform
        int64_t first;    // index of its first value
        uint32_t shift;   // bytes of the staged units before that value
        uint32_t staged;  // values staged; 0: gathered from memory
    };
    auto row_index = [&](uint32_t k) { return int64_t(blockIdx.x) + int64_t(k) * groups; };
    // Its entry of row_offsets and the next one, as every lane loads them: the compiler would wait for a uniform load on the
    // spot, with everything that is in flight before it.
    struct Entries {
        int64_t first, next;
    };
    uint32_t zero;
    asm("v_mov_b32 %0, 0" : "=v"(zero));
    auto entries = [&](uint32_t k) {
        const int64_t i = row_index(k < nrows ? k : 0);
        const int64_t *at = C.row_offsets + i + zero;
        Entries e;
        e.first = at[0];
        e.next = at[i + 1 < C.rows ? 1 : 0];
        return e;
    };
    auto uniform = [](int64_t v) {
        return static_cast<int64_t>(uint64_t(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)))) << 32 |
                                    static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v))));
    };
    // the row's values asked for; more than fit, or over an end of the array: none
    auto ask = [&](uint32_t k, const Entries &loaded, u32x4 *buf, Row &R) {
        const int64_t i = row_index(k < nrows ? k : 0);
        Entries e;
        e.first = uniform(loaded.first);
        e.next = i + 1 < C.rows ? uniform(loaded.next) : C.nnz;
        const uintptr_t vaddr = vbeg + E * static_cast<uintptr_t>(e.first), a16 = vaddr & ~uintptr_t(15);
        const uint64_t count = e.first >= 0 && e.next > e.first && e.next <= C.nnz ? static_cast<uint64_t>(e.next - e.first) : 0;
        const uint64_t units = ((vaddr - a16) + E * count + 15) >> 4;
        const bool fits = k < nrows && count != 0 && units < kUnits && a16 >= vbeg && a16 + 16 * units <= vend;
        R.first = e.first;
        R.shift = static_cast<uint32_t>(vaddr - a16);
        R.staged = fits ? static_cast<uint32_t>(count) : 0u;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(fits ? a16 : vbeg), 0,
                                                                           fits ? static_cast<int>(16 * units) : 0, 0x00020000);
#pragma unroll
        for (int i = 0; i < Sh::kRounds; ++i)
            if ((i + 1) * kThreads <= int(kUnits) || i * kThreads + 64 * wave < kUnits)  // wave-uniform
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(buf + i * kThreads + 64 * wave), 16,
                                                         (i * kThreads + threadIdx.x) * 16, 0, 0, 2);
    };
    // this thread's word of the row's bitmap, in two halves: the loads, and what they mean
    struct Words {
        uint64_t lo, hi;
    };
    auto load_words = [&](uint32_t k) {
        const int64_t w0 = ((row_index(k < nrows ? k : 0) * C.cols) >> 6) + (threadIdx.x < nvw ? threadIdx.x : 0u);
        Words w;
        w.lo = C.bitmap[w0 < nwords ? w0 : nwords - 1];
        w.hi = C.bitmap[w0 + 1 < nwords ? w0 + 1 : nwords - 1];
        return w;
    };
    auto word_of = [&](uint32_t k, const Words &w) -> uint64_t {
        const int64_t row_bit = row_index(k) * C.cols;
        const uint32_t bs = static_cast<uint32_t>(row_bit & 63);
        uint64_t x = w.lo >> bs;
        if ((row_bit >> 6) + threadIdx.x + 1 < nwords) x |= (w.hi << 1) << (63 - bs);
        const int64_t left = C.cols - 64 * int64_t(threadIdx.x);
        if (left < 64) x = left > 0 ? x & ((uint64_t(1) << left) - 1) : 0;
        return x;
    };

    Entries e2 = entries(0);  // of the row whose values are asked for next
    Words w2 = load_words(0);
    uint64_t word1 = 0;       // of the row whose ranks are finished next: its word, and the 1 bits of the wave's words before
    uint32_t excl1 = 0;
    // Step j: the queries of row j - 2 are answered from `now`, the values of row j - 1 asked for.
    auto step = [&](uint32_t j, u32x4 *next, Row &Rn, const u32x4 *now, const Row &R) __attribute__((always_inline)) {
        const Entries e = e2;
        e2 = entries(j);
        __builtin_amdgcn_sched_barrier(0);
        ask(j - 1, e, next, Rn);
        __builtin_amdgcn_sched_barrier(0);

        // queries of row j - 2
        const uint32_t k = j - 2;
        const bool valid = k < nrows;  // (j < 2: no)
        const uint32_t carry = s_total[k & 1];
        const int64_t i = row_index(valid ? k : 0);
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(static_cast<uint8_t *>(C.out) + E * i * C.nsel, 0,
                                                                             valid ? static_cast<int>(E * C.nsel) : 0, 0x00020000);
        const uint64_t *pairs = reinterpret_cast<const uint64_t *>(s_pairs[k & 1]);
        uint32_t v[kQ], rank[kQ];
        bool hit[kQ];
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint64_t pair = pairs[col[u] >> 5];
            const uint32_t piece = static_cast<uint32_t>(pair), b = col[u] & 31;
            rank[u] = valid ? static_cast<uint32_t>(pair >> 32) + __popc(piece & ((1u << b) - 1)) : 0u;
            hit[u] = ((piece >> b) & 1) != 0;
        }
        // (carry: the row's 1 bits.  More than are staged: the next entry of row_offsets is not this row's end.)
        if (!valid || static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(carry))) <= R.staged) {
            const uint8_t *values = reinterpret_cast<const uint8_t *>(now) + R.shift;
#pragma unroll
            for (int u = 0; u < kQ; ++u)  // (a rank is at most the row's 1 bits: one value past them, in a spare unit)
                v[u] = (E == 2) ? uint32_t(reinterpret_cast<const uint16_t *>(values)[rank[u]]) : uint32_t(values[rank[u]]);
        } else {
            const uint64_t room = R.first >= 0 && R.first <= C.nnz ? static_cast<uint64_t>(C.nnz - R.first) : 0;
            const uint8_t *values = static_cast<const uint8_t *>(C.values) + E * R.first;
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                hit[u] = hit[u] && rank[u] < room;
                const uint8_t *at = hit[u] ? values + size_t(E) * rank[u] : reinterpret_cast<const uint8_t *>(C.sel);
                v[u] = (E == 2) ? uint32_t(*reinterpret_cast<const uint16_t *>(at)) : uint32_t(*at);
            }
            wait_loads_to_lds();
        }
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const Elem x = static_cast<Elem>(hit[u] ? v[u] : 0u);
            if constexpr (E == 2)
                __builtin_amdgcn_raw_buffer_store_b16(x, out, to[u], 0, 0);
            else
                __builtin_amdgcn_raw_buffer_store_b8(x, out, to[u], 0, 0);
        }

        if (wave < scan_waves) {
            // ranks of row j - 1 finished
            uint32_t before = 0, total = 0;
            const uint32_t c = lane < scan_waves ? s_count[(j - 1) & 1][lane < kWaves ? lane : 0] : 0u;
            before = wave_sum(lane < wave ? c : 0u);
            total = wave_sum(c);
            if (threadIdx.x == 0) s_total[(j - 1) & 1] = total;
            const uint32_t lo = static_cast<uint32_t>(word1), hi = static_cast<uint32_t>(word1 >> 32);
            u32x4 p;
            p.x = lo;
            p.y = before + excl1;
            p.z = hi;
            p.w = p.y + __popc(lo);
            s_pairs[(j - 1) & 1][threadIdx.x] = p;
            // the words of row j counted
            word1 = word_of(j < nrows ? j : 0, w2);
            const uint32_t pc = __popcll(word1), incl = wave_inclusive_scan(pc);
            excl1 = incl - pc;
            if (lane == 63) s_count[j & 1][wave] = incl;
            w2 = load_words(j + 1);
        }
        // the values asked for have arrived: behind them went the stores
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        wait_all_but<kQ>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    wait_loads_to_lds();
    Row R0{}, R1{};
    for (uint32_t j = 0; j < nrows + 2; j += 2) {
        step(j, s_v1, R1, s_v0, R0);
        step(j + 1, s_v0, R0, s_v1, R1);
    }
}

}  // namespace

#endif  // ENDOR_COLS_STREAM_H_
