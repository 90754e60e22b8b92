// Early rejection at the large heights of a tree call (early.hip): the head copies (heads.hip) of all pairs of a node's blocks, with the
// right blocks' copies held in registers.
//
// A copy is short (up to 384 elements of six bits), so a wavefront can keep those of 128 right blocks in registers, as MFMA operands, and
// let the left blocks go by: every left fragment is read from LDS once per wavefront and feeds four MFMAs, a left row crosses
// L2 -> LDS once per 512 right blocks, no right row does at all, and the workgroup meets at a barrier every 64 left rows.  The
// test of a pair is what its product starts from, by one MFMA (items.h), so that all that is left to do with an accumulator is to look at its
// sign.  A workgroup has four wavefronts and a compute unit holds two, whose barriers, tests and first loads the other one's
// products cover.
//
// What bounds it: power.  At the largest heights the MFMA units are busy 64 to 67 % of the cycles at 1.65 to 1.8 GHz; the same instructions on the
// same kind of data do not get beyond 1.4 GHz from registers (5.8 PFLOP/s against 9.9 at 2.4 GHz on zeros).  With heads of bfloat16 from the
// pool (10 or 11 slices, 22 MFMAs of 32 x 32 x 16 instead of 6 of 32 x 32 x 64 and the test's) the largest node of 512 ragged requests (8
// groups, some 45 000 blocks in each set) took 9.1 ms, now 3.2; the whole fusion of these 32.2 -> 18.6 ms, of 64 requests x 128 blocks in 256
// groups 18.8 -> 17.8 ms.
// Tried and dropped: three stages in LDS instead of two (unchanged); the accumulators looked at two by two with the next rows' products
// begun behind that, across the barrier (1 % fewer cycles, the same time); loads into LDS between products (registers spill); wavefronts of
// a workgroup or around products at a higher priority (unchanged); eight wavefronts of 64 right blocks, each at its own pace, with counts
// in LDS instead of the barrier (10 % slower: two round trips to LDS per 32 rows).
#include <type_traits>

#include "items.h"

namespace kvfuse {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

typedef short i16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx16 test_mma(const u32x2 a, const u32x2 b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(i16x4, a), __builtin_bit_cast(i16x4, b), c, 0, 0, 0);
}

__device__ __forceinline__ floatx16 panel_mma(const u32x4 a, const u32x4 b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 64 elements of e2m3 (format 2), 32 of them in a lane's six registers.
typedef int32_t i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));
__device__ __forceinline__ floatx16 head_mma(const u32x6 a, const u32x6 b, floatx16 c)
{
    auto wide = [](const u32x6 x) { return i32x8{(int)x[0], (int)x[1], (int)x[2], (int)x[3], (int)x[4], (int)x[5], 0, 0}; };
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wide(a), wide(b), c, 2, 2, 0, 0, 0, 0);
}
// A step's six registers from the three pieces of its pair of steps.
template <bool HIGH>
__device__ __forceinline__ u32x6 of_pieces(const u32x4 x, const u32x4 y, const u32x4 z)
{
    return HIGH ? u32x6{y[2], y[3], z[0], z[1], z[2], z[3]} : u32x6{x[0], x[1], x[2], x[3], y[0], y[1]};
}

// body(0), ..., body(N - 1) with the index a constant from the start: register arrays that loops index before they are unrolled
// would live in scratch memory.
template <int N, typename F>
__device__ __forceinline__ void each(F body)
{
    if constexpr (N > 0) {
        each<N - 1>(body);
        body(std::integral_constant<int, N - 1>{});
    }
}

// Nothing behind this waits for loads into these registers any more.
__device__ __forceinline__ void landed_regs(u32x6 &a) { asm volatile("" : "+v"(a)); }

__device__ __forceinline__ u32x4 lds_read(const char *at) { return *reinterpret_cast<const u32x4 *>(at); }

// Five loads of 16 bytes a lane into LDS: 64 bytes on in memory, QUAD on in LDS (an instruction's offset counts on either side).  In
// assembly, because the compiler makes every LDS read wait for all such loads of its own, whichever buffer they are for; who issues
// them waits for them by hand.  (No register is loaded.  The pause is for scalar registers that a vector instruction has just written, and for m0.)
template <int QUAD>
__device__ __forceinline__ void quads_to_lds(uint64_t base, uint32_t off, uint32_t to)
{
    typedef uint32_t desc_t __attribute__((ext_vector_type(4)));
    const desc_t desc = {(uint32_t)base, (uint32_t)(base >> 32), 0xFFFFFFFFu, 0x00020000u};
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\t"
                 "buffer_load_dwordx4 %0, %1, 0 offen lds\n\t"
                 "s_add_i32 m0, %2, %3\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %0, %1, 0 offen offset:64 lds\n\t"
                 "s_add_i32 m0, %2, 2 * %3\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %0, %1, 0 offen offset:128 lds\n\t"
                 "s_add_i32 m0, %2, 3 * %3\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %0, %1, 0 offen offset:192 lds\n\t"
                 "s_add_i32 m0, %2, 4 * %3\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %0, %1, 0 offen offset:256 lds" ::"v"(off), "s"(desc), "s"(to), "n"(QUAD - 64) : "memory", "m0", "scc");
}

struct PanelArgs {
    PoolDesc pool;
    WorkDesc w;
    int32_t height;
    float thr_floor;
};

template <bool LONG>
__global__ __launch_bounds__(256, 2) void similarity_panel_kernel(PanelArgs args)
{
    using S = HeadShape<LONG>;
    const WorkDesc &w = args.w;
    constexpr int STEPS = S::steps, HEAD = S::bytes, ROWS = S::rows, COLS = S::cols, NC = COLS / 128, QUAD = ROWS * 64, STAGE = HEAD / 64 * QUAD;
    constexpr int MAXC = 2048, TEST = 3 * STEPS / 2;
    // Open pairs of a wavefront's 32 x 64 from which they are multiplied whole: as many as the list has room for (as one or two wavefronts
    // walk along a piece's rows alone while the rest of the chip is done: 128 pieces in a height, 120 us with them in the list, 336 without).
    constexpr int DENSE = LONG ? 256 : 64;
    // Two stages of left rows, four pieces of 16 bytes of a row side by side, as many times as a copy has four.
    __shared__ __attribute__((aligned(1024))) char stages[2 * STAGE];
    __shared__ int lds_n, lds_full[2], lds_first;
    __shared__ uint32_t lds_pair[MAXC];         // row of the item << 16 | column of the panel
    __shared__ __attribute__((aligned(1024))) u32x2 right_fc[4][NC][64];       // right blocks' operands of the test: [wavefront][32 columns][lane]
    constexpr int DENSE_WORDS = kPanelRun * ROWS / 32 * (COLS / 64) / 32;
    __shared__ uint32_t lds_dense[DENSE_WORDS];          // a bit per (32 rows, 64 columns)

    static_assert(4 * (ROWS / 32) * (NC / 2) * DENSE <= MAXC / 2, "a stage's pairs fit half the list");

    const int total = w.panel_total[args.height];
    const int seat = blockIdx.x >> 3;
    const int v = (seat >> 6 << 9) + (int)((blockIdx.x & 7) << 6) + (seat & 63);      // the XCDs take 64 consecutive items in turn
    if (v >= total)
        return;
    const int4 item = w.panel_items[2 * (int64_t)v], item2 = w.panel_items[2 * (int64_t)v + 1];
    const int g = item.x, n_rows = item.w >> 16, n_cols = item.w & 0xFFFF, steps = item2.z;
    const int n_stages = (n_rows + ROWS - 1) / ROWS;
    const int32_t *__restrict__ l_places = w.set_slot + (int64_t)g * w.n + item.y;
    const int32_t *__restrict__ r_places = w.set_slot + (int64_t)g * w.n + item.z;
    const char *__restrict__ heads = w.heads + (int64_t)g * w.n * HEAD;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, half = lane >> 5;

    // A panel of more than half its right blocks: a wavefront per quarter of them.  A narrower one: per quarter two wavefronts, which take
    // turns at the left rows, at 32 at a time.
    const bool wide = n_cols > COLS / 2;
    const int my_col = (wide ? wave : wave & 1) * (COLS / 4);
    const int sub0 = wide || ROWS == 32 ? 0 : wave >> 1, sub_step = wide ? 1 : 2;

    // ---- loaders: this lane's row of a stage, and its (swizzled) piece of every four
    // (a wavefront takes 16 rows, or half of their pieces)
    constexpr int PARTS = 64 / ROWS;
    const int ld_wave = wave % (ROWS / 16), ld_part = wave / (ROWS / 16);
    static_assert(PARTS * 320 == HEAD, "five loads of 64 bytes a row for each part");
    const uint64_t heads_at = (uint64_t)heads;
    const uint32_t stage_at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)stages) + (uint32_t)ld_wave * 1024u + (uint32_t)ld_part * (5u * QUAD);
    const int ld_row = ld_wave * 16 + (lane >> 2);
    const uint32_t ld_off = (uint32_t)((lane & 3) ^ ((lane >> 4) & 3)) * 16u + (uint32_t)ld_part * 320u;
    auto row_of = [&](int t) __attribute__((always_inline)) { return (uint32_t)l_places[min(t * ROWS + ld_row, n_rows - 1)] * (uint32_t)HEAD; };
    auto load_stage = [&](uint32_t row, uint32_t at) __attribute__((always_inline)) { quads_to_lds<QUAD>(heads_at, row + ld_off, stage_at + at); };

    if (tid == 0)
        lds_n = lds_full[0] = lds_full[1] = 0;
    if (tid < DENSE_WORDS)
        lds_dense[tid] = 0;
    uint32_t row = row_of(0);
    load_stage(row, 0);
    row = row_of(1);
    const int frag = l31 * 64 + ((half ^ ((l31 >> 2) & 3)) * 16);         // piece 2 m + half: every second m, 32 bytes on; another quad every two
    const int test_at = (TEST >> 1) * QUAD + ((l31 * 64 + ((l31 >> 2) & 3) * 16) ^ (TEST & 1 ? 32 : 0)) + half * 8;       // the piece behind the codes: eight bytes for either half
    // Once through this loop, unless the list of open pairs fills up on the way: then it is emptied, and the right blocks, whose
    // registers that takes, are loaded again.
    for (int t = 0;;) {
        u32x6 fb[STEPS][NC];
        each<NC>([&](auto c) __attribute__((always_inline)) {
            const int col = my_col + 32 * c + l31;
            const char *src = heads + ((int64_t)r_places[min(col, n_cols - 1)] * HEAD + half * 16);
            each<STEPS / 2>([&](auto p) __attribute__((always_inline)) {
                u32x4 x[3];
                each<3>([&](auto j) __attribute__((always_inline)) { x[j] = *reinterpret_cast<const u32x4 *>(src + (3 * p + j) * 32); });
                fb[2 * p][c] = of_pieces<false>(x[0], x[1], x[2]);
                fb[2 * p + 1][c] = of_pieces<true>(x[0], x[1], x[2]);
            });
            u32x2 test = *reinterpret_cast<const u32x2 *>(src + (2 * TEST + 1) * 16 - 8 * half);
            // past the last column: a floor of 2^30 times the left norm, above every product
            if (col >= n_cols)
                test = panel_right(0x1p30f, 0.0f, 0.0f, 0.0f, half);
            right_fc[wave][c][lane] = test;
        });
        // whole before the loop: nothing in it may wait for these loads behind the ones into LDS
        each<STEPS>([&](auto s) __attribute__((always_inline)) { each<NC>([&](auto c) __attribute__((always_inline)) { landed_regs(fb[s][c]); }); });

        for (; t < n_stages; ++t) {
            // this wavefront's loads of stage t have landed; behind the barrier all have, and nobody reads stage t - 1 any more
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            // half full in stage t - 1?  (What stage t marks is the other word's, so that no wavefront runs ahead of another's look.)
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(__hip_atomic_load(&lds_full[(t + 1) & 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)), 0))
                break;
            if (t + 1 < n_stages) {
                load_stage(row, (uint32_t)((t + 1) & 1) * STAGE);
                row = row_of(t + 2);
            }
            if (my_col >= n_cols || (ROWS == 32 && !wide && (t & 1) != wave >> 1))
                continue;
            const char *stage = stages + (t & 1) * STAGE;
            // A step's fragment of 32 left rows (at `rows`): pieces 3 p, 3 p + 1 and 3 p + 2 of a pair of steps hold its first 16 bytes, eight
            // of either step, and the second's last 16.
            auto fragment = [&](const char *rows, auto s) __attribute__((always_inline)) {
                constexpr int m = 3 * (s / 2) + 2 * (s & 1), y = 3 * (s / 2) + 1;
                const u32x4 x4 = lds_read(rows + (m & 1 ? frag ^ 32 : frag) + (m >> 1) * QUAD);
                const u32x2 x2 = *reinterpret_cast<const u32x2 *>(rows + (y & 1 ? frag ^ 32 : frag) + (y >> 1) * QUAD + 8 * (s & 1));
                return s & 1 ? u32x6{x2[0], x2[1], x4[0], x4[1], x4[2], x4[3]} : u32x6{x4[0], x4[1], x4[2], x4[3], x2[0], x2[1]};
            };
            // Three fragments are on their way or in use at a time: a step's place is asked for anew as soon as its products are issued.
            u32x6 fa[3];
            each<3>([&](auto s) __attribute__((always_inline)) { fa[s] = fragment(stage + sub0 * 2048, s); });
#pragma unroll 1
            for (int sub = sub0; sub < ROWS / 32; sub += sub_step) {
                const char *rows = stage + sub * 2048;
                int n_steps = steps;
                asm volatile("" : "+s"(n_steps));      // (or the comparisons below are kept for the whole loop, in two registers each)
                floatx16 acc[NC];
                {
                    const u32x2 fl = *reinterpret_cast<const u32x2 *>(rows + test_at);
                    floatx16 zero;
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        zero[e] = 0.0f;
                    each<NC>([&](auto c) __attribute__((always_inline)) { acc[c] = test_mma(fl, right_fc[wave][c][lane], zero); });
                }
                __builtin_amdgcn_sched_barrier(0);
                each<STEPS>([&](auto s) __attribute__((always_inline)) {
                    if (s < n_steps)
                        each<NC>([&](auto c) __attribute__((always_inline)) { acc[c] = head_mma(fa[s % 3], fb[s][c], acc[c]); });
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (s + 3 < STEPS)
                        fa[s % 3] = fragment(rows, std::integral_constant<int, s + 3>{});
                    else if constexpr (ROWS > 32)             // (behind the last rows: whatever is there, not used)
                        fa[s % 3] = fragment(rows + 2048, std::integral_constant<int, s + 3 - STEPS>{});
                    __builtin_amdgcn_sched_barrier(0);
                });
                float mx[NC], most = -1.0f;
                each<NC>([&](auto c) __attribute__((always_inline)) {
                    mx[c] = -1.0f;
#pragma unroll
                    for (int e = 0; e < 16; e += 2)
                        mx[c] = fmaxf(fmaxf(acc[c][e], acc[c][e + 1]), mx[c]);
                });
                each<NC>([&](auto c) __attribute__((always_inline)) { most = fmaxf(most, mx[c]); });
                if (__builtin_expect(!__any(most >= 0.0f), 1))
                    continue;
                const int r0 = sub * 32 + 4 * half;               // element e: row r0 + 8 (e / 4) + e % 4 of the stage
                each<NC / 2>([&](auto cc) __attribute__((always_inline)) {
                    uint32_t closed = 0;                          // bit 31 - e: the first 32 columns, bit 15 - e: the others; their signs
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        closed = __builtin_amdgcn_alignbit(closed, __float_as_uint(acc[2 * cc][e]), 31);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        closed = __builtin_amdgcn_alignbit(closed, __float_as_uint(acc[2 * cc + 1][e]), 31);
                    uint32_t mask = ~closed;
                    int open = 0;
                    unsigned long long lanes;
                    for (uint32_t m = mask; (lanes = __ballot(m != 0)) != 0 && open <= DENSE; m &= m - 1)
                        open += __popcll(lanes);
                    if (open == 0)
                        return;
                    if (__builtin_expect(open <= DENSE, 1)) {
                        int k = 0;
                        if (lane == 0) {
                            k = atomicAdd(&lds_n, open);       // (MAXC / 2 a stage at most: never beyond MAXC)
                            if (k + open > MAXC / 2)
                                lds_full[t & 1] = 1;
                        }
                        k = __builtin_amdgcn_readfirstlane(k);
                        for (; (lanes = __ballot(mask != 0)) != 0; mask &= mask - 1) {
                            if (mask) {
                                const int bit = __builtin_ctz(mask), e = 15 - (bit & 15);
                                const int slot = k + __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0));
                                lds_pair[slot] = (uint32_t)(t * ROWS + r0 + 8 * (e >> 2) + (e & 3)) << 16 |
                                                 (uint32_t)(my_col + 64 * cc + (bit < 16 ? 32 : 0) + l31);
                            }
                            k += __popcll(lanes);
                        }
                    } else if (lane == 0) {
                        const int bit = (t * (ROWS / 32) + sub) * (COLS / 64) + (my_col >> 6) + cc;
                        atomicOr(&lds_dense[bit >> 5], 1u << (bit & 31));
                    }
                });
            }
        }

        // ---- the list's pairs go out to the pair list; what does not fit there is finished here, a wavefront per pair
        __syncthreads();
        const PanelArgs &again = kernel_args_again<PanelArgs>();
        const PoolDesc &pool = again.pool;
        const WorkDesc &w = again.w;
        const int row_bytes = pool.r * 2, row0 = item2.y;
        const char *__restrict__ kg = (const char *)pool.k + (int64_t)g * pool.P * row_bytes;
        const int32_t *__restrict__ l_ids = w.set_ids + (int64_t)g * w.n + item.y;
        const int32_t *__restrict__ r_ids = w.set_ids + (int64_t)g * w.n + item.z;
        const float thr_floor = again.thr_floor;
        const int64_t cbase = (int64_t)g * w.r_stride + item2.x;
        const float *__restrict__ inv = pool.inv_norm_k + (int64_t)g * pool.P;
        const int n = lds_n;
        if (tid == 0 && n > 0) {
            lds_first = atomicAdd(w.n_pairs, n);
            atomicAdd(&w.open_cnt[g], n);
            if (n > kWholeTile)
                w.whole[g] = -1;                 // (some: how many, only the ring kernel counts)
        }
        __syncthreads();
        const int first = n > 0 ? lds_first : 0;
        for (int k = tid; k < n; k += 256) {
            const int row = (int)(lds_pair[k] >> 16), col = (int)(lds_pair[k] & 0xFFFFu);
            const bool real = row < n_rows;              // (a row past the end is the last one again)
            if (first + k < w.pair_cap)
                w.pairs[first + k] = make_int4(real ? (int)(cbase + col) : -1, (row0 + row) | kPairWhole, l_ids[min(row, n_rows - 1)], r_ids[col]);
        }
        for (int k = max(0, w.pair_cap - first) + wave; k < n; k += 4) {
            const int row = (int)(lds_pair[k] >> 16), col = (int)(lds_pair[k] & 0xFFFFu);
            if (row >= n_rows)
                continue;
            const int a = l_ids[row], b = r_ids[col];
            float dot = product_from<bf16_t>((const bf16_t *)(kg + (int64_t)a * row_bytes), (const bf16_t *)(kg + (int64_t)b * row_bytes), 0,
                                             row_bytes >> 4, lane, 64);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
                dot += __shfl_xor(dot, off, 64);
            const float cs = dot * inv[a] * inv[b];
            if (lane == 0 && cs > thr_floor)
                emit_candidate(w.cand_cnt, w.cand_idx, w.cand_val, cbase + col, w.cand_cap, row0 + row, cs);
        }
        __syncthreads();
        if (t < n_stages) {
            if (tid == 0)
                lds_n = lds_full[0] = lds_full[1] = 0;
            __syncthreads();
            continue;
        }

        // ---- pieces of 32 x 64 with many open pairs: whole products, straight from memory, and the candidates at once
        for (int word = 0; word < DENSE_WORDS; ++word) {
            uint32_t bits = __builtin_amdgcn_readfirstlane(lds_dense[word]);
            for (int i = 0; bits; bits &= bits - 1, ++i) {
                if ((i & 3) != wave)
                    continue;
                const int piece = word * 32 + __builtin_ctz(bits);
                const int r0 = piece / (COLS / 64) * 32, c0 = piece % (COLS / 64) * 64;
                floatx16 acc0, acc1;
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    acc0[e] = acc1[e] = 0.0f;
                const char *pa = kg + ((int64_t)l_ids[min(r0 + l31, n_rows - 1)] * row_bytes + half * 16);
                const char *pb0 = kg + ((int64_t)r_ids[min(c0 + l31, n_cols - 1)] * row_bytes + half * 16);
                const char *pb1 = kg + ((int64_t)r_ids[min(c0 + 32 + l31, n_cols - 1)] * row_bytes + half * 16);
                for (int s = 0; s < row_bytes; s += 128) {
                    u32x4 xa[4], x0[4], x1[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        xa[q] = *reinterpret_cast<const u32x4 *>(pa + s + 32 * q);
                        x0[q] = *reinterpret_cast<const u32x4 *>(pb0 + s + 32 * q);
                        x1[q] = *reinterpret_cast<const u32x4 *>(pb1 + s + 32 * q);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        acc0 = panel_mma(xa[q], x0[q], acc0);
                        acc1 = panel_mma(xa[q], x1[q], acc1);
                    }
                }
                const float ir0 = inv[r_ids[min(c0 + l31, n_cols - 1)]], ir1 = inv[r_ids[min(c0 + 32 + l31, n_cols - 1)]];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = r0 + 4 * half + 8 * (e >> 2) + (e & 3);
                    const float il = inv[l_ids[min(row, n_rows - 1)]];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int col = c0 + 32 * c + l31;
                        const float cs = (c == 0 ? acc0[e] * il * ir0 : acc1[e] * il * ir1);
                        if (row < n_rows && col < n_cols && cs > thr_floor)
                            emit_candidate(w.cand_cnt, w.cand_idx, w.cand_val, cbase + col, w.cand_cap, row0 + row, cs);
                    }
                }
                if (lane == 0) {
                    atomicAdd(&w.open_cnt[g], DENSE + 1);
                    w.whole[g] = -1;
                }
            }
        }
        break;
    }
}

// The panel kernel's share of a height's similarity step; the ring kernel takes the groups that are not panel_on.
void launch_similarity_panel(hipStream_t s, const PoolDesc &pool, const WorkDesc &w, const HeightDesc &h, int height, float thr_floor)
{
    const int64_t items = ((int64_t)w.G * h.panel_items[w.long_heads] + 511) / 512 * 512;
    const PanelArgs args{pool, w, height, thr_floor};
    if (w.long_heads)
        similarity_panel_kernel<true><<<(unsigned)items, 256, 0, s>>>(args);
    else
        similarity_panel_kernel<false><<<(unsigned)items, 256, 0, s>>>(args);
}

}  // namespace kvfuse
