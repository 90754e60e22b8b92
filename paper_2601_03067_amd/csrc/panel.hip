// Early rejection at the large heights of a tree call (early.hip): the heads of all pairs of a node's blocks, with the right
// blocks' heads held in registers.
//
// The head is short (nk of 64 slices, 10 at thr 0.9), so a wavefront can keep the heads of 64 right blocks in registers,
// as MFMA operands, and let the left blocks go by: every left fragment is read from LDS once per wavefront and feeds two MFMAs,
// a left row crosses L2 -> LDS once per 512 right blocks instead of once per 256, no right row does at all, and the
// workgroup meets at a barrier every 64 left rows instead of every 64-byte slice.  The test of a pair,
//     <a_head, b_head> > floor |a| |b| - (tail_a |a|) (tail_b |b|),
// is of rank two in (a, b): its right side is subtracted by the MFMA that starts a product (the two terms, each factor as three
// bfloat16 parts: panel_left, panel_right), so that all that is left to do with an accumulator is to look at its sign.
//
// What bounds it: the MFMA units, busy 65 % of the cycles at the largest heights, at a clock of 1.8 to 1.9 GHz
// (profiles/cases_kernels.md); the rest is the step from one 64-row stage to the next, where all wavefronts meet.  The ring kernel
// (similarity.hip) had them busy 43 % there: it spends 14 000 of the 24 000 cycles of a 256 x 256 tile on the tests and on the way
// from tile to tile.  Similarity of the largest node of 512 ragged requests (8 groups, some 45 000 blocks in each set): 14.2 -> 9.4 ms;
// the whole fusion of these 43.8 -> 32.5 ms, of 64 requests x 128 blocks in 256 groups (sets of 256 blocks and more) 19.9 -> 18.9 ms.
// Tried and dropped: each wavefront at its own pace, with counts in LDS of what has landed and what is done instead of the
// barrier (10 % slower: two round trips to LDS per 32 rows); fragments waited for where they are read (58 % busy).
#include <type_traits>

#include "items.h"

namespace kvfuse {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ floatx16 panel_mma(const u32x4 a, const u32x4 b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
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
__device__ __forceinline__ void landed_regs(u32x4 &a, u32x4 &b, u32x4 &c, u32x4 &d) { asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d)); }

__device__ __forceinline__ u32x4 lds_read(const char *at) { return *reinterpret_cast<const u32x4 *>(at); }

struct PanelArgs {
    PoolDesc pool;
    WorkDesc w;
    HeightDesc h;
    int32_t height;
    float thr_floor;
};

__global__ __launch_bounds__(512, 1) void similarity_panel_kernel(PanelArgs args)
{
    const PoolDesc &pool = args.pool;
    const WorkDesc &w = args.w;
    const HeightDesc &h = args.h;
    constexpr int NK = kPanelSlices, SLICE = kPanelRows * 64, MAXC = 2048;
    constexpr int DENSE = 32;           // open pairs of a wavefront's 32 x 64 from which they are multiplied whole
    __shared__ __attribute__((aligned(1024))) char stage[2][NK * SLICE];
    __shared__ __attribute__((aligned(1024))) u32x4 left_fc[2][2][2][32];      // left blocks' fragments of the test: [stage][32 rows][half][row]
    __shared__ int lds_n, lds_full[2], lds_first;
    __shared__ uint32_t lds_pair[MAXC];         // row of the item << 16 | column of the panel
    __shared__ __attribute__((aligned(1024))) u32x4 right_fc[8][2][64];        // right blocks': [wavefront][32 columns][lane]
    __shared__ uint32_t lds_dense[kPanelRun / 2];        // a bit per (stage, 32 rows of it, wavefront)

    const int total = w.panel_total[args.height];
    const int seat = blockIdx.x >> 3;
    const int v = (seat >> 5 << 8) + (int)((blockIdx.x & 7) << 5) + (seat & 31);      // the XCDs take 32 consecutive items in turn
    if (v >= total)
        return;
    const int4 item = w.panel_items[v];
    const int g = item.x, node = item.y, col0 = item.z, row0 = item.w;
    const int ml = w.set_cnt[(int64_t)g * w.n_slots + h.l_slot[node]];
    const int mr = w.set_cnt[(int64_t)g * w.n_slots + h.r_slot[node]];
    const int n_rows = min(ml - row0, panel_rows_per_item(ml, h.panel_run));
    const int n_stages = (n_rows + kPanelRows - 1) / kPanelRows;
    const int32_t *__restrict__ l_ids = w.set_ids + (int64_t)g * w.n + h.l_off[node] + row0;
    const int32_t *__restrict__ r_ids = w.set_ids + (int64_t)g * w.n + h.r_off[node] + col0;
    const int n_cols = min(mr - col0, kPanelCols);
    const int nk = w.early_nk[g];
    const int row_bytes = pool.r * 2;
    const char *__restrict__ kg = (const char *)pool.k + (int64_t)g * pool.P * row_bytes;
    const u32x4 *__restrict__ rows = w.panel_rows + ((int64_t)g * w.l_stride + h.l_base[node] + row0) * 2;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, half = lane >> 5;

    // A panel of more than 256 right blocks: a wavefront per 64 of them.  A narrower one: per 64 blocks two wavefronts, which take
    // turns at the left rows.
    const bool wide = n_cols > kPanelCols / 2;
    const int my_col = (wide ? wave : wave & 3) * 64;
    const int sub0 = wide ? 0 : wave >> 2, sub_step = wide ? 1 : 2;

    // ---- loaders: this lane's row of a stage, and its (swizzled) 16 bytes of every other slice of it.  (Buffer loads, whose
    // offsets have 32 bits: the compiler counts global loads into LDS among the LDS's own operations, whose order it then takes for
    // unknown, so that every wait for a fragment would be for all fragments on their way.)
    const __amdgpu_buffer_rsrc_t pool_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)kg, 0, 0xFFFFFFFFu, 0x00020000);
    const __amdgpu_buffer_rsrc_t rows_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)rows, 0, 0xFFFFFFFFu, 0x00020000);
    const int ld_row = (wave & 3) * 16 + (lane >> 2);
    const uint32_t ld_off = (uint32_t)((lane & 3) ^ ((lane >> 4) & 3)) * 16u;
    auto row_at = [&](int t) __attribute__((always_inline)) { return min(t * kPanelRows + ld_row, n_rows - 1); };
    auto load_stage = [&](int t, int id) __attribute__((always_inline)) {
        char *dst = stage[t & 1] + (wave >> 2) * SLICE + (wave & 3) * 1024;
        const uint32_t src = (uint32_t)id * (uint32_t)row_bytes + ld_off;
        for (int s = wave >> 2; s < nk; s += 2) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(pool_rsrc, (__attribute__((address_space(3))) void *)dst, 16, src, s * 64, 0, 0);
            dst += 2 * SLICE;
        }
        if (wave >= 6) {
            const int row = min(t * kPanelRows + (wave - 6) * 32 + l31, n_rows - 1);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rows_rsrc, (__attribute__((address_space(3))) void *)left_fc[t & 1][wave - 6], 16,
                                                     (uint32_t)(2 * row + half) * 16u, 0, 0, 0);
        }
    };

    if (tid == 0)
        lds_n = lds_full[0] = lds_full[1] = 0;
    if (tid < kPanelRun / 2)
        lds_dense[tid] = 0;
    int id = l_ids[row_at(0)];
    load_stage(0, id);
    id = l_ids[row_at(1)];
    const int frag = l31 * 64 + ((half ^ ((l31 >> 2) & 3)) * 16);
    // Once through this loop, unless the list of open pairs fills up on the way: then it is emptied, and the right blocks, whose
    // registers that takes, are loaded again.
    for (int t = 0;;) {
        u32x4 fb[NK][2][2];
        // (a row has more than NK slices: those past the group's nk are loaded and not used)
        each<2>([&](auto c) __attribute__((always_inline)) {
            const int col = my_col + 32 * c + l31;
            const int rid = r_ids[min(col, n_cols - 1)];
            const char *src = kg + ((int64_t)rid * row_bytes + half * 16);
            each<NK>([&](auto s) __attribute__((always_inline)) {
                fb[s][0][c] = *reinterpret_cast<const u32x4 *>(src + 64 * s);
                fb[s][1][c] = *reinterpret_cast<const u32x4 *>(src + 64 * s + 32);
            });
            const int64_t b = (int64_t)g * pool.P + rid;
            const float norm = panel_norm(pool, b);
            // past the last column: a floor of 16 times the norms, above every cosine (thr_floor > 1/4)
            right_fc[wave][c][lane] = panel_right(col < n_cols ? norm : 16.0f * norm, col < n_cols ? w.rem_k[b] * norm : 0.0f, half);
        });
        // whole before the loop: nothing in it may wait for these loads behind the ones into LDS
        each<NK>([&](auto s) __attribute__((always_inline)) { landed_regs(fb[s][0][0], fb[s][0][1], fb[s][1][0], fb[s][1][1]); });

        for (; t < n_stages; ++t) {
            // this wavefront's loads of stage t have landed; behind the barrier all have, and nobody reads stage t - 1 any more
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            // half full in stage t - 1?  (What stage t marks is the other word's, so that no wavefront runs ahead of another's look.)
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(__hip_atomic_load(&lds_full[(t + 1) & 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)), 0))
                break;
            if (t + 1 < n_stages) {
                load_stage(t + 1, id);
                id = l_ids[row_at(t + 2)];
            }
            if (my_col >= n_cols)
                continue;
#pragma unroll 1
            for (int sub = sub0; sub < 2; sub += sub_step) {
                int n_slices = nk;
                asm volatile("" : "+s"(n_slices));      // (or the comparisons below are kept for the whole loop, in two registers each)
                const char *at0 = stage[t & 1] + frag + sub * 2048, *at1 = stage[t & 1] + (frag ^ 32) + sub * 2048;
                // Four fragments are on their way or in use at a time: one is asked for as soon as the products of its place's last one are
                // issued, the products of three fragments ahead of its own.  (Behind the last slice: whatever is there, not used.)
                u32x4 fa[4] = {lds_read(at0), lds_read(at1), lds_read(at0 + SLICE), lds_read(at1 + SLICE)};
                floatx16 acc0, acc1;
                {
                    const u32x4 fl = left_fc[t & 1][sub][half][l31];
                    floatx16 zero;
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        zero[e] = 0.0f;
                    acc0 = panel_mma(fl, right_fc[wave][0][lane], zero);
                    acc1 = panel_mma(fl, right_fc[wave][1][lane], zero);
                }
                __builtin_amdgcn_sched_barrier(0);
                each<NK>([&](auto s) __attribute__((always_inline)) {
                    if (s < n_slices) {
                        constexpr int i = 2 * (s & 1);
                        acc0 = panel_mma(fa[i], fb[s][0][0], acc0);
                        acc1 = panel_mma(fa[i], fb[s][0][1], acc1);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (s + 2 < NK)
                            fa[i] = lds_read(at0 + (s + 2) * SLICE);
                        __builtin_amdgcn_sched_barrier(0);
                        acc0 = panel_mma(fa[i + 1], fb[s][1][0], acc0);
                        acc1 = panel_mma(fa[i + 1], fb[s][1][1], acc1);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (s + 2 < NK)
                            fa[i + 1] = lds_read(at1 + (s + 2) * SLICE);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
                float mx0 = -1.0f, mx1 = -1.0f;
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    mx0 = fmaxf(fmaxf(acc0[e], acc0[e + 1]), mx0);
                    mx1 = fmaxf(fmaxf(acc1[e], acc1[e + 1]), mx1);
                }
                if (__builtin_expect(__any(fmaxf(mx0, mx1) >= 0.0f), 0)) {
                    const int r0 = sub * 32 + 4 * half;               // element e: row r0 + 8 (e / 4) + e % 4 of the stage
                    uint32_t closed = 0;                              // bit 31 - e: acc0[e], bit 15 - e: acc1[e]; their signs
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        closed = __builtin_amdgcn_alignbit(closed, __float_as_uint(acc0[e]), 31);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        closed = __builtin_amdgcn_alignbit(closed, __float_as_uint(acc1[e]), 31);
                    uint32_t mask = ~closed;
                    int open = 0;
                    unsigned long long lanes;
                    for (uint32_t m = mask; (lanes = __ballot(m != 0)) != 0 && open <= DENSE; m &= m - 1)
                        open += __popcll(lanes);
                    if (__builtin_expect(open <= DENSE, 1)) {
                        int k = 0;
                        if (lane == 0) {
                            k = atomicAdd(&lds_n, open);       // (16 x DENSE a stage at most: never beyond MAXC)
                            if (k + open > MAXC / 2)
                                lds_full[t & 1] = 1;
                        }
                        k = __builtin_amdgcn_readfirstlane(k);
                        for (; (lanes = __ballot(mask != 0)) != 0; mask &= mask - 1) {
                            if (mask) {
                                const int bit = __builtin_ctz(mask), e = 15 - (bit & 15);
                                const int slot = k + __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0));
                                lds_pair[slot] = (uint32_t)(t * kPanelRows + r0 + 8 * (e >> 2) + (e & 3)) << 16 |
                                                 (uint32_t)(my_col + (bit < 16 ? 32 : 0) + l31);
                            }
                            k += __popcll(lanes);
                        }
                    } else if (lane == 0) {
                        atomicOr(&lds_dense[t >> 1], 1u << ((t & 1) * 16 + sub * 8 + wave));
                    }
                }
            }
        }

        // ---- the list's pairs go out to the pair list; what does not fit there is finished here, a wavefront per pair
        __syncthreads();
        const PanelArgs &again = kernel_args_again<PanelArgs>();
        const PoolDesc &pool = again.pool;
        const WorkDesc &w = again.w;
        const HeightDesc &h = again.h;
        const float thr_floor = again.thr_floor;
        const int64_t cbase = (int64_t)g * w.r_stride + h.r_base[node] + col0;
        const float *__restrict__ inv = pool.inv_norm_k + (int64_t)g * pool.P;
        const int n = lds_n;
        if (tid == 0 && n > 0) {
            lds_first = atomicAdd(w.n_pairs, n);
            atomicAdd(&w.open_cnt[g], n);
            if (n > kWholeTile)
                w.whole[g] = 1;                  // (some: how many, only the ring kernel counts)
        }
        __syncthreads();
        const int first = n > 0 ? lds_first : 0;
        for (int k = tid; k < n; k += 512) {
            const int row = (int)(lds_pair[k] >> 16), col = (int)(lds_pair[k] & 0xFFFFu);
            const bool real = row < n_rows;              // (a row past the end is the last one again)
            if (first + k < w.pair_cap)
                w.pairs[first + k] = make_int4(real ? (int)(cbase + col) : -1, (row0 + row) | kPairWhole, l_ids[min(row, n_rows - 1)], r_ids[col]);
        }
        for (int k = max(0, w.pair_cap - first) + wave; k < n; k += 8) {
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
        for (int word = 0; word < (n_stages + 1) / 2; ++word) {
            uint32_t bits = __builtin_amdgcn_readfirstlane(lds_dense[word]);
            for (int i = 0; bits; bits &= bits - 1, ++i) {
                if ((i & 7) != wave)
                    continue;
                const int bit = __builtin_ctz(bits);
                const int r0 = (2 * word + (bit >> 4)) * kPanelRows + ((bit >> 3) & 1) * 32, c0 = (wide ? bit & 7 : bit & 3) * 64;
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
                    w.whole[g] = 1;
                }
            }
        }
        break;
    }
}

// The panel kernel's share of a height's similarity step; the ring kernel takes the groups that are not panel_on.
void launch_similarity_panel(hipStream_t s, const PoolDesc &pool, const WorkDesc &w, const HeightDesc &h, int height, float thr_floor)
{
    const int64_t items = ((int64_t)w.G * h.panel_items + 255) / 256 * 256;
    similarity_panel_kernel<<<(unsigned)items, 512, 0, s>>>(PanelArgs{pool, w, h, height, thr_floor});
}

}  // namespace kvfuse
