// A whole tree call (norms, every height's similarity, assignment and merge, table rewrite) on groups of at most 64 table entries, in
// one launch of a workgroup per group.
//
// Everything of such a call is latency: as separate launches it is some nineteen kernels of 2 to 11 us, each waiting for the one
// before it.  A group is no one else's business, so one workgroup can take it from end to end: sets, norms, assignments and the
// remap table live in LDS, blocks come from the L2, and the steps of Algorithm 1 are separated by barriers.  With so few pairs there is
// nothing to screen: every cosine is taken in binary64, by the operations of the re-check (assign.hip) in their order, and
// merges and norms are summed in the order of the kernels they stand in for, so tables, blocks and norms are the same bits.
//
// What it costs now: vector instructions of the cosines (a row is widened for every column it meets) and, between them, chains through
// LDS: of 32 us the norms take 2, the cosines 10, sets and merges 14, the rewrite 5.  4 requests of 8 blocks in binary32, 2
// groups: 40.6 -> 31.9 us since keys stay in LDS, four rows share the exchanges of their sums and a division, and blocks are asked for
// one ahead; with statistics and the restoring of the blocks between calls 71 -> 64 us (134 launch by launch).
#include "common.h"

namespace kvfuse {

// Sixteen wavefronts, or eight where a lane's share of a merge takes more than half of sixteen wavefronts' registers.
template <typename T, int CPL>
constexpr int kTinyThreads = CPL * Elem<T>::PER16 > 16 ? 512 : 1024;

// Bytes of a group's keys that fit beside the tables (27 KB) in a compute unit's LDS.
constexpr int64_t kTinyStage = 132 << 10;

struct TinyArgs {
    PoolDesc pool;
    TableDesc tab;
    WorkDesc w;
    const int32_t *slot_init;
    int32_t n_heights;
    double thr, band;
    float thr_floor;
    int32_t *free_list, *n_free, *n_phys;
};

// (The orders of summation below are those of block_norms_kernel, cosines_f64_reg and merge_group_kernel.)
// STAGED: the group's keys stay in LDS from the norm pass on (kTinyStage bytes of it), where a row is a tenth of a trip to the L2 away.
template <typename T, int CPL, bool STAGED>
__global__ __launch_bounds__((kTinyThreads<T, CPL>)) void tiny_tree_kernel(TinyArgs A)
{
    constexpr int PER = Elem<T>::PER16, KW = !STAGED && CPL * PER == 16 ? 2 : 4;      // left rows side by side
    constexpr int NT = kTinyThreads<T, CPL>, NW = NT / 64;
    constexpr bool PAIR = PER == 4 && CPL == 4;      // a merge that merge_group_kernel gives to two wavefronts: two partial sums
    __shared__ double nk[kTinyPool], nv[kTinyPool];
    __shared__ int32_t refs[kTinyPool], remap[kTinyPool];
    __shared__ int32_t bt[kTinyEntries], ids[kTinyEntries], was[kTinyEntries], assign[kTinyEntries];
    __shared__ unsigned long long tgt_mask[kTinyEntries];      // merges of a height: members (bits of the right set) of a target ...
    __shared__ int32_t tgt[kTinyEntries], tgt_right[kTinyEntries];      // ... its place in ids, and the right set's
    __shared__ int32_t cnt[kTinySlots], counters[8], n_tgt;
    // by column, as the work arrays have them at the end: assignments, and the last height's cosines above the screen's floor
    __shared__ int32_t col_assign[kTinyEntries], col_cnt[kTinyEntries];
    __shared__ float col_val[kTinyEntries][kTinyEntries];
    __shared__ int4 nodes[kTinySlots];               // (a node is two of them, and fewer than half the slots are nodes')
    extern __shared__ uint4 keys[];                  // STAGED: [P][chunks]

    const PoolDesc &pool = A.pool;
    const TableDesc &tab = A.tab;
    const WorkDesc &w = A.w;
    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = w.n, P = pool.P, chunks = pool.r / PER;
    const int64_t gp = (int64_t)g * P, gn = (int64_t)g * n;
    T *const kp = (T *)pool.k + gp * pool.r, *const vp = (T *)pool.v + gp * pool.r;
    auto chunk_of = [&](int c) __attribute__((always_inline)) { return min(lane + 64 * c, chunks - 1); };
    auto in_block = [&](int c) __attribute__((always_inline)) { return lane + 64 * c < chunks; };
    // chunk c of a lane's share of a key block
    auto key_chunk = [&](int b, int c) __attribute__((always_inline)) {
        return STAGED ? keys[b * chunks + chunk_of(c)] : reinterpret_cast<const uint4 *>(kp + (int64_t)b * pool.r)[chunk_of(c)];
    };
    auto rows = [&](const T *pool_g, int b) __attribute__((always_inline)) { return reinterpret_cast<const uint4 *>(pool_g + (int64_t)b * pool.r); };

    // ---- the table: references, leaf sets, caller errors (tree_entries_kernel)
    for (int p = tid; p < P; p += NT) {
        refs[p] = 0;
        remap[p] = -1;
    }
    for (int s = tid; s < w.n_slots; s += NT) {
        cnt[s] = A.slot_init[s];
        nodes[s] = w.tiny_nodes[s];
    }
    if (tid < 8)
        counters[tid] = 0;
    if (tid == 0)
        n_tgt = 0;
    if (tid < w.r_stride) {
        col_assign[tid] = -1;
        col_cnt[tid] = 0;
    }
    __syncthreads();
    if (tid < n) {
        const int p = tab.bt[gn + tid], src = w.leaf_src[tid];
        bt[tid] = p;
        if (p < 0 || p >= P) {
            atomicAdd(&counters[4], 1);
        } else {
            const int before = atomicAdd(&refs[p], 1);
            if (before > 0)
                atomicAdd(&counters[5], before == 1 ? 2 : 1);
        }
        const int q = src >= 0 ? tab.bt[gn + src] : 0;
        ids[tid] = min(max(q, 0), P - 1);
    }

    // ---- norms of all stored blocks, a wavefront per block, the next one on its way
    uint4 ahead[CPL];
    auto fetch = [&](int b) __attribute__((always_inline)) {
        const uint4 *src = b >= P ? rows(vp, b - P) : rows(kp, b);
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            ahead[c] = src[chunk_of(c)];
    };
    if (wave < 2 * P)
        fetch(wave);
    for (int b = wave; b < 2 * P; b += NW) {
        const bool is_v = b >= P;
        const int p = is_v ? b - P : b;
        uint4 raw[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            raw[c] = ahead[c];
        if (b + NW < 2 * P)
            fetch(b + NW);
        double ss = 0.0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            if (STAGED && !is_v && in_block(c))
                keys[p * chunks + lane + 64 * c] = raw[c];
            double x[PER];
            Elem<T>::widen(raw[c], x);
            if (in_block(c))
#pragma unroll
                for (int i = 0; i < PER; ++i)
                    ss = fma(x[i], x[i], ss);
        }
        const double nrm = sqrt(wave_sum(ss));
        if (lane == 0) {
            (is_v ? nv : nk)[p] = nrm;
            (is_v ? pool.norm_v : pool.norm_k)[gp + p] = nrm;
            if (!is_v)
                pool.inv_norm_k[gp + p] = nrm > 0.0 ? (float)(1.0 / nrm) : 0.0f;
        }
    }
    __syncthreads();
    double orig_k = 0.0, orig_v = 0.0;
    if (tid < n) {
        const int p = bt[tid];
        const bool ok = p >= 0 && p < P;
        orig_k = ok ? nk[p] : 0.0;
        orig_v = ok ? nv[p] : 0.0;
        tab.orig_norm_k[gn + tid] = orig_k;
        tab.orig_norm_v[gn + tid] = orig_v;
        if (orig_k != 0.0 && !(orig_k >= 0x1p-40 && orig_k <= 0x1p40))
            atomicAdd(&counters[6], 1);
    }

    for (int hgt = 0; hgt < A.n_heights; ++hgt) {
        const int n0 = w.tiny_ptr[hgt], n1 = w.tiny_ptr[hgt + 1];
        // ---- similarity and assignment, a wavefront per right block
        for (int k = n0, j = wave; k < n1; ++k) {
            const int4 nd = nodes[2 * k];                   // left and right offset, left and right slot
            const int col0 = nodes[2 * k + 1].y;
            const int ml = cnt[nd.z], mr = cnt[nd.w];
            for (; j < mr; j += NW) {
                const int b = __builtin_amdgcn_readfirstlane(ids[nd.y + j]);
                const double nb = nk[b];
                uint4 braw[CPL];
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    braw[c] = key_chunk(b, c);
                double bv = -INFINITY, mine = -INFINITY;     // the largest cosine, its row; the cosine of row `lane`
                int bi = -1;
                for (int i0 = 0; i0 < ml; i0 += KW) {
                    int a[KW];
                    uint4 araw[KW][STAGED ? 1 : CPL];
#pragma unroll
                    for (int q = 0; q < KW; ++q) {
                        a[q] = __builtin_amdgcn_readfirstlane(ids[nd.x + min(i0 + q, ml - 1)]);
                        if constexpr (!STAGED)
#pragma unroll
                            for (int c = 0; c < CPL; ++c)
                                araw[q][c] = key_chunk(a[q], c);
                    }
                    double dot[KW];
#pragma unroll
                    for (int q = 0; q < KW; ++q)
                        dot[q] = 0.0;
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        if constexpr (STAGED)
#pragma unroll
                            for (int q = 0; q < KW; ++q)
                                araw[q][0] = key_chunk(a[q], c);
                        if (in_block(c)) {
                            double y[PER];
                            Elem<T>::widen(braw[c], y);
#pragma unroll
                            for (int q = 0; q < KW; ++q) {
                                double x[PER];
                                Elem<T>::widen(araw[q][STAGED ? 0 : c], x);
#pragma unroll
                                for (int i = 0; i < PER; ++i)
                                    dot[q] = fma(x[i], y[i], dot[q]);
                            }
                        }
                    }
                    double all = 0.0;                        // four rows: their sums share exchanges and a division
                    if constexpr (KW == 4) {
                        const int row = wave_sum4_of(lane);
                        const double na = nk[row == 0 ? a[0] : row == 1 ? a[1] : row == 2 ? a[KW - 2] : a[KW - 1]];
                        const double d = wave_sum4(dot[0], dot[1], dot[KW - 2], dot[KW - 1]);
                        all = na == 0.0 || nb == 0.0 ? 0.0 : d / (na * nb);
                    }
#pragma unroll
                    for (int q = 0; q < KW; ++q) {
                        double cs;
                        if constexpr (KW == 4) {
                            cs = read_lane(all, wave_sum4_lane(q));
                        } else {
                            const double na = nk[a[q]], d = wave_sum(dot[q]);
                            cs = na == 0.0 || nb == 0.0 ? 0.0 : d / (na * nb);
                        }
                        if (i0 + q < ml) {
                            mine = lane == i0 + q ? cs : mine;
                            if (cs > bv) {                   // ascending rows: the lowest of equal ones
                                bv = cs;
                                bi = i0 + q;
                            }
                        }
                    }
                }
                // what the screen in binary32 would have sent to the re-check: counted, as there
                const float val = (float)mine;
                const bool listed = lane < ml && val > A.thr_floor;
                float top = listed ? val : -INFINITY;
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1)
                    top = fmaxf(top, __shfl_xor(top, off, 64));
                const int n_listed = __popcll(__ballot(listed));
                const int contenders = __popcll(__ballot(listed && (double)val >= (double)top - 2.0 * A.band));
                if (hgt + 1 == A.n_heights)
                    col_val[col0 + j][lane] = listed ? val : -INFINITY;
                if (lane == 0) {
                    assign[nd.y + j] = col_assign[col0 + j] = bv > A.thr ? bi : -1;
                    col_cnt[col0 + j] = hgt + 1 == A.n_heights ? n_listed : 0;
                    if (n_listed > w.cand_cap || (n_listed > 0 && !(contenders == 1 && (double)top > A.thr + 2.0 * A.band))) {
                        atomicAdd(&counters[2], 1);
                        if (fabs(bv - A.thr) <= A.band)
                            atomicAdd(&counters[1], 1);
                        if (n_listed > w.cand_cap)
                            atomicAdd(&counters[3], 1);
                    }
                }
            }
            j -= mr;
        }
        __syncthreads();
        // ---- targets and their members, evicted blocks, surviving sets: a wavefront per node, a lane per block
        for (int k = n0 + wave; k < n1; k += NW) {
            const int4 nd = nodes[2 * k];
            const int out_slot = nodes[2 * k + 1].x;
            const int ml = cnt[nd.z], mr = cnt[nd.w];
            int id = -1, a = -1;
            if (lane < mr) {
                id = ids[nd.y + lane];
                a = assign[nd.y + lane];
                was[nd.y + lane] = id;
            }
            unsigned long long members = 0;
            for (int i = 0; i < ml; ++i) {
                const unsigned long long m = __ballot(a == i);
                members = lane == i ? m : members;
            }
            const unsigned long long targets = __ballot(members != 0), kept = __ballot(lane < mr && a < 0);
            const unsigned long long below = (1ull << lane) - 1ull;
            int base = 0;
            if (lane == 0 && targets)
                base = atomicAdd(&n_tgt, __popcll(targets));
            base = __builtin_amdgcn_readfirstlane(base);
            if (members) {
                const int s = base + __popcll(targets & below);
                tgt[s] = nd.x + lane;
                tgt_right[s] = nd.y;
                tgt_mask[s] = members;
            }
            if (a >= 0)
                remap[id] = ids[nd.x + a];
            __builtin_amdgcn_wave_barrier();
            if (lane < mr && a < 0)
                ids[nd.x + ml + __popcll(kept & below)] = id;
            if (lane == 0) {
                cnt[out_slot] = ml + __popcll(kept);
                atomicAdd(&counters[0], mr - __popcll(kept));
                atomicAdd(&counters[7], __popcll(targets));
            }
        }
        __syncthreads();
        // ---- merge, a wavefront per target and tensor
        const int items = 2 * n_tgt;
        for (int it = wave; it < items; it += NW) {
            const int t = it >> 1;
            const bool is_v = it & 1;
            T *const pool_g = is_v ? vp : kp;
            const double *norm = is_v ? nv : nk;
            const int a = __builtin_amdgcn_readfirstlane(ids[tgt[t]]);
            auto chunk = [&](int b, int c) __attribute__((always_inline)) {
                return STAGED && !is_v ? key_chunk(b, c) : rows(pool_g, b)[chunk_of(c)];
            };
            auto member = [&](unsigned long long m) __attribute__((always_inline)) {
                return __builtin_amdgcn_readfirstlane(was[tgt_right[t] + __builtin_ctzll(m)]);
            };
            double acc[CPL][PER];
            unsigned long long m = tgt_mask[t];      // (a target has a member)
            uint4 mraw[CPL];
            {
                uint4 araw[CPL];
                const int b = member(m);
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    araw[c] = chunk(a, c);
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    mraw[c] = chunk(b, c);
                const double na = norm[a], ia = na == 0.0 ? 0.0 : 1.0 / na;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    Elem<T>::widen(araw[c], acc[c]);
#pragma unroll
                    for (int e = 0; e < PER; ++e)
                        acc[c][e] = in_block(c) ? acc[c][e] * ia : 0.0;
                }
            }
            while (m) {
                const double nb = norm[member(m)], ib = nb == 0.0 ? 0.0 : 1.0 / nb;
                m &= m - 1;
                uint4 braw[CPL];
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    braw[c] = mraw[c];
                if (m)
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
                        mraw[c] = chunk(member(m), c);
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    double y[PER];
                    Elem<T>::widen(braw[c], y);
#pragma unroll
                    for (int e = 0; e < PER; ++e)
                        acc[c][e] = in_block(c) ? fma(y[e], ib, acc[c][e]) : 0.0;
                }
            }
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int c = 0; c < CPL; ++c)
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    double &s = PAIR && (c & 1) ? s1 : s0;
                    s = fma(acc[c][e], acc[c][e], s);
                }
            const double len = sqrt(PAIR ? wave_sum(s0) + wave_sum(s1) : wave_sum(s0));
            const double il = len == 0.0 ? 0.0 : 1.0 / len;
            uint4 *dst = reinterpret_cast<uint4 *>(pool_g + (int64_t)a * pool.r);
            s0 = s1 = 0.0;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                double u[PER], back[PER];
#pragma unroll
                for (int e = 0; e < PER; ++e)
                    u[e] = acc[c][e] * il;
                const uint4 packed = Store16<T>::pack(u, back);
                if (in_block(c)) {
                    dst[lane + 64 * c] = packed;
                    if (STAGED && !is_v)
                        keys[a * chunks + lane + 64 * c] = packed;
#pragma unroll
                    for (int e = 0; e < PER; ++e) {
                        double &s = PAIR && (c & 1) ? s1 : s0;
                        s = fma(back[e], back[e], s);
                    }
                }
            }
            const double nrm = sqrt(PAIR ? wave_sum(s0) + wave_sum(s1) : wave_sum(s0));
            if (lane == 0) {                  // (nobody else reads this block or its norm before the barrier)
                (is_v ? nv : nk)[a] = nrm;
                (is_v ? pool.norm_v : pool.norm_k)[gp + a] = nrm;
                if (!is_v)
                    pool.inv_norm_k[gp + a] = nrm > 0.0 ? (float)(1.0 / nrm) : 0.0f;
            }
        }
        __syncthreads();
        if (tid == 0)
            n_tgt = 0;
        // (the next height's first atomics on it are behind the barrier after its assignments)
    }

    // ---- rewrite
    const TinyArgs &again = kernel_args_again<TinyArgs>();
    const TableDesc &tab_end = again.tab;
    const WorkDesc &w_end = again.w;
    for (int p = tid; p < P; p += NT)
        refs[p] = 0;
    __syncthreads();
    int p = -1;
    if (tid < n) {
        p = bt[tid];
        if (p < 0 || p >= P) {
            p = -1;
        } else {
            for (int hop = 0; hop < 64; ++hop) {
                const int q = remap[p];
                if (q < 0 || q >= P || q == p)
                    break;
                p = q;
            }
            tab_end.bt[gn + tid] = p;
            atomicAdd(&refs[p], 1);
        }
    }
    __syncthreads();
    if (tid < n) {
        float sk = 0.0f, sv = 0.0f;
        if (p >= 0) {
            const double mk = nk[p], mv = nv[p];
            const bool own = refs[p] <= 1;
            sk = own ? 1.0f : mk == 0.0 ? 0.0f : (float)(orig_k / mk);
            sv = own ? 1.0f : mv == 0.0 ? 0.0f : (float)(orig_v / mv);
        }
        tab_end.scale_k[gn + tid] = sk;
        tab_end.scale_v[gn + tid] = sv;
    }
    for (int q = tid; q < P; q += NT) {
        tab_end.refcount[gp + q] = refs[q];
        tab_end.remap[gp + q] = remap[q];
    }
    for (int s = tid; s < w_end.n_slots; s += NT)
        w_end.set_cnt[(int64_t)g * w_end.n_slots + s] = cnt[s];
    // What the plan's view shows and single steps behind the call go by: sets, columns with the last height's candidates, and lists
    // that hold nothing to do.  (Stored here, where no barrier waits for it, by the last wavefronts first: the first one has the free
    // list to write.)
    const int back = NT - 1 - tid;
    if (back < n)
        w_end.set_ids[gn + back] = ids[back];
    if (back < w_end.r_stride) {
        const int64_t at = (int64_t)g * w_end.r_stride + back;
        w_end.assign[at] = col_assign[back];
        w_end.cand_cnt[at] = col_cnt[back];
        w_end.best_packed[at] = 0ull;
    }
    for (int c = NW - 1 - wave; c < w_end.r_stride; c += NW)
        if (col_cnt[c] > 0) {
            const float val = col_val[c][lane];
            const unsigned long long listed = __ballot(val > -INFINITY);
            const int slot = __popcll(listed & ((1ull << lane) - 1ull));
            if (val > -INFINITY && slot < w_end.cand_cap) {
                const int64_t at = ((int64_t)g * w_end.r_stride + c) * w_end.cand_cap + slot;
                w_end.cand_idx[at] = lane;
                w_end.cand_val[at] = val;
            }
        }
    if (g == 0 && back < again.n_heights)
        w_end.n_active[back] = w_end.n_refine[back] = w_end.n_pairs_all[back] = 0;
    if (tid < 8)
        w_end.counters[(int64_t)g * 8 + tid] = counters[tid];
    if (wave == 0) {
        int freed = 0, live = 0;
        for (int q0 = 0; q0 < P; q0 += 64) {
            const int q = q0 + lane;
            const bool is_free = q < P && remap[q] >= 0;
            const unsigned long long m = __ballot(is_free);
            if (is_free && again.free_list)
                again.free_list[gp + freed + __popcll(m & ((1ull << lane) - 1ull))] = q;
            freed += __popcll(m);
            live += __popcll(__ballot(q < P && refs[q] > 0));
        }
        if (lane == 0) {
            if (again.n_free)
                again.n_free[g] = freed;
            if (again.n_phys)
                again.n_phys[g] = live;
        }
    }
}

void launch_tiny_tree(hipStream_t s, const PoolDesc &pool, const TableDesc &tab, const WorkDesc &w, const int32_t *slot_init, int n_heights,
                      double thr, double band, float thr_floor, int32_t *free_list, int32_t *n_free, int32_t *n_phys)
{
    const TinyArgs A{pool, tab, w, slot_init, n_heights, thr, band, thr_floor, free_list, n_free, n_phys};
    const int cpl = (pool.r * (pool.dtype == KVFUSE_BF16 ? 2 : 4) / 16 + 63) / 64;
    const int64_t key_bytes = (int64_t)pool.P * pool.r * (pool.dtype == KVFUSE_BF16 ? 2 : 4);
    const bool staged = key_bytes <= kTinyStage && n_heights > 0;
#define KVF_TINY_CPL(T, CPL)                                                                                \
    do {                                                                                                    \
        if (staged) tiny_tree_kernel<T, CPL, true><<<pool.G, kTinyThreads<T, CPL>, (unsigned)key_bytes, s>>>(A); \
        else tiny_tree_kernel<T, CPL, false><<<pool.G, kTinyThreads<T, CPL>, 0, s>>>(A);                    \
    } while (0)
#define KVF_TINY(T)                            \
    do {                                       \
        if (cpl <= 1) KVF_TINY_CPL(T, 1);      \
        else if (cpl <= 2) KVF_TINY_CPL(T, 2); \
        else KVF_TINY_CPL(T, 4);               \
    } while (0)
    if (pool.dtype == KVFUSE_BF16)
        KVF_TINY(bf16_t);
    else
        KVF_TINY(float);
#undef KVF_TINY
#undef KVF_TINY_CPL
}

}  // namespace kvfuse
