// Work items of a height, laid out on the device from the sizes the sets have now, for the ring kernel (similarity.hip) and the panel
// kernel (panel.hip): where a height may be either's, both in the same two launches, since either may have nothing to do and a launch is 5 us.
#pragma once
#include "common.h"

namespace kvfuse {

__device__ __forceinline__ int items_of_node(int ml, int mr, int bm, int bn, int most, int &n_cp, int &rt, int &n_rc)
{
    n_cp = (mr + bn - 1) / bn;
    const int n_rtile = (ml + bm - 1) / bm;
    rt = min((n_rtile + 3) / 4, most);

    n_rc = rt > 0 ? (n_rtile + rt - 1) / rt : 0;
    return n_cp * n_rc;
}

// A binary32 number as three bfloat16 parts (upper halves of what is left): exact.
struct Parts {
    uint32_t h, m, l;      // in the upper halves
    __device__ __forceinline__ explicit Parts(float x)
    {
        h = __float_as_uint(x) & 0xFFFF0000u;
        x -= __uint_as_float(h);
        m = __float_as_uint(x) & 0xFFFF0000u;
        x -= __uint_as_float(m);
        l = __float_as_uint(x) & 0xFFFF0000u;
    }
};
__device__ __forceinline__ uint32_t pair16(uint32_t lo, uint32_t hi) { return (lo >> 16) | hi; }

// Fragments of the MFMA that starts a product.  The 16 summation indices hold, for each of the two terms, the six products of
// parts that reach 2^-24 of the term: h h, h m, m h, m m, h l, l h.
__device__ __forceinline__ u32x4 panel_left(float x, float y, int half)
{
    const Parts p(x), q(y);
    return half == 0 ? u32x4{pair16(p.h, p.h), pair16(p.m, p.m), pair16(p.h, p.l), pair16(q.h, q.h)}
                     : u32x4{pair16(q.m, q.m), pair16(q.h, q.l), 0u, 0u};
}
__device__ __forceinline__ u32x4 panel_right(float x, float y, int half)
{
    const Parts p(x), q(y);
    return half == 0 ? u32x4{pair16(p.h, p.m), pair16(p.h, p.m), pair16(p.l, p.h), pair16(q.h, q.m)}
                     : u32x4{pair16(q.h, q.m), pair16(q.l, q.h), 0u, 0u};
}

// The two factors of a block: its norm (1 for a zero block, whose products then stay below the floor), and its tail's length.  The
// left norm carries - floor, lowered by 4e-6 of itself: the roundings of the MFMAs (a few 2^-24 of floor |a| |b|) then only leave
// more pairs open, which finish_pairs_kernel tests whole.
__device__ __forceinline__ float panel_norm(const PoolDesc &pool, int64_t b)
{
    const float norm = (float)pool.norm_k[b];
    return norm == 0.0f ? 1.0f : norm;
}
__device__ __forceinline__ float panel_floor(float thr_floor) { return -thr_floor * (1.0f - 4e-6f); }

// The left blocks' operands, one thread per block of a left set: thread i of a launch over [groups][left blocks of the height].
__device__ __forceinline__ void panel_row(const PoolDesc &pool, const WorkDesc &w, const HeightDesc &h, float thr_floor, int64_t i)
{
    if (i >= (int64_t)w.G * h.total_l_cap)
        return;
    const int g = (int)(i / h.total_l_cap);
    const int c = (int)(i - (int64_t)g * h.total_l_cap);
    if (!w.panel_on[g])
        return;
    int lo = 0, hi = h.n_nodes;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (h.l_base[mid] <= c)
            lo = mid;
        else
            hi = mid;
    }
    const int row = c - h.l_base[lo];
    if (row >= w.set_cnt[(int64_t)g * w.n_slots + h.l_slot[lo]])
        return;
    const int64_t b = (int64_t)g * pool.P + w.set_ids[(int64_t)g * w.n + h.l_off[lo] + row];
    const float norm = panel_norm(pool, b);
    u32x4 *out = w.panel_rows + ((int64_t)g * w.l_stride + c) * 2;
    out[0] = panel_left(panel_floor(thr_floor) * norm, w.rem_k[b] * norm, 0);
    out[1] = panel_left(panel_floor(thr_floor) * norm, w.rem_k[b] * norm, 1);
}

// Rows of a node's items: whole stages, at most `run`, the same number for all but the last.
__device__ __forceinline__ int panel_rows_per_item(int ml, int run)
{
    const int stages = (ml + kPanelRows - 1) / kPanelRows;
    const int n = max((stages + run - 1) / run, 1);
    return max((stages + n - 1) / n, 1) * kPanelRows;
}

// A workgroup of 256 for group g: whether the panel kernel takes it at this height, and if so its work items, behind those of the groups
// that came first.  An item is (group, node, panel of 512 right blocks, run of left blocks); consecutive items of a node share
// the run, so that the workgroups an XCD holds at a time read the same left rows.  The panel kernel takes a group
//   - whose head fits its registers,
//   - whose tests left few pairs open at the height before (of `prev`, which has no nodes before the first height),
//   - and, where the ring kernel is faster on blocks that have little to do with each other (panel_from, host.hip), only if tiles were
//     multiplied whole at the height before, or there was none.  A whole tile takes the ring kernel some 50 us (4 KiB blocks), and a
//     height of few tiles ends with it: 13 requests of 492 blocks, a quarter of them common, 8 groups, a height 73 us against 60.
__device__ __forceinline__ bool panel_items_of_group(const WorkDesc &w, const HeightDesc &h, const HeightDesc &prev, int height, int g)
{
    __shared__ int64_t lds4[4];
    __shared__ int node0[256], node_cp[256], node_rows[256];
    __shared__ int first;
    const int tid = threadIdx.x;
    // pairs that the tests of the height before left open, against the pairs there were
    double pairs = 0.0;
    __shared__ double red[4];
    for (int k = tid; k < prev.n_nodes; k += 256)
        pairs += (double)w.set_cnt[(int64_t)g * w.n_slots + prev.l_slot[k]] * (double)w.set_cnt[(int64_t)g * w.n_slots + prev.r_slot[k]];
    pairs = block_sum_256(pairs, red);
    const bool on = w.early_nk[g] <= kPanelSlices && (!w.group_enable || w.group_enable[g]) &&
                    (double)w.open_cnt[g] * kPanelOpen <= pairs && (w.early_nk[g] >= h.panel_from || prev.n_nodes == 0 || w.whole[g]);
    auto items_of = [&](int k, int &n_cp, int &rows) {
        const int ml = w.set_cnt[(int64_t)g * w.n_slots + h.l_slot[k]], mr = w.set_cnt[(int64_t)g * w.n_slots + h.r_slot[k]];
        n_cp = (mr + kPanelCols - 1) / kPanelCols;
        rows = panel_rows_per_item(ml, h.panel_run);
        return n_cp * ((ml + rows - 1) / rows);
    };
    int64_t total = 0;
    if (on) {
        int64_t mine = 0;
        for (int k = tid; k < h.n_nodes; k += 256) {
            int n_cp, rows;
            mine += items_of(k, n_cp, rows);
        }
        (void)block_exscan<256>(mine, lds4, total);
    }
    __syncthreads();
    if (tid == 0) {
        first = total > 0 ? atomicAdd(&w.panel_total[height], (int)total) : 0;
        w.panel_on[g] = on;
    }
    __syncthreads();
    int run = first;
    for (int k0 = 0; on && k0 < h.n_nodes; k0 += 256) {
        int n_cp = 1, rows = 0;
        const int64_t c = k0 + tid < h.n_nodes ? items_of(k0 + tid, n_cp, rows) : 0;
        int64_t sum;
        const int64_t pre = block_exscan<256>(c, lds4, sum);
        node0[tid] = (int)pre;
        node_cp[tid] = n_cp;
        node_rows[tid] = rows;
        __syncthreads();
        for (int i = tid; i < (int)sum; i += 256) {
            int lo = 0, hi = 256;            // the last node whose first item is not behind i (empty ones share their successor's)
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (node0[mid] <= i)
                    lo = mid;
                else
                    hi = mid;
            }
            const int q = i - node0[lo];
            w.panel_items[run + i] = make_int4(g, k0 + lo, (q % node_cp[lo]) * kPanelCols, q / node_cp[lo] * node_rows[lo]);
        }
        run += (int)sum;
        __syncthreads();
    }
    return on;
}

}  // namespace kvfuse
