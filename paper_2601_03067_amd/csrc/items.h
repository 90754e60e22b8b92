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

// The first two bfloat16 parts of a binary32 number (upper halves of what is left): both of its sign, less than 2^-14 of it is missing.
struct Parts {
    uint32_t h, m;         // in the upper halves
    __device__ __forceinline__ explicit Parts(float x)
    {
        h = __float_as_uint(x) & 0xFFFF0000u;
        m = __float_as_uint(x - __uint_as_float(h)) & 0xFFFF0000u;
    }
};
__device__ __forceinline__ uint32_t pair16(uint32_t lo, uint32_t hi) { return (lo >> 16) | hi; }

// A bfloat16 number not below x >= 0, in the upper half.
__device__ __forceinline__ uint32_t up16(float x) { return (__float_as_uint(x) + 0xFFFFu) & 0xFFFF0000u; }

// Operands of the MFMA that starts a product of heads: the test of a pair (heads.hip),
//     <q_a, q_b> > floor |a| |b| - tail_a tail_b - E_a H_b - H_a E_b,
// is of rank four in (a, b), and its right side is what the product starts from.  The eight summation indices hold h h, h m, m h of
// either of the first two terms and the last two rounded up to bfloat16 (they are a hundredth of the first, 2^-7 of which is the rounding).
// What the three products of parts miss is not negative and at most 3 / 2^14 of the term: the first term's share of it
// leaves more pairs open, and the tails are lengthened by 2^-13 for the second's.  x: the norm, y: the tail.
__device__ __forceinline__ u32x2 panel_left(float x, float y, float e, float h, int half)
{
    const Parts p(x), q(y * (1.0f + 0x1p-13f));
    return half == 0 ? u32x2{pair16(p.h, p.h), pair16(p.m, q.h)} : u32x2{pair16(q.h, q.m), pair16(up16(e), up16(h))};
}
__device__ __forceinline__ u32x2 panel_right(float x, float y, float e, float h, int half)
{
    const Parts p(x), q(y * (1.0f + 0x1p-13f));
    return half == 0 ? u32x2{pair16(p.h, p.m), pair16(p.h, q.h)} : u32x2{pair16(q.m, q.h), pair16(up16(h), up16(e))};
}

// The left norm carries - floor, lowered by 8e-6 of itself: the roundings of the MFMAs (a few 2^-24 of floor |a| |b|) and of the norms
// then only leave more pairs open, which finish_pairs_kernel tests whole.
__device__ __forceinline__ float panel_floor(float thr_floor) { return -thr_floor * (1.0f - 8e-6f); }

// Rows of a node's items: whole stages of `rows`, at most `run`, the same number for all but the last.
__device__ __forceinline__ int panel_rows_per_item(int ml, int rows, int run)
{
    const int stages = (ml + rows - 1) / rows;
    const int n = max((stages + run - 1) / run, 1);
    return max((stages + n - 1) / n, 1) * rows;
}

// A workgroup of 256 for group g: whether the panel kernel takes it at this height, and if so its work items, behind those of the groups
// that came first.  An item is (group, node, panel of right blocks, run of left blocks); consecutive items of a node share
// the run, so that the workgroups an XCD holds at a time read the same left rows.  The panel kernel takes a group
//   - whose head fits its registers (head_steps),
//   - whose blocks repeat little: few pairs left open by the tests of the height before (`prev`, which has no nodes before the first height)
//     and hardly any in tiles that the ring kernel multiplied whole there, or at the first height no related pair in the sample
//     (early.hip).  Of a whole tile, 50 us on one compute unit of 256, every related pair goes to finish_pairs_kernel instead, 1.6 ns
//     each for blocks of 4 KiB, and a tile without any takes 30 ns (of the chip) less here than there (128 requests of 256 popular blocks
//     at 0.8, 16 groups, first height: 2600 us in this kernel, 740 in that one);
//   - that has its head copies, or pairs enough ahead for making them (kHeadPairs);
//   - and, where the ring kernel is faster on blocks that have little to do with each other (panel_few, host.hip), only if tiles were
//     multiplied whole at the height before, or there was none.  A whole tile takes the ring kernel some 50 us (4 KiB blocks), and a
//     height of few tiles ends with it: 13 requests of 492 blocks, a quarter of them common, 8 groups, a height 73 us against 60.
__device__ __forceinline__ bool panel_items_of_group(const WorkDesc &w, const HeightDesc &h, const HeightDesc &prev, int height, int g)
{
    __shared__ int64_t lds4[4];
    __shared__ int node0[256], node_cp[256], node_rows[256];
    __shared__ int first;
    const int tid = threadIdx.x, cols = panel_cols(w.long_heads), stage = panel_rows(w.long_heads), run_most = h.panel_run[w.long_heads];
    // (nothing is summed up for a group whose heads are too long, or whose blocks repeat too much whatever the sum)
    if (w.head_steps[g] == 0 || (prev.n_nodes > 0 && (double)w.dense_cnt[g] * kPanelDense > (double)prev.total_s)) {
        if (tid == 0)
            w.panel_on[g] = 0;
        return false;
    }
    // pairs that the tests of the height before left open, against the pairs there were
    double pairs = 0.0;
    __shared__ double red[4];
    for (int k = tid; k < prev.n_nodes; k += 256)
        pairs += (double)w.set_cnt[(int64_t)g * w.n_slots + prev.l_slot[k]] * (double)w.set_cnt[(int64_t)g * w.n_slots + prev.r_slot[k]];
    pairs = block_sum_256(pairs, red);
    bool on = (!w.group_enable || w.group_enable[g]) &&
                    (prev.n_nodes == 0 ? w.whole[g] == 0
                                       : (double)w.open_cnt[g] * kPanelOpen <= pairs && (double)w.dense_cnt[g] * kPanelDense <= pairs) &&
                    (!h.panel_few || prev.n_nodes == 0 || w.whole[g]);
    auto items_of = [&](int k, int &n_cp, int &rows) {
        const int ml = w.set_cnt[(int64_t)g * w.n_slots + h.l_slot[k]], mr = w.set_cnt[(int64_t)g * w.n_slots + h.r_slot[k]];
        n_cp = (mr + cols - 1) / cols;
        rows = panel_rows_per_item(ml, stage, run_most);
        return n_cp * ((ml + rows - 1) / rows);
    };
    int64_t total = 0;
    if (on) {
        int64_t mine = 0;
        double now = 0.0, blocks = 0.0;
        for (int k = tid; k < h.n_nodes; k += 256) {
            int n_cp, rows;
            mine += items_of(k, n_cp, rows);
            const double ml = w.set_cnt[(int64_t)g * w.n_slots + h.l_slot[k]], mr = w.set_cnt[(int64_t)g * w.n_slots + h.r_slot[k]];
            now += ml * mr;
            blocks += ml + mr;
        }
        (void)block_exscan<256>(mine, lds4, total);
        if (w.head_made[g] == 0) {
            __syncthreads();
            now = block_sum_256(now, red);
            __syncthreads();
            blocks = block_sum_256(blocks, red);
            if (now * h.panel_left < (1 + w.long_heads) * kHeadPairs * blocks)
                on = false;
        }
    }
    if (!on)
        total = 0;
    __syncthreads();
    if (tid == 0) {
        first = total > 0 ? atomicAdd(&w.panel_total[height], (int)total) : 0;
        w.panel_on[g] = on;
        if (total > 0 && w.head_made[g] == 0) {
            w.head_made[g] = height + 1;
            w.new_groups[atomicAdd(&w.n_new[height], 1)] = g;
        }
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
            const int k = k0 + lo, col = (q % node_cp[lo]) * cols, row = q / node_cp[lo] * node_rows[lo];
            const int ml = w.set_cnt[(int64_t)g * w.n_slots + h.l_slot[k]], mr = w.set_cnt[(int64_t)g * w.n_slots + h.r_slot[k]];
            int4 *out = w.panel_items + 2 * (int64_t)(run + i);
            out[0] = make_int4(g, h.l_off[k] + row, h.r_off[k] + col, min(ml - row, node_rows[lo]) << 16 | min(mr - col, cols));
            out[1] = make_int4(h.r_base[k] + col, row, w.head_steps[g], 0);
        }
        run += (int)sum;
        __syncthreads();
    }
    return on;
}

}  // namespace kvfuse
