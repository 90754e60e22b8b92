// Head copies: the first elements of the key blocks in six bits each, for the panel kernel (panel.hip).
//
// With p elements of a block's head multiplied, cos(a, b) <= <a_head, b_head> / (|a| |b|) + tail(a) tail(b) (early.hip).  The head's
// share of the cosine is small (p is a fifth of a block), so its product need not be exact: with q the copy and d = head - q,
//     <a_head, b_head> = <q_a, q_b> + <d_a, q_b + d_b / 2> + <q_a + d_a / 2, d_b> <= <q_a, q_b> + E_a H_b + H_a E_b,
// E = |d|, measured when the copy is made, H = |head| + 3 E / 2.  A pair whose bound stays below the candidate floor is ruled out as
// surely as by the exact head; the others are tested whole (finish_pairs_kernel), so that candidates are the same.  Elements
// are e2m3 (six bits, three of mantissa, on blocks scaled by a power of two to 1.25 .. 2.5 root mean square): E is 3 % of the head for
// white-noise-like keys, which costs a head of 11 slices half a slice, and the matrix units multiply e2m3 at four times the rate of
// bfloat16 (measured from registers on random data: 5.8 against 1.67 PFLOP/s).
//
// A copy of up to six steps of 64 elements has 320 bytes, one of up to twelve 640 (HeadShape): 18 or 36 pieces of 16 bytes of codes,
// piece 2 m + h the m-th of what half h of a wavefront multiplies, 48 bytes for every two steps, in the order of an MFMA operand; then the
// operands of the test (items.h) for the block on the left and on the right, eight bytes for either half.
//
// Copies of a group's blocks are made at the first height that the panel kernel takes the group at, of the blocks that are still there; a
// copy's place (slot) is its block's position in the set lists then, and set_slot follows the block when the lists are compacted.  Blocks that
// a merge has rewritten get their copy anew.
#pragma once
#include "items.h"

namespace kvfuse {

typedef __bf16 bf16x32 __attribute__((ext_vector_type(32)));

// 16 or 32 lanes per block: lane `sub` holds the elements 32 sub ... (`raw`), four of those left over write the operands of the test.
// `dst` null: nothing (all lanes stay, for the exchanges).
template <bool LONG>
__device__ __forceinline__ void head_copy(const u32x4 (&raw)[4], double norm, int steps, char *__restrict__ dst, float thr_floor, int sub)
{
    constexpr int UNITS = 2 * HeadShape<LONG>::steps, LANES = LONG ? 32 : 16;
    const bool codes = dst && sub < 2 * steps;
    float x[32], head = 0.0f;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const uint32_t word = raw[e >> 3][(e >> 1) & 3];
        x[e] = __uint_as_float(e & 1 ? word & 0xFFFF0000u : word << 16);
        head = fmaf(x[e], x[e], head);
    }
    if (!codes)
        head = 0.0f;
#pragma unroll
    for (int off = LANES / 2; off >= 1; off >>= 1)
        head += __shfl_xor(head, off, 64);
    // The scale 2^k brings the head's root mean square to 1.25 .. 2.5.  A head far below the norm is scaled less (its copy is then
    // coarse or zero, which E says), so that |block| 2^k stays within 2^21 and the operands of the test within binary32.
    int k = 0;
    if (norm > 0.0) {
        const int most = 20 - ((int)(__float_as_uint((float)norm) >> 23) - 127);
        k = most;
        if (head > 0.0f)
            k = (int)(__float_as_uint(2.5f * rsqrtf(head / (64.0f * (float)max(steps, 1)))) >> 23 & 255) - 127;
        k = max(min(k, min(most, 100)), -100);
    }
    const float up = __uint_as_float((uint32_t)(127 + k) << 23), down = __uint_as_float((uint32_t)(127 - k) << 23);
    bf16x32 elements;
    __builtin_memcpy(&elements, raw, sizeof elements);
    const auto q = __builtin_amdgcn_cvt_scalef32_pk32_fp6_bf16(elements, down);          // (divides by its scale)
    const auto back = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(q, down);
    float miss = 0.0f;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const float d = x[e] - back[e];
        miss = fmaf(d, d, miss);
    }
    if (!codes)
        miss = 0.0f;
#pragma unroll
    for (int off = LANES / 2; off >= 1; off >>= 1)
        miss += __shfl_xor(miss, off, 64);
    if (!dst)
        return;
    if (sub < UNITS) {
        // unit u of step u / 2, half u % 2: the first or second 24 of that half's 48 bytes
        char *at = dst + (sub >> 2) * 96 + (sub & 1) * 16;
        if (!(sub & 2)) {
            *reinterpret_cast<u32x4 *>(at) = u32x4{q[0], q[1], q[2], q[3]};
            *reinterpret_cast<u32x2 *>(at + 32) = u32x2{q[4], q[5]};
        } else {
            *reinterpret_cast<u32x2 *>(at + 40) = u32x2{q[0], q[1]};
            *reinterpret_cast<u32x4 *>(at + 64) = u32x4{q[2], q[3], q[4], q[5]};
        }
        return;
    }
    if (sub >= UNITS + 4)
        return;
    // The test's numbers in units of the copy, the roundings (sums of fewer than 2^9 binary32 terms, each within 2^-23 of itself; roots,
    // conversions) upwards; |q| is at most |head| + E.
    const float err = sqrtf(miss * (1.0f + 0x1p-13f)) * (1.0f + 0x1p-20f);
    const float both = sqrtf(head * (1.0f + 0x1p-13f)) * (1.0f + 0x1p-20f) + 1.5f * err;
    const double rest = fma(norm, norm * (1.0 + 0x1p-44), -(double)head * (1.0 - 0x1p-13));
    const float tail = (float)sqrt(rest > 0.0 ? rest : 0.0) * (1.0f + 0x1p-20f);
    const float whole = norm == 0.0 ? 1.0f : (float)norm * up;             // (a zero block: every product below the floor)
    const float t = tail * up, e = err * up, f = both * up;
    *reinterpret_cast<u32x2 *>(dst + UNITS * 24 + (sub - UNITS) * 8) =
        sub < UNITS + 2 ? panel_left(panel_floor(thr_floor) * whole, t, e, f, sub & 1) : panel_right(whole, t, e, f, sub & 1);
}

template <bool LONG>
__device__ __forceinline__ void head_copy_of(const PoolDesc &pool, const WorkDesc &w, bool live, int g, int id, int slot, float thr_floor, int sub)
{
    if (!__any(live))
        return;
    const int64_t b = live ? (int64_t)g * pool.P + id : 0;
    const u32x4 *src = reinterpret_cast<const u32x4 *>((const char *)pool.k + b * pool.r * 2 + (sub < 2 * HeadShape<LONG>::steps ? sub : 0) * 64);
    const u32x4 raw[4] = {src[0], src[1], src[2], src[3]};
    head_copy<LONG>(raw, pool.norm_k[b], live ? w.head_steps[g] : 0, live ? w.heads + ((int64_t)g * w.n + slot) * HeadShape<LONG>::bytes : nullptr, thr_floor, sub);
}

// Workgroup `wg` of `n_wg` of 256 threads: the targets that the merge step of a height has rewritten (the work list of the assignment step), of
// groups that had copies by then.
template <bool LONG>
__device__ __forceinline__ void heads_of_targets(const PoolDesc &pool, const WorkDesc &w, int height, float thr_floor, int wg, int n_wg)
{
    constexpr int LANES = LONG ? 32 : 16, PER = 256 / LANES;
    const int n = w.n_active[height], sub = threadIdx.x % LANES;
    for (int t0 = wg * PER; t0 < n; t0 += n_wg * PER) {
        const int64_t t = min(t0 + (int)threadIdx.x / LANES, n - 1);
        const int4 rec = w.active[2 * t];
        const int made = w.head_made[rec.x];
        head_copy_of<LONG>(pool, w, t0 + (int)threadIdx.x / LANES < n && made > 0 && made <= height + 1, rec.x, rec.y, w.active[2 * t + 1].z, thr_floor, sub);
    }
}

// Likewise, before the products of a height: all blocks that are still there, of the groups that have no copies yet, and the targets of the
// height before of those that have.
// What bounds it: memory, 768 bytes read and 320 written per block (1.7 million blocks of 4 KiB: 0.5 ms, 3.7 TB/s), or twice that.  One position a
// wavefront and trip, behind the five loads that find its block, took 0.8 ms.
template <bool LONG>
__device__ __forceinline__ void heads_of_height(const PoolDesc &pool, const WorkDesc &w, int height, float thr_floor, int wg, int n_wg)
{
    constexpr int LANES = LONG ? 32 : 16, PER = 256 / LANES;
    __shared__ int32_t block_of[256];            // the block of a position, or -1
    const int tid = threadIdx.x, sub = tid % LANES, per_group = (w.n + 255) / 256;
    const int64_t n = (int64_t)w.n_new[height] * per_group;
    for (int64_t v = wg; v < n; v += n_wg) {
        const int g = w.new_groups[v / per_group], at0 = (int)(v % per_group) * 256, at = at0 + tid;
        {
            int s = at < w.n ? w.pos_leaf[at] : -1, up = -1;
            if (s >= 0)              // the set that the position belongs to now
                while ((up = w.node_parent[s]) >= 0 && w.node_height[up] <= height)
                    s = up;
            const bool live = up >= 0 && at - w.node_off[s] < w.set_cnt[(int64_t)g * w.n_slots + s];
            block_of[tid] = live ? w.set_ids[(int64_t)g * w.n + at] : -1;
            if (live)
                w.set_slot[(int64_t)g * w.n + at] = at;
        }
        __syncthreads();
        for (int k = tid / LANES; k < 256; k += PER)
            head_copy_of<LONG>(pool, w, block_of[k] >= 0, g, block_of[k], at0 + k, thr_floor, sub);
        __syncthreads();
    }
    if (height > 0)
        heads_of_targets<LONG>(pool, w, height - 1, thr_floor, wg, n_wg);
}

}  // namespace kvfuse
