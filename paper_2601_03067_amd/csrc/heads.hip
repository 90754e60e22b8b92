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
// A copy has kHeadBytes = 320 bytes: 18 pieces of 16 bytes of codes, piece 2 m + h the m-th of what half h of a wavefront multiplies,
// 48 bytes for every two steps of 64 elements, in the order of an MFMA operand; then the operands of the test (items.h) for the block on
// the left and on the right, eight bytes for either half.  A copy's place (slot) is its block's first position in the
// set lists; set_slot follows the block when the lists are compacted.  Blocks that a merge has rewritten get their copy anew.
#include <algorithm>

#include "items.h"

namespace kvfuse {

typedef __bf16 bf16x32 __attribute__((ext_vector_type(32)));

// What bounds it: memory, 768 bytes read and 320 written per block (2.1 million blocks of 4 KiB: 0.55 ms, 4.1 TB/s).  16 lanes per block:
// 12 take 32 elements each, then the last four the operands of the test.  `b` < 0: nothing (all lanes stay, for the exchanges).
__device__ __forceinline__ void head_copy(const PoolDesc &pool, int64_t b, int steps, char *__restrict__ dst, float thr_floor, int sub)
{
    if (!__any(b >= 0))
        return;
    u32x4 raw[4];
    const bool codes = b >= 0 && sub < 2 * steps;             // unit `sub`: elements 32 sub ...
    const u32x4 *src = reinterpret_cast<const u32x4 *>((const char *)pool.k + max(b, (int64_t)0) * pool.r * 2 + (sub < 12 ? sub : 0) * 64);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        raw[i] = src[i];
    const double norm = pool.norm_k[max(b, (int64_t)0)];
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
    for (int off = 8; off >= 1; off >>= 1)
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
    for (int off = 8; off >= 1; off >>= 1)
        miss += __shfl_xor(miss, off, 64);
    if (b < 0)
        return;
    if (sub < 12) {
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
    // The test's numbers in units of the copy, the roundings (sums of fewer than 2^9 binary32 terms, each within 2^-23 of itself; roots,
    // conversions) upwards; |q| is at most |head| + E.
    const float err = sqrtf(miss * (1.0f + 0x1p-13f)) * (1.0f + 0x1p-20f);
    const float both = sqrtf(head * (1.0f + 0x1p-13f)) * (1.0f + 0x1p-20f) + 1.5f * err;
    const double rest = fma(norm, norm * (1.0 + 0x1p-44), -(double)head * (1.0 - 0x1p-13));
    const float tail = (float)sqrt(rest > 0.0 ? rest : 0.0) * (1.0f + 0x1p-20f);
    const float whole = norm == 0.0 ? 1.0f : (float)norm * up;             // (a zero block: every product below the floor)
    const float t = tail * up, e = err * up, f = both * up;
    *reinterpret_cast<u32x2 *>(dst + 288 + (sub - 12) * 8) =
        sub < 14 ? panel_left(panel_floor(thr_floor) * whole, t, e, f, sub & 1) : panel_right(whole, t, e, f, sub & 1);
}

__global__ __launch_bounds__(256) void heads_kernel(PoolDesc pool, WorkDesc w, float thr_floor)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;           // position in the leaf sets
    const int sub = threadIdx.x & 15;
    const int g = (int)(i / w.n), at = (int)(i - (int64_t)g * w.n);
    const bool live = i < (int64_t)w.G * w.n && w.leaf_src[at] >= 0 && w.head_steps[g] > 0;
    if (live && sub == 0)
        w.set_slot[i] = at;
    head_copy(pool, live ? (int64_t)g * pool.P + w.set_ids[i] : -1, live ? w.head_steps[g] : 0, w.heads + i * kHeadBytes, thr_floor, sub);
}

// The targets that the merge step of this height has rewritten (the work list of the assignment step).
__global__ __launch_bounds__(256) void heads_of_targets_kernel(PoolDesc pool, WorkDesc w, int height, float thr_floor)
{
    const int n = w.n_active[height], sub = threadIdx.x & 15;
    for (int t0 = blockIdx.x * 16; t0 < n; t0 += gridDim.x * 16) {
        const int t = t0 + (threadIdx.x >> 4);
        const int4 rec = w.active[2 * (int64_t)min(t, n - 1)];
        const int slot = w.active[2 * (int64_t)min(t, n - 1) + 1].z;
        const int steps = w.head_steps[rec.x];
        const bool live = t < n && steps > 0;
        head_copy(pool, live ? (int64_t)rec.x * pool.P + rec.y : -1, steps, w.heads + ((int64_t)rec.x * w.n + slot) * kHeadBytes, thr_floor, sub);
    }
}

void launch_heads(hipStream_t s, const PoolDesc &pool, const WorkDesc &w, float thr_floor)
{
    const int64_t total = ((int64_t)w.G * w.n + 15) / 16;
    if (total > 0)
        heads_kernel<<<(unsigned)total, 256, 0, s>>>(pool, w, thr_floor);
}

void launch_heads_of_targets(hipStream_t s, const PoolDesc &pool, const WorkDesc &w, int height, float thr_floor)
{
    const unsigned grid = (unsigned)std::min<int64_t>(((int64_t)w.G * w.l_stride + 15) / 16, 256 * 8);
    if (grid > 0)
        heads_of_targets_kernel<<<grid, 256, 0, s>>>(pool, w, height, thr_floor);
}

}  // namespace kvfuse
