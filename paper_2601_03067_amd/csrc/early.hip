// Early rejection in the full-length similarity screen of a tree call (Algorithm 1: sim <- k_l k_r^T; only the entries
// above the threshold matter).
//
// After the product has run over the first p elements of two key blocks, cos(a, b) <= <a[0:p], b[0:p]> / (|a| |b|) +
// tail(a) tail(b) with tail(x) = |x[p:]| / |x| (Cauchy-Schwarz).  The similarity kernel tests every tile of the product
// once, after the p of its group: a tile in which no pair's bound reaches the candidate floor is done there; the few pairs
// of a tile that do reach it are written to a list, from which finish_pairs_kernel completes their products one by one;
// and a tile with too many of them simply goes on to its full length.  Either way a candidate list receives exactly the
// pairs whose whole screened cosine clears the floor, so nothing downstream knows the difference, whatever the data; what
// depends on the data is how much of the product is spared.
//
// p is chosen per group and per call from a sample of the group's own blocks (sample_bounds_kernel): unrelated blocks of
// white-noise-like keys at thr 0.9 are ruled out after a sixth of their length, keys that share a direction need more, and
// where even three quarters of a block would not do, the group's product runs at full length (its tests cost nothing then).
#include <algorithm>

#include "common.h"

namespace kvfuse {

constexpr int kSamples = 64;      // sampled pairs per group: one per lane of a wavefront; twice as many where there is room for their bounds
constexpr int kSteps = 32;        // lengths considered: (k / 32) of the block's slices
static_assert(kSteps * kSamples * sizeof(float) <= 256 * 2 * sizeof(int4), "the bounds of a group fit its share of the merge work list");

// Fixed pseudo-random logical entries: the sample depends on the sizes alone.  The mixing steps and constants are those of
// "lowbias32", the published result of Chris Wellons' search for 32-bit integer hashes of low bias (hash-prospector).
__device__ __forceinline__ uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    return x ^ (x >> 16);
}

// One wavefront per (group, sampled pair): the pair's bound after every length considered, in binary32 (the result only
// steers how much work the product does).  Reads half a megabyte per group of 4 KiB blocks, twice that where there is room for 128
// pairs: HBM-bound for many groups (268 MB for 256 of them, 73 us; 64 pairs 33 us) and a few microseconds for few.  (One workgroup per group, the first form of this, took 95 us for
// 256 groups and 174 us for 16 groups of 8 KiB blocks.)
template <typename T>
__global__ __launch_bounds__(256) void sample_bounds_kernel(const T *__restrict__ kpool, const int32_t *__restrict__ bt, int G, int P, int n,
                                                            int r, int n_samples, float *__restrict__ bounds)
{
    constexpr int PER = Elem<T>::PER16, BATCH = 4;
    __shared__ float seg[4][3][kSteps];               // <a, b>, <a, a>, <b, b> of every segment
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int id = blockIdx.x * 4 + wave, g = id / n_samples, s = id % n_samples;      // (the grid is exactly G * n_samples / 4)
    const int chunks = r / PER, nk = chunks / 4;
    const int per_seg = chunks / kSteps;
    const int lanes_per_seg = chunks % (64 * kSteps) == 0 || (chunks % kSteps == 0 && (per_seg & (per_seg - 1)) == 0) ? min(per_seg, 64) : 1;
    for (int i = lane; i < 3 * kSteps; i += 64)
        (&seg[wave][0][0])[i] = 0.0f;
    __builtin_amdgcn_wave_barrier();
    const int x = (int)(((uint64_t)mix32(2u * s + 1u) * (uint32_t)n) >> 32);
    const int y = (int)(((uint64_t)mix32(2u * s + 2u) * (uint32_t)(n - 1)) >> 32);
    const int pa = min(max(bt[(int64_t)g * n + x], 0), P - 1);
    const int pb = min(max(bt[(int64_t)g * n + (x + 1 + y) % n], 0), P - 1);
    const uint4 *a = reinterpret_cast<const uint4 *>(kpool + ((int64_t)g * P + pa) * r);
    const uint4 *b = reinterpret_cast<const uint4 *>(kpool + ((int64_t)g * P + pb) * r);
    for (int c0 = lane; c0 < chunks; c0 += 64 * BATCH) {
        uint4 ra[BATCH], rb[BATCH];
#pragma unroll
        for (int q = 0; q < BATCH; ++q) {
            const int c = min(c0 + 64 * q, chunks - 1);
            ra[q] = a[c];
            rb[q] = b[c];
        }
#pragma unroll
        for (int q = 0; q < BATCH; ++q) {
            const int c = c0 + 64 * q;
            float u[PER], v[PER], ab = 0.0f, aa = 0.0f, bb = 0.0f;
            widen_f32<T>(ra[q], u);
            widen_f32<T>(rb[q], v);
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                ab = fmaf(u[e], v[e], ab);
                aa = fmaf(u[e], u[e], aa);
                bb = fmaf(v[e], v[e], bb);
            }
            // where a segment is a power of two of neighbouring lanes (the usual block sizes) these are summed first: eight
            // lanes adding to one LDS word took twice as long as everything else here
            for (int off = 1; off < lanes_per_seg; off <<= 1) {
                ab += __shfl_xor(ab, off, 64);
                aa += __shfl_xor(aa, off, 64);
                bb += __shfl_xor(bb, off, 64);
            }
            if (c < chunks && (lane & (lanes_per_seg - 1)) == 0) {
                const int k = (kSteps * ((c >> 2) + 1) - 1) / nk;       // segment k: slices [k nk / 32, (k + 1) nk / 32)
                atomicAdd(&seg[wave][0][k], ab);
                atomicAdd(&seg[wave][1][k], aa);
                atomicAdd(&seg[wave][2][k], bb);
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    const int len = lane & (kSteps - 1);              // lane = length of `len` segments
    float head = 0.0f, ha = 0.0f, hb = 0.0f, A = 0.0f, B = 0.0f;
#pragma unroll 4
    for (int k = 0; k < kSteps; ++k) {
        const float sa = seg[wave][1][k], sb = seg[wave][2][k];
        head += k < len ? seg[wave][0][k] : 0.0f;
        ha += k < len ? 0.0f : sa;                    // (tails)
        hb += k < len ? 0.0f : sb;
        A += sa;
        B += sb;
    }
    float bound = (head + sqrtf(ha * hb)) / sqrtf(A * B);
    if (A == 0.0f || B == 0.0f)
        bound = 0.0f;                                 // a zero block has cosine 0 with everything
    if (!(bound < 1e30f))
        bound = 1e30f;                                // blocks beyond binary32's range: no early test
    if (lane < kSteps)
        bounds[((int64_t)g * kSteps + len) * n_samples + s] = bound;
}

// Numbers that are in the order of the floats.
__device__ __forceinline__ uint32_t ordered_bits(float x)
{
    const uint32_t b = __float_as_uint(x);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

// One workgroup per group: for every length, of the bounds of all pairs, with their median m and the 16th and 84th
// percentiles, m + 4 s estimates what one unrelated pair in 30 000 reaches, about two of a 256 x 256 tile.  The
// shortest length for which that stays below the candidate floor is taken.  Ranks instead of moments because a few per cent
// of the pairs may be related ones; s is half the distance of the two percentiles (which varies less from sample to sample than
// either's distance from the median), but not much less than the upper one's, where the bounds are skewed.
// PER: sampled pairs per lane.  One pair and the upper percentile alone: 10, 12 or 14 slices of 64 for groups of one kind, 55 of 256
// of them 12 or more.
//
// The three order statistics of a length are found bit by bit, by counting what lies below: every pair's rank against every other
// took 30 us at two pairs a lane (11 at one), these counts take 15 over all 32 bits and 12 over 20.
//
// head_steps (or null): likewise the steps of 64 elements of the head copies (heads.hip), `wide` slices each, whose test is wider by what the copies
// miss, some 6.5 % of their share of a block; 0 where `steps_most` of them would not do, or for a group that is switched off.
template <int PER>
__global__ __launch_bounds__(1024) void choose_early_kernel(const float *__restrict__ bounds, int nk, float thr_floor,
                                                            int32_t *__restrict__ early_nk, int32_t *__restrict__ head_steps, int steps_most, int wide,
                                                            const uint8_t *__restrict__ group_enable, int32_t *__restrict__ related)
{
    constexpr int N = PER * kSamples;
    __shared__ float reach[kSteps];
    __shared__ int best, best_steps;
    const int g = blockIdx.x, lane = threadIdx.x & 63;
    for (int len = threadIdx.x >> 6; len < kSteps; len += 16) {
        uint32_t bound[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i)
            bound[i] = ordered_bits(bounds[((int64_t)g * kSteps + len) * N + i * 64 + lane]);
        constexpr int rank[3] = {N * 16 / 100, N / 2, N * 84 / 100 + 1};
        uint32_t at[3] = {0u, 0u, 0u};           // the largest number that at most so many bounds lie below: the one of that rank
#pragma unroll 4
        for (uint32_t bit = 0x80000000u; bit >= 0x1000u; bit >>= 1)          // (20 bits are 2^-11 of a bound, below the margin of the choice)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                int below = 0;
#pragma unroll
                for (int i = 0; i < PER; ++i)
                    below += __popcll(__ballot(bound[i] < (at[k] | bit)));
                if (below <= rank[k])
                    at[k] |= bit;
            }
        float value[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            value[k] = __uint_as_float(at[k] ^ ((at[k] >> 31) ? 0x80000000u : 0xFFFFFFFFu));
        if (len == kSteps - 1) {             // (sampled pairs that are near copies: all but a 32nd of their products is in)
            int n = 0;
#pragma unroll
            for (int i = 0; i < PER; ++i)
                n += __popcll(__ballot(bound[i] >= ordered_bits(thr_floor)));
            if (lane == 0)
                related[g] = n;
        }
        if (lane == 0)
            reach[len] = value[1] + 4.0f * fmaxf(0.5f * (value[2] - value[0]), 0.85f * (value[2] - value[1]));
    }
    if (threadIdx.x == 0) {
        best = nk;
        best_steps = steps_most + 1;
    }
    __syncthreads();
    // between two lengths the reach is taken as a straight line
    auto reach_at = [&](int slices) {
        const int len = slices * kSteps / nk, rest = slices * kSteps % nk;
        const float r0 = reach[len], r1 = reach[min(len + 1, kSteps - 1)];
        return r0 + (r1 - r0) * ((float)rest / (float)nk);
    };
    for (int slices = 2 + threadIdx.x; 4 * slices <= 3 * nk; slices += 1024)
        if (reach_at(slices) < thr_floor - 1e-3f)
            atomicMin(&best, slices);
    const int steps = 1 + threadIdx.x;
    if (steps <= steps_most && 4 * steps * wide <= 3 * nk && reach_at(steps * wide) + 0.065f * (float)(steps * wide) / (float)nk < thr_floor - 1e-3f)
        atomicMin(&best_steps, steps);
    __syncthreads();
    if (threadIdx.x == 0) {
        early_nk[g] = best;
        if (head_steps)
            head_steps[g] = best_steps <= steps_most && (!group_enable || group_enable[g]) ? best_steps : 0;
    }
}

void launch_choose_early(hipStream_t s, const PoolDesc &pool, const WorkDesc &w, const TableDesc &tab, float thr_floor)
{
    float *bounds = reinterpret_cast<float *>(w.active);      // (free until the first assignment step; l_stride >= 256 is room enough)
    const bool twice = w.l_stride >= 512;
    const int n_samples = twice ? 2 * kSamples : kSamples;
    const unsigned grid = (unsigned)pool.G * n_samples / 4;
    if (pool.dtype == KVFUSE_BF16)
        sample_bounds_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t *)pool.k, tab.bt, pool.G, pool.P, tab.n, pool.r, n_samples, bounds);
    else
        sample_bounds_kernel<float><<<grid, 256, 0, s>>>((const float *)pool.k, tab.bt, pool.G, pool.P, tab.n, pool.r, n_samples, bounds);
    const int nk = pool.r * (pool.dtype == KVFUSE_BF16 ? 2 : 4) / 64;
    const int wide = pool.dtype == KVFUSE_BF16 ? 2 : 4;
    if (twice)
        choose_early_kernel<2><<<pool.G, 1024, 0, s>>>(bounds, nk, thr_floor, w.early_nk_mem, w.head_steps, head_steps_most(w.long_heads), wide, w.group_enable, w.whole);
    else
        choose_early_kernel<1><<<pool.G, 1024, 0, s>>>(bounds, nk, thr_floor, w.early_nk_mem, w.head_steps, head_steps_most(w.long_heads), wide, w.group_enable, w.whole);
}

// The pairs that the tests left open, 16 lanes per pair: the rest of the product, and the pair's entry in its column's
// candidate list if the whole cosine clears the floor.  HBM-bound: what is left of two blocks per pair (their heads
// were read by the product); a sixteenth of a wavefront's lanes each hold 16 bytes of one row, so a load instruction
// covers 256 consecutive bytes of each of four rows.
template <typename T>
__global__ __launch_bounds__(256) void finish_pairs_kernel(PoolDesc pool, WorkDesc w, float thr_floor)
{
    const int n = min(w.n_pairs[0], w.pair_cap);
    const int sub = threadIdx.x & 15;
    for (int q = (blockIdx.x * 256 + threadIdx.x) >> 4; q < n; q += gridDim.x * 16) {
        const int4 rec = w.pairs[q];
        if (rec.x < 0)
            continue;
        const int g = rec.x / w.r_stride;
        const bool from_start = rec.y < 0;           // (kPairWhole)
        const int64_t pa = (int64_t)g * pool.P + rec.z, pb = (int64_t)g * pool.P + rec.w;
        const float ia = pool.inv_norm_k[pa], ib = pool.inv_norm_k[pb];
        float dot = product_from<T>((const T *)pool.k + pa * pool.r, (const T *)pool.k + pb * pool.r, from_start ? 0 : 4 * w.early_nk[g],
                                    pool.r / Elem<T>::PER16, sub, 16);
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1)
            dot += __shfl_xor(dot, off, 64);
        const float cs = (from_start ? dot : w.pair_head[q] + dot) * ia * ib;
        if (sub == 0 && cs > thr_floor)
            emit_candidate(w.cand_cnt, w.cand_idx, w.cand_val, rec.x, w.cand_cap, rec.y & ~kPairWhole, cs);
    }
}

void launch_finish_pairs(hipStream_t s, const PoolDesc &pool, const WorkDesc &w, float thr_floor)
{
    const unsigned grid = (unsigned)std::min<int64_t>(((int64_t)w.pair_cap + 15) / 16, 256 * 8);
    if (grid == 0)
        return;
    if (pool.dtype == KVFUSE_BF16)
        finish_pairs_kernel<bf16_t><<<grid, 256, 0, s>>>(pool, w, thr_floor);
    else
        finish_pairs_kernel<float><<<grid, 256, 0, s>>>(pool, w, thr_floor);
}

}  // namespace kvfuse
