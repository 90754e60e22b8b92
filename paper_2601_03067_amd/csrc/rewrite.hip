// a5: block-table rewrite (Algorithm 1: "evict fused blocks", "update block-table"; results section: the runner
// hands the scheduler the updated tables so that it can free unused blocks and raise reference counts).
//
// Integer gather/scatter, HBM-bound and small: one pass over the table follows the remap chain of each entry to
// its surviving block and recounts references; a second one refreshes the per-logical scales and lists every group's
// freed ids in ascending order.
#include "common.h"

namespace kvfuse {

__global__ void rewrite_clear_kernel(int32_t *__restrict__ refcount, int64_t total)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < total)
        refcount[i] = 0;
}

__global__ void rewrite_chase_kernel(TableDesc tab, int G, int P)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)G * tab.n)
        return;
    const int64_t gp = (i / tab.n) * P;
    int p = tab.bt[i];
    if (p < 0 || p >= P)
        return;
    // A block fused at one height can be fused again higher up: follow the chain.  Its length is at most the
    // number of heights; the bound only guards against a malformed (cyclic) remap table.
    for (int hop = 0; hop < 64; ++hop) {
        const int q = tab.remap[gp + p];
        if (q < 0 || q >= P || q == p)
            break;
        p = q;
    }
    tab.bt[i] = p;
    atomicAdd(&tab.refcount[gp + p], 1);
}

// The scales of table entry i.
__device__ __forceinline__ void rewrite_scale(const TableDesc &tab, int64_t i, int P, const double *__restrict__ norm_k,
                                              const double *__restrict__ norm_v)
{
    const int64_t gp = (i / tab.n) * P;
    const int p = tab.bt[i];
    if (p < 0 || p >= P)
        return;
    if (tab.refcount[gp + p] <= 1) {      // never fused: the entry still is its own raw block
        tab.scale_k[i] = 1.0f;
        tab.scale_v[i] = 1.0f;
        return;
    }
    const double nk = norm_k[gp + p], nv = norm_v[gp + p];
    tab.scale_k[i] = nk == 0.0 ? 0.0f : (float)(tab.orig_norm_k[i] / nk);
    tab.scale_v[i] = nv == 0.0 ? 0.0f : (float)(tab.orig_norm_v[i] / nv);
}

// Two passes that do not depend on each other, in one launch.  The first n_lists workgroups take a group at a time: freed ids
// (blocks that were fused away) in ascending order, and the live count; their walk over the pool is a chain of barriers, so they
// start first, are as wide as can be and load a step ahead (141 355 blocks a group: 394 us with 256 threads, 109 us).  Groups of
// at most 256 blocks are one step either way, which 256 threads take (whole rewrite, us, 1024 / 256 threads: 100 000 groups of 8
// blocks 235 / 62, 20 000 of 100 71 / 32).  The others refresh the scales.
template <int NT>
__global__ __launch_bounds__(NT) void rewrite_finish_kernel(TableDesc tab, int G, int P, const double *__restrict__ norm_k,
                                                            const double *__restrict__ norm_v, int n_lists,
                                                            int32_t *__restrict__ free_list, int32_t *__restrict__ n_free,
                                                            int32_t *__restrict__ n_phys)
{
    constexpr int NW = NT / 64;
    __shared__ int wave_tot[2][NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if ((int)blockIdx.x >= n_lists) {
        const int64_t step = (int64_t)(gridDim.x - n_lists) * NT;
        for (int64_t i = (int64_t)(blockIdx.x - n_lists) * NT + tid; i < (int64_t)G * tab.n; i += step)
            rewrite_scale(tab, i, P, norm_k, norm_v);
        return;
    }
    for (int g = blockIdx.x; g < G; g += n_lists) {
        const int64_t gp = (int64_t)g * P;
        int freed = 0, live = 0;
        int next_remap = tid < P ? tab.remap[gp + tid] : -1, next_refs = tid < P ? tab.refcount[gp + tid] : 0;
        for (int p0 = 0, buf = 0; p0 < P; p0 += NT, buf ^= 1) {
            const int p = p0 + tid, ahead = p + NT;
            const unsigned long long mf = __ballot(next_remap >= 0);
            const unsigned long long ml = __ballot(next_refs > 0);
            const bool is_free = next_remap >= 0;
            next_remap = ahead < P ? tab.remap[gp + ahead] : -1;
            next_refs = ahead < P ? tab.refcount[gp + ahead] : 0;
            if (lane == 0)
                wave_tot[buf][wave] = __popcll(mf);
            __syncthreads();                 // (one barrier a step: the other buffer is written before the next one)
            int pre = 0, tot = 0;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                const int c = wave_tot[buf][k];
                pre += k < wave ? c : 0;
                tot += c;
            }
            if (is_free && free_list)
                free_list[gp + freed + pre + __popcll(mf & ((1ull << lane) - 1ull))] = p;
            freed += tot;
            live += __popcll(ml);
        }
        // live counts are per wave: add them up
        __syncthreads();
        if (lane == 0)
            wave_tot[0][wave] = live;
        __syncthreads();
        if (tid == 0) {
            if (n_free)
                n_free[g] = freed;
            if (n_phys) {
                int sum = 0;
                for (int k = 0; k < NW; ++k)
                    sum += wave_tot[0][k];
                n_phys[g] = sum;
            }
        }
        __syncthreads();         // the counts are read before the next group's are written
    }
}

template <int NT>
static void launch_finish(hipStream_t s, const PoolDesc &pool, const TableDesc &tab, int32_t *free_list, int32_t *n_free, int32_t *n_phys)
{
    // (at most 2^30 threads for the lists and 2^31 for the scales: a launch has fewer than 2^32)
    const int64_t ne = (int64_t)pool.G * tab.n;
    const int n_lists = free_list || n_free || n_phys ? std::min(pool.G, (1 << 30) / NT) : 0;
    const int64_t grid = n_lists + std::min<int64_t>((ne + NT - 1) / NT, (1ll << 31) / NT);
    if (grid > 0)
        rewrite_finish_kernel<NT><<<(unsigned)grid, NT, 0, s>>>(tab, pool.G, pool.P, pool.norm_k, pool.norm_v, n_lists, free_list, n_free, n_phys);
}

void launch_rewrite(hipStream_t s, const PoolDesc &pool, const TableDesc &tab, int32_t *free_list, int32_t *n_free,
                    int32_t *n_phys)
{
    const int64_t nb = (int64_t)pool.G * pool.P;
    const int64_t ne = (int64_t)pool.G * tab.n;
    if (nb > 0)
        rewrite_clear_kernel<<<(unsigned)((nb + 255) / 256), 256, 0, s>>>(tab.refcount, nb);
    if (ne > 0)
        rewrite_chase_kernel<<<(unsigned)((ne + 255) / 256), 256, 0, s>>>(tab, pool.G, pool.P);
    if (pool.P <= 256)
        launch_finish<256>(s, pool, tab, free_list, n_free, n_phys);
    else
        launch_finish<1024>(s, pool, tab, free_list, n_free, n_phys);
}

}  // namespace kvfuse
