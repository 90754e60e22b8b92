// Head copies (heads.h) of the blocks that a merge has rewritten, before a height whose launches do not see to them.
#include <algorithm>

#include "heads.h"

namespace kvfuse {

template <bool LONG>
__global__ __launch_bounds__(256) void heads_of_targets_kernel(PoolDesc pool, WorkDesc w, int height, float thr_floor)
{
    heads_of_targets<LONG>(pool, w, height, thr_floor, blockIdx.x, gridDim.x);
}

void launch_heads_of_targets(hipStream_t s, const PoolDesc &pool, const WorkDesc &w, int height, float thr_floor)
{
    const unsigned grid = (unsigned)std::min<int64_t>(((int64_t)w.G * w.l_stride + 15) / 16, 256 * 8);
    if (grid == 0)
        return;
    if (w.long_heads)
        heads_of_targets_kernel<true><<<grid, 256, 0, s>>>(pool, w, height, thr_floor);
    else
        heads_of_targets_kernel<false><<<grid, 256, 0, s>>>(pool, w, height, thr_floor);
}

}  // namespace kvfuse
