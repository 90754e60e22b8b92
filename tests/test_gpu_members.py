"""Re-check and merge launch by launch (csrc/assign.hip, csrc/merge.hip) over what their loops go by: left rows that come close to a
right block (rounds of four, of two, of one; more than the list holds), members of a target (the first two, pairs after them, more
than a wavefront has lanes), and blocks of every number of pieces per lane, whole and with a rest.  Exactly the oracle's tables, pools,
counts, scales and norms."""
import numpy as np
import pytest
import torch

from paper_2601_03067_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# copies of one block: so many on the left, so many on the right
SETS = [(1, 1), (1, 2), (1, 3), (1, 4), (2, 9), (3, 7), (5, 131), (6, 33), (9, 20), (20, 41), (1, 66), (1, 67), (1, 131)]
BLOCKS = [(1, 64, torch.bfloat16), (8, 104, torch.bfloat16), (16, 72, torch.bfloat16), (16, 128, torch.bfloat16),
          (32, 104, torch.bfloat16), (32, 128, torch.bfloat16), (4, 64, torch.float32), (16, 36, torch.float32),
          (16, 64, torch.float32), (16, 104, torch.float32), (16, 128, torch.float32)]


def _recipe(left, right, t, d, dtype):
    n = left + right
    start, cnt = np.asarray([0, left], np.int32), np.asarray([left, right], np.int32)
    return wl.Recipe("members", 8, 2, 1, 1, t, d, dtype, 0.9, np.zeros(n, np.int64), np.full(n, 0.03, np.float32), 1, start, cnt, cnt * t,
                     start, cnt, np.arange(3, dtype=np.int32))


@pytest.mark.parametrize("t,d,dtype", BLOCKS, ids=[f"{t}x{d}-{str(dtype)[6:]}" for t, d, dtype in BLOCKS])
@pytest.mark.parametrize("rule", ["argmax", "first_row"])
def test_rounds_and_members(oracle, t, d, dtype, rule):
    for left, right in SETS:
        print("members", left, right, t, d, dtype, rule, flush=True)
        rec = _recipe(left, right, t, d, dtype)
        mat = wl.materialise(rec, DEV, phys_perm=True)
        host = gu.host_copy(mat)
        cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, timing=True, rule=rule)      # (timed stages: never the whole call in one launch)
        res = gu.oracle_fuse(oracle, rec, host, rule=rule)
        gu.check_ambiguity(res, f"{left} {right} {rule}")
        for g, r in enumerate(res):
            gu.compare_group(r, cache, g, dtype == torch.float32, f"{left} {right} {t} {d} {dtype} {rule}")
        assert stats.fused == sum(int(r.stats[1]) for r in res) == 2 * right
