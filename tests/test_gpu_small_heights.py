"""Similarity of small heights (32 x 32 tiles, the row shared out among the wavefronts of a workgroup) and the line to the
tiled kernel above it: whole trees against the oracle, exactly."""
import pytest
import torch

from paper_2601_03067_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (requests, blocks each, layers, KV heads, block size, head dim, dtype)
CASES = [(5, 1, 1, 2, 16, 64, torch.bfloat16),           # sets of one block, an odd unit carried up
         (4, 31, 1, 1, 16, 128, torch.bfloat16),         # one ragged tile, then 2 x 2
         (3, 33, 2, 1, 16, 64, torch.float32),           # a tile and one row more, both directions
         (2, 32, 1, 3, 32, 128, torch.bfloat16),         # exactly one tile, the longest rows
         (9, 20, 4, 8, 16, 64, torch.bfloat16),          # one tile per node at the low height, too many tiles above: tiled kernel
         (2, 500, 1, 2, 16, 64, torch.bfloat16),         # 512 tiles: the last height of the small kernel
         (2, 520, 1, 2, 16, 64, torch.float32)]          # 578: the tiled kernel


@pytest.mark.parametrize("rule", ["argmax", "first_row"])
@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_tree_matches_oracle(oracle, case, rule):
    n_req, blocks, layers, kv_heads, t, d, dtype = case
    print("small heights", case, rule, flush=True)
    rec = wl.llama8b_bff(n_req=n_req, tokens=blocks * t, prefix_tokens=blocks // 4 * t, near_pool=max(8, blocks // 3), layers=layers,
                         kv_heads=kv_heads, t=t, d=d, dtype=dtype)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    host = gu.host_copy(mat)
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, rule=rule)
    res = gu.oracle_fuse(oracle, rec, host, rule=rule)
    gu.check_ambiguity(res, str(case))
    for g, r in enumerate(res):
        gu.compare_group(r, cache, g, dtype == torch.float32, str(case))
    assert stats.fused == sum(int(r.stats[1]) for r in res)
    assert stats.near_threshold == sum(int(r.stats[2]) for r in res)
