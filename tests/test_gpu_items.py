"""Work items of the ring kernel (csrc/similarity.hip): laid out by one workgroup or by two launches, for groups that have many, few or
none, with runs of one to four row tiles.  One tree of several units per group, all groups fused differently; compared with the oracle
exactly."""
import numpy as np
import pytest
import torch

from paper_2601_03067_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# groups, units, blocks per unit, copies, off: every off-th group is switched off
CASES = [(1, 2, 1, 0, 0),          # a tile of one pair
         (3, 3, 129, 40, 2),       # a unit that waits a height; one group switched off
         (2, 2, 700, 100, 0),      # more than four row tiles of 128: an item each
         (5, 2, 513, 500, 0),      # five groups in one workgroup's slots
         (300, 2, 40, 7, 7),       # slots of many groups per workgroup
         (1030, 2, 34, 9, 0),      # more nodes than one workgroup takes
         (40, 9, 300, 11, 3),      # several heights, two launches at the first
         (4096, 3, 140, 9, 5),     # items of all groups without gaps, for the last time ...
         (4097, 3, 140, 9, 5),     # ... and every group with room of its own: four items of a node, none of a switched-off group
         (2, 2, 4200, 60, 0)]      # room for more items than one workgroup lays out; single tiles, 34 rows of them


@pytest.mark.parametrize("groups,units,count,copies,off", CASES)
def test_tree_matches_oracle(oracle, groups, units, count, copies, off):
    kb = gu.load_binding()
    n = units * count
    src = np.arange(n, dtype=np.int64)
    src[count:][np.arange(n - count) % 5 == 0] = np.arange(n - count)[np.arange(n - count) % 5 == 0] % max(copies, 1)
    start = np.arange(units, dtype=np.int32) * count
    cnt = np.full(units, count, np.int32)
    rec = wl.Recipe("items", 12, groups, 1, 1, 4, 32, torch.bfloat16, 0.9, src, np.full(n, 0.02, np.float32), n, start, cnt, cnt * 4, start, cnt,
                    np.arange(units + 1, dtype=np.int32))
    print("items", groups, units, count, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    on = np.ones(groups, np.uint8)
    if off:
        on[::off] = 0
    pick = sorted({0, 1 % groups, groups // 2, groups - 1})
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    ctx = kb.Context(DEV)
    cache = kb.Cache(mat["K"], mat["V"], mat["bt"], rec.t, rec.d)
    plan = kb.Plan(ctx, cache, kb.tree_spec(rec.leaf_start, rec.leaf_count, rec.unit_leaf_ptr), 64)
    # (the whole tree in one launch and the kernel for small heights have no items: a switched-off group or the fp8 copies rule them out)
    kb.set_screen_fp8(ctx, plan)
    if off:
        kb.set_group_mask(ctx, plan, torch.from_numpy(on).to(DEV))
    kb.fuse_tree(ctx, plan, rec.thr)
    torch.cuda.synchronize()
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, "items")
    for r, g in zip(res, pick):
        if on[g]:
            gu.compare_group(r, cache, g, False, f"{groups} x {units} x {count}")
        else:
            assert int(cache.n_phys[g]) == n and int(cache.n_free[g]) == 0
    fused = kb.group_counters(ctx, plan)[:, 0]
    assert np.all(fused[on == 0] == 0)
    assert n == 2 or min(int(fused[g]) for g in pick if on[g]) > 0


@pytest.mark.parametrize("shared", [0, 300])
def test_first_tiles_expected_whole(oracle, shared):
    """Four requests, the first two and the last two copies of each other: a tile of every node runs to its full length at the first height,
    so that the second height's first tiles are multiplied whole at once, with nothing in them (shared = 0) or copies (300).  Keys
    with a common direction, whose heads are too long for the panel kernel."""
    kb = gu.load_binding()
    groups, count = 60, np.full(4, 300, np.int32)
    base = np.arange(300)
    src = np.concatenate([base, base, base + 300 - shared, base + 300 - shared]).astype(np.int64)
    start = np.arange(4, dtype=np.int32) * 300
    rec = wl.Recipe("whole first", 13, groups, 1, 1, 16, 64, torch.bfloat16, 0.9, src, np.full(1200, 0.03, np.float32), 600, start, count,
                    count * 16, start, count, np.arange(5, dtype=np.int32))
    print("whole first", shared, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    for g in range(groups):
        mat["K"][g] = (mat["K"][g].float() + 1.3 * torch.randn(rec.r, generator=gen, device=DEV)).to(rec.dtype)
    pick = [0, groups - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, rec.name)
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, rec.name)
    slices, open_pairs, room = kb.early_counts(ctx, plan)
    assert room > 0 and np.all((slices > 11) & (slices < 32))                 # tests there are, and not the panel kernel's
    assert stats.fused == groups * (600 + shared)
