"""The panel kernel of the similarity step (csrc/panel.hip; heights of large sets whose tests stop early) at the edges of its panels
of 512 right blocks, stages of 64 and runs of left blocks, and of its list of open pairs.  One node per tree (at the first height it
takes every group whose head it can), in enough groups for early rejection; groups are independent, so the first and the last are
compared with the oracle exactly."""
import numpy as np
import pytest
import torch

from paper_2601_03067_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T, D = 16, 64                    # rows of 2 KiB: 32 slices, of which some 6 are multiplied before the test


def _recipe(left, right, related, groups):
    """related: which base the right block j and the left block i copy"""
    rng = np.random.default_rng(left * 10007 + right)
    n = left + right
    src = np.full(n, -1, np.int64)
    if related == "few":                                      # one right block in eight
        src[:left] = np.arange(left)
        src[left + rng.choice(right, right // 8, replace=False)] = rng.integers(0, left, right // 8)
    elif related == "diagonal":                               # 32 open pairs in the 32 x 64 blocks along the diagonal: the list fills up
        src[:left] = np.arange(left)
        src[left:] = np.arange(right) % left
    elif related == "dense":                                  # one pair in 24 in every corner: pieces are multiplied whole
        src[:] = rng.integers(0, 24, n)
    sigma = np.where(np.arange(n) >= left, np.where(np.arange(n) % 3 == 0, 0.0, 0.05), 0.0).astype(np.float32)
    start = np.array([0, left], np.int32)
    count = np.array([left, right], np.int32)
    return wl.Recipe("panel", 9, groups, 1, 1, T, D, torch.bfloat16, 0.9, src, sigma, max(left, 24), start, count, count * T, start, count,
                     np.arange(3, dtype=np.int32))


CASES = [(256, 512, "few", 190),            # one panel, four stages
         (257, 513, "few", 190),            # a panel of one column (two wavefronts per 64 columns), a stage of one row
         (700, 257, "few", 140),            # the smallest panel that takes a wavefront per 64 columns
         (319, 800, "few", 100),            # panels of 512 and 288
         (2100, 256, "few", 50),            # five runs
         (2048, 1100, "diagonal", 12),      # every list is emptied more than once
         (600, 700, "dense", 60)]


@pytest.mark.parametrize("left,right,related,groups", CASES)
def test_tree_matches_oracle(oracle, left, right, related, groups):
    kb = gu.load_binding()
    rec = _recipe(left, right, related, groups)
    print("panel", left, right, related, flush=True)
    assert 2.0 * left * right * T * D * groups >= 5e10        # (the line from which tests stop early)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    for g in range(rec.G):                                    # zero blocks in both sets
        mat["K"][g][mat["bt"][g][torch.tensor([3, 40, left + 5, left + right - 1], device=DEV).long()].long()] = 0
    pick = [0, rec.G - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, f"{left} x {right}")
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, f"{left} x {right} {related}")
    slices, open_pairs, room = kb.early_counts(ctx, plan)
    assert room > 0 and np.all(slices <= 11)                  # the kernel's own limit
    per_group = kb.group_counters(ctx, plan)
    assert per_group[pick, 0].tolist() == [int(r.stats[1]) for r in res]
    assert per_group[pick, 1].tolist() == [int(r.stats[2]) for r in res]
    if related != "dense":                                    # a pair that fuses was left open by the test
        assert open_pairs.sum() >= stats.fused
    else:
        assert open_pairs.sum() < stats.fused


def test_groups_of_both_kernels_at_one_height(oracle):
    """Every second group's keys share a direction, so that their heads are too long for the panel kernel: the ring kernel takes them
    at the same height, and the list of open pairs is one."""
    kb = gu.load_binding()
    left, right, groups = 600, 700, 60
    rec = _recipe(left, right, "few", groups)
    print("panel and ring", left, right, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(6)
    for g in range(1, groups, 2):
        mat["K"][g] = (mat["K"][g].float() + 1.3 * torch.randn(rec.r, generator=gen, device=DEV)).to(rec.dtype)
    pick = [0, 1, groups - 2, groups - 1]
    _compare(oracle, kb, rec, mat, pick)


def _compare(oracle, kb, rec, mat, pick):
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, rec.name)
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, rec.name)
    slices, open_pairs, room = kb.early_counts(ctx, plan)
    per_group = kb.group_counters(ctx, plan)
    assert room > 0 and per_group[pick, 0].tolist() == [int(r.stats[1]) for r in res] and min(per_group[pick, 0]) > 0
    long = np.arange(rec.G) % 2 == 1 if len(pick) == 4 else np.zeros(rec.G, bool)
    assert np.array_equal(slices > 11, long)


@pytest.mark.parametrize("common", [0, 40, 200])
def test_heights_behind_each_other(oracle, common):
    """Four requests of 300 blocks: at the second height either kernel may take a group, by what the first has left open (no tile
    multiplied whole, none, one in every node)."""
    groups, count = 60, np.full(4, 300, np.int32)
    src = np.arange(1200) + 300
    for u in range(4):
        src[300 * u:300 * u + common] = np.arange(common)
    src[1190:1200] = src[290:300] = 1                            # and a few that fuse in any case
    start = np.arange(4, dtype=np.int32) * 300
    rec = wl.Recipe("panel heights", 10, groups, 1, 1, T, D, torch.bfloat16, 0.9, src.astype(np.int64), np.full(1200, 0.03, np.float32), 1500,
                    start, count, count * T, start, count, np.arange(5, dtype=np.int32))
    print("panel heights", common, flush=True)
    _compare(oracle, gu.load_binding(), rec, wl.materialise(rec, DEV, phys_perm=True), [0, groups - 1])
