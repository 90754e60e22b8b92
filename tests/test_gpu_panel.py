"""The panel kernel of the similarity step (csrc/panel.hip; heights of large sets whose tests stop early) at the edges of its panels
of 512 right blocks, stages of 64 and runs of left blocks, and of its lists of open pairs.  One node per tree, in enough groups for the
plan to choose it; groups are independent, so the first and the last are compared with the oracle exactly."""
import math

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
    elif related == "overflow":                               # 2.4 open pairs per left block, the call's list holds 1.6
        src[:] = rng.integers(0, 290, n)
    elif related == "dense":                                  # one pair in 24 in every corner: pieces are multiplied whole
        src[:] = rng.integers(0, 24, n)
    sigma = np.where(np.arange(n) >= left, np.where(np.arange(n) % 3 == 0, 0.0, 0.05), 0.0).astype(np.float32)
    start = np.array([0, left], np.int32)
    count = np.array([left, right], np.int32)
    return wl.Recipe("panel", 9, groups, 1, 1, T, D, torch.bfloat16, 0.9, src, sigma, max(left, 290), start, count, count * T, start, count,
                     np.arange(3, dtype=np.int32))


CASES = [(256, 512, "few", 1160),           # one panel, four stages
         (257, 513, "few", 190),            # a panel of one column (two wavefronts per 64 columns), a stage of one row
         (700, 257, "few", 256),            # the smallest panel that takes a wavefront per 64 columns
         (319, 800, "few", 100),            # panels of 512 and 288
         (2100, 300, "few", 100),           # five runs
         (2048, 1100, "diagonal", 400),     # every list is emptied more than once
         (600, 700, "overflow", 60),
         (600, 700, "dense", 60)]


def _chosen(left, right, groups):
    """panel_run of csrc/host.hip for one node: whether the plan lays out panel items"""
    up = lambda a, b: -(-a // b)
    run, stages, panels, tiles = 32, up(left, 64), up(right, 512), up(left, 256)
    while run > 8 and groups * panels * up(stages, run) < 2048:
        run //= 2
    rt, n = min(up(tiles, 4), 4), up(stages, run)
    cols = right // 512 + (0 if right % 512 == 0 else 0.75 if right % 512 <= 256 else 1)
    rounds = lambda total, item: item * math.ceil(total * groups / 256 / item - 1e-9)
    ring = rounds(up(right, 256) * (8.4 * up(tiles, rt) + 7.94 * tiles), 8.4 + 7.94 * rt)
    return rounds(14.5 * n * panels + 3.31 * stages * cols, 14.5 + 3.31 * up(stages, n)) + 14 < 0.95 * ring


@pytest.mark.parametrize("left,right,related,groups", CASES)
def test_tree_matches_oracle(oracle, left, right, related, groups):
    kb = gu.load_binding()
    rec = _recipe(left, right, related, groups)
    print("panel", left, right, related, flush=True)
    assert 2.0 * left * right * T * D * groups >= 5e10        # (the line from which tests stop early)
    assert _chosen(left, right, groups)
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
    assert (open_pairs.max() > room) == (related == "overflow")
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
    assert _chosen(left, right, groups)
    print("panel and ring", left, right, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(6)
    for g in range(1, groups, 2):
        mat["K"][g] = (mat["K"][g].float() + 1.3 * torch.randn(rec.r, generator=gen, device=DEV)).to(rec.dtype)
    pick = [0, 1, groups - 2, groups - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, "panel and ring")
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, "panel and ring")
    slices, open_pairs, room = kb.early_counts(ctx, plan)
    assert room > 0 and np.all(slices[0::2] <= 11) and np.all(slices[1::2] > 11)
    per_group = kb.group_counters(ctx, plan)
    assert per_group[pick, 0].tolist() == [int(r.stats[1]) for r in res] and min(per_group[pick, 0]) > 0
