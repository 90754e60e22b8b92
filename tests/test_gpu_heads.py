"""The head copies of the panel kernel (csrc/heads.hip, csrc/panel.hip): blocks whose copies are bad or whose bound is tight, among
ordinary ones, so that groups still take the kernel.  One node per tree; the first and the last group are compared with the oracle
exactly.  The bound itself: tests/test_screen_bounds.py."""
import numpy as np
import pytest
import torch

from paper_2601_03067_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T, D, LEFT, RIGHT, GROUPS = 16, 64, 1100, 1100, 21        # about the smallest trees of this shape that copies are made for


def _spoil(K, kind, gen, thr=0.9):
    """K [n][r] float64, changed in place: blocks 0 .. 39 of the left set and as many of the right one, which are their near copies"""
    n, r = K.shape
    left, right = torch.arange(40, device=K.device), torch.arange(LEFT, LEFT + 40, device=K.device)
    noise = torch.randn(40, r, generator=gen, device=K.device, dtype=torch.float64)
    scale = torch.ones(80, 1, device=K.device, dtype=torch.float64)
    if kind == "spike in the head":                       # beyond the copy's largest value: the whole head is mostly error
        K[left, 7 + left % 50] = 40.0
    elif kind == "spike in the tail":
        K[left, 900] = 40.0
    elif kind == "quiet head":                            # far below the norm, down to nothing
        K[left, :384] *= torch.logspace(0, -40, 40, device=K.device, dtype=torch.float64)[:, None]
        K[left[30:], :384] = 0.0
    elif kind == "loud head":                             # nothing behind the head, which then decides alone
        K[left, 64 * (1 + left % 6)[0]:] = 0.0
    elif kind == "scales":
        scale = torch.exp2(torch.arange(80, device=K.device, dtype=torch.float64).clamp(max=78)[:, None] - 39.0) / r ** 0.5      # norms of 2^-39 to 2^39
    # near copies at cosines of thr +- 0.02, on both sides of the threshold
    c = torch.linspace(thr - 0.02, thr + 0.02, 40, device=K.device, dtype=torch.float64)[:, None]
    u = K[left]
    noise -= (noise * u).sum(1, keepdim=True) / (u * u).sum(1, keepdim=True) * u
    if kind == "loud head":
        noise[:, 64:] *= (u != 0)[:, 64:]
        noise -= (noise * u).sum(1, keepdim=True) / (u * u).sum(1, keepdim=True) * u
    noise *= u.norm(dim=1, keepdim=True) / noise.norm(dim=1, keepdim=True)
    K[right] = c * u + (1 - c * c).sqrt() * noise
    K[left] *= scale[:40]
    K[right] *= scale[40:].flip(0)


@pytest.mark.parametrize("kind", ["spike in the head", "spike in the tail", "quiet head", "loud head", "scales"])
def test_blocks_with_bad_copies(oracle, kind):
    kb = gu.load_binding()
    n = LEFT + RIGHT
    start, count = np.array([0, LEFT], np.int32), np.array([LEFT, RIGHT], np.int32)
    rec = wl.Recipe("heads", 12, GROUPS, 1, 1, T, D, torch.bfloat16, 0.9, np.full(n, -1, np.int64), np.zeros(n, np.float32), 1, start, count,
                    count * T, start, count, np.arange(3, dtype=np.int32))
    print("heads", kind, flush=True)
    mat = wl.materialise(rec, DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    for g in range(GROUPS):
        k = mat["K"][g].double()
        _spoil(k, kind, gen)
        mat["K"][g] = k.to(torch.bfloat16)
    pick = [0, GROUPS - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, kind)
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, kind)
    slices, _, room = kb.early_counts(ctx, plan)
    assert room > 0 and np.all(slices <= 11)                  # heads that the copies hold
    per_group = kb.group_counters(ctx, plan)
    assert per_group[pick, 0].tolist() == [int(r.stats[1]) for r in res] and 10 <= min(per_group[pick, 0]) and max(per_group[pick, 0]) <= 30


@pytest.mark.parametrize("thr", [0.7, 0.8, 0.9, 0.95, 0.98])
def test_heads_of_every_length(oracle, thr):
    """Two requests of four chunks: heads of other lengths (at 0.7 long copies), made at the first height or a later one, and blocks that
    a merge has rewritten, whose copies are made anew."""
    groups, n, count = 12, 8 * 650, np.full(8, 650, np.int32)
    rng = np.random.default_rng(5)
    src = np.where(rng.random(n) < 0.1, rng.integers(0, 650, n), np.arange(n) + 650).astype(np.int64)
    start = np.arange(8, dtype=np.int32) * 650
    rec = wl.Recipe("heads lengths", 13, groups, 1, 1, T, D, torch.bfloat16, thr, src, np.full(n, 0.02, np.float32), n + 650, start, count, count * T,
                    start, count, np.array([0, 4, 8], np.int32))
    print("heads at", thr, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    pick = [0, groups - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, rec.name)
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, rec.name)
    assert min(int(r.stats[1]) for r in res) > 100


# left, right, thr, groups: ends of panels (512 and, at 0.7, 256 right blocks), stages (64, 32) and runs, panels of few columns
SHAPES = [(1100, 1025, 0.9, 22), (1153, 1100, 0.9, 20), (2049, 770, 0.9, 16), (2100, 2049, 0.7, 6), (2113, 2180, 0.7, 6)]


@pytest.mark.parametrize("left,right,thr,groups", SHAPES)
@pytest.mark.parametrize("related", ["few", "diagonal"])
def test_edges_of_panels(oracle, left, right, thr, groups, related):
    """Few related pairs, or one for every right block along the diagonal: the list of open pairs then fills up and is emptied on the way."""
    kb = gu.load_binding()
    n = left + right
    rng = np.random.default_rng(n)
    src = np.full(n, -1, np.int64)
    src[:left] = np.arange(left)
    if related == "few":
        src[left + rng.choice(right, right // 16, replace=False)] = rng.integers(0, left, right // 16)
    else:
        src[left:] = np.arange(right) % left
    start, count = np.array([0, left], np.int32), np.array([left, right], np.int32)
    rec = wl.Recipe("panel ends", 14, groups, 1, 1, T, D, torch.bfloat16, thr, src, np.where(np.arange(n) >= left, 0.05, 0.0).astype(np.float32), left, start,
                    count, count * T, start, count, np.arange(3, dtype=np.int32))
    print("panel ends", left, right, thr, related, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    for g in range(groups):                                   # zero blocks in both sets
        mat["K"][g][mat["bt"][g][torch.tensor([3, left - 1, left + 5, n - 1], device=DEV).long()].long()] = 0
    pick = [0, groups - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, rec.name)
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, rec.name)
    _, open_pairs, room = kb.early_counts(ctx, plan)
    assert room > 0 and open_pairs.sum() >= stats.fused       # (the ring kernel multiplies whole tiles along the diagonal, whose pairs are not left open)


def test_height_between_that_is_not_the_panel_kernels(oracle):
    """The sets of the second height are too unequal for big tiles; what the merges of the first two rewrite has new copies at the third."""
    kb = gu.load_binding()
    groups, count = 5, np.array([1100, 1100, 40, 40] * 2, np.int32)
    n = int(count.sum())
    start = (np.cumsum(count) - count).astype(np.int32)
    rng = np.random.default_rng(8)
    src = np.where(rng.random(n) < 0.08, rng.integers(0, 200, n), np.arange(n) + 200).astype(np.int64)
    rec = wl.Recipe("panel between", 15, groups, 1, 1, T, D, torch.bfloat16, 0.9, src, np.full(n, 0.1, np.float32), n + 200, start, count, count * T,
                    start, count, np.arange(9, dtype=np.int32))
    print("panel between", flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    pick = [0, groups - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=64)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, rec.name)
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, False, rec.name)
    assert kb.early_counts(ctx, plan)[2] > 0 and min(int(r.stats[1]) for r in res) > 100
