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


def _up(a, b):
    return -(-a // b)


def _layout(src, units, count, groups, n_on):
    """What the plan and the device are to do with a tree of `units` sets of `count` blocks, a right block fusing where its base is
    in the left set: by height (how items are laid out, row tiles of the nodes' items).  few: by one workgroup; list: by two launches,
    without gaps; rooms: by two launches, every group in its own room."""
    heights = {}

    def over(lo, hi):
        if hi - lo == 1:
            return count, src[lo * count:(lo + 1) * count], 0
        mid = lo + (hi - lo) // 2
        a, b = over(lo, mid), over(mid, hi)
        h = 1 + max(a[2], b[2])
        heights.setdefault(h, []).append((a[0], b[0], len(a[1]), len(b[1])))
        return a[0] + b[0], np.concatenate([a[1], b[1][~np.isin(b[1], a[1])]]), h

    over(0, units)
    out = []
    for h in sorted(heights):
        nodes = heights[h]
        big = sum(l * r * min(l, r) for l, r, _, _ in nodes) >= 256 * sum(l * r for l, r, _, _ in nodes)
        bm = 256 if big else 128
        room = sum(_up(r, bm) * (_up(l, bm) if _up(l, bm) < 4 else max(4, _up(_up(l, bm), 4))) for l, r, _, _ in nodes)
        tiles = sum(_up(l, bm) * _up(r, bm) for _, _, l, r in nodes)
        how = "few" if groups * len(nodes) <= 1024 and groups * room <= 1024 else "list" if groups <= 4096 else "rooms"
        most = 4
        if max(max(l, r) for l, r, _, _ in nodes) > 4 * bm:
            if how == "few" and tiles * n_on <= groups * room:
                most = 1
            elif how != "few" and tiles <= room:
                most = min(max(tiles * groups // 4096, 1), 4)
        out.append((how, sorted({min(_up(_up(l, bm), 4), most) for _, _, l, _ in nodes})))
    return out


def _some_copies(units, count, copies):
    """Every fifth block behind the first set is one of the first `copies` blocks"""
    n = units * count
    src = np.arange(n, dtype=np.int64)
    src[count:][np.arange(n - count) % 5 == 0] = np.arange(n - count)[np.arange(n - count) % 5 == 0] % max(copies, 1)
    return src


def _repeated(units, count, keep):
    """Every other set repeats the one before it, but for its last `keep` blocks"""
    src = np.arange(units * count, dtype=np.int64)
    for q in range(1, units, 2):
        src[q * count:(q + 1) * count - keep] = src[(q - 1) * count:q * count - keep]
    return src


# groups, units, blocks per unit, how they repeat and its argument, off: every off-th group is switched off; by height, how the items
# are laid out and row tiles of an item
CASES = [(1, 2, 1, _some_copies, 0, 0, [("few", [1])]),                                     # a tile of one pair
         (3, 3, 129, _some_copies, 40, 2, [("few", [1]), ("few", [1])]),                    # a unit that waits a height; one group switched off
         (2, 2, 700, _some_copies, 100, 0, [("few", [1])]),                                 # three row tiles of 256
         (5, 2, 513, _some_copies, 500, 0, [("few", [1])]),
         (300, 2, 40, _some_copies, 7, 7, [("few", [1])]),                                  # an item each, or none
         (1030, 2, 34, _some_copies, 9, 0, [("list", [1])]),                                # more nodes than one workgroup takes; slots of many groups
         (40, 9, 300, _some_copies, 11, 3, [("few", [1])] * 4),                             # several nodes and heights; short items at the last one
         (4096, 3, 140, _some_copies, 9, 5, [("list", [1])] * 2),                           # items of all groups without gaps, for the last time ...
         (4097, 3, 140, _some_copies, 9, 5, [("rooms", [1])] * 2),                          # ... and every group with room of its own, some empty
         (2, 2, 4200, _some_copies, 60, 0, [("few", [4])]),                                 # runs of four row tiles, the last one short
         (80, 9, 300, _repeated, 60, 7, [("list", [1]), ("list", [1]), ("few", [1]), ("list", [1])]),   # several nodes of several items in two launches
         (2, 4, 2600, _repeated, 50, 0, [("few", [3]), ("few", [1])]),                      # sets shrink: runs of three, then single tiles
         (70, 4, 2600, _repeated, 50, 3, [("list", [3]), ("list", [2])]),                   # ... then of two
         (40, 4, 1300, _repeated, 30, 0, [("list", [2]), ("list", [1])])]


@pytest.mark.parametrize("groups,units,count,repeat,arg,off,layout", CASES, ids=["-".join(str(x) for x in c[:3]) for c in CASES])
def test_tree_matches_oracle(oracle, groups, units, count, repeat, arg, off, layout):
    kb = gu.load_binding()
    n = units * count
    src = repeat(units, count, arg)
    on = np.ones(groups, np.uint8)
    if off:
        on[::off] = 0
    assert _layout(src, units, count, groups, int(on.sum())) == layout
    start = np.arange(units, dtype=np.int32) * count
    cnt = np.full(units, count, np.int32)
    rec = wl.Recipe("items", 12, groups, 1, 1, 4, 32, torch.bfloat16, 0.9, src, np.full(n, 0.02, np.float32), n, start, cnt, cnt * 4, start, cnt,
                    np.arange(units + 1, dtype=np.int32))
    print("items", groups, units, count, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
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


def _marked(plan, groups, mark):
    """Whether the plan's work items hold, one after the other for every group, the first item of node 0 with this mark (row tiles, and 64
    for a first tile that is multiplied whole at once)"""
    words = plan.workspace[-plan.workspace.data_ptr() % 256:]
    items = words[:words.numel() // 16 * 16].view(torch.int32).view(-1, 4).cpu().numpy()
    want = np.array([(0, 0, mark, g) for g in range(groups)], np.int32)
    at = np.nonzero((items == want[0]).all(1))[0]
    return any(i + groups <= len(items) and np.array_equal(items[i:i + groups], want) for i in at)


def _fuse_with_common_direction(oracle, name, src, groups, count, n_base):
    """Tree of four sets; keys share a direction, so that heads are too long for the panel kernel"""
    kb = gu.load_binding()
    start, cnt = np.arange(4, dtype=np.int32) * count, np.full(4, count, np.int32)
    rec = wl.Recipe(name, 13, groups, 1, 1, 16, 64, torch.bfloat16, 0.9, src, np.full(4 * count, 0.03, np.float32), n_base, start, cnt,
                    cnt * 16, start, cnt, np.arange(5, dtype=np.int32))
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
    return plan, stats


@pytest.mark.parametrize("shared", [0, 300])
def test_first_tiles_expected_whole(oracle, shared):
    """Four requests, the first two and the last two copies of each other: a tile of every node runs to its full length at the first height,
    so that the second height's first tiles are multiplied whole at once, with nothing in them (shared = 0) or copies (300)."""
    groups, base = 60, np.arange(300)
    src = np.concatenate([base, base, base + 300 - shared, base + 300 - shared]).astype(np.int64)
    print("whole first", shared, flush=True)
    plan, stats = _fuse_with_common_direction(oracle, "whole first", src, groups, 300, 600)
    assert stats.fused == groups * (600 + shared)
    assert _marked(plan, groups, 64 + 1)


@pytest.mark.parametrize("where", ["nowhere", "first tile", "second row tile"])
def test_row_tiles_behind_a_first_tile_expected_whole(oracle, where):
    """Runs of three row tiles whose first one is multiplied whole at once: the others are tested first, and settled by the test or
    multiplied whole in their turn."""
    groups, count, copies = 6, 1300, 256
    src = np.arange(4 * count, dtype=np.int64)
    src[count:count + copies] = np.arange(copies)                             # a first tile of copies in either node of the first height
    src[3 * count:3 * count + copies] = 2 * count + np.arange(copies)
    if where != "nowhere":
        first = 0 if where == "first tile" else 256
        src[2 * count:2 * count + copies] = first + np.arange(copies)
        src[3 * count:3 * count + copies] = first + np.arange(copies)
    print("behind a whole first tile", where, flush=True)
    plan, stats = _fuse_with_common_direction(oracle, "behind " + where, src, groups, count, 4 * count)
    assert stats.fused == groups * copies * (2 if where == "nowhere" else 3)
    assert _layout(src, 4, count, groups, groups)[1][1] == [3]
    assert _marked(plan, groups, 64 + 3)
