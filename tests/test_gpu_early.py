"""Early rejection in the similarity step of a tree call (csrc/early.hip) against the oracle.  It is used from a product of
5e10 operations (binary32: a sixteenth of that) and rows of 2 KiB on, which takes more groups than the oracle has time for:
groups are independent, so two of them are compared exactly (tables, pools, counts, scales, norms)."""
import numpy as np
import pytest
import torch

from paper_2601_03067_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _case(which):
    """-> (recipe, offset that every key block of a group shares, candidate slots)"""
    bff = dict(t=16, d=64)                                   # 2 KiB rows: 32 slices
    if which == "white":                                     # a few pairs per tile stay open, sets ragged against the tiles
        return wl.llama8b_bff(n_req=9, tokens=16 * 150, layers=20, kv_heads=2, prefix_tokens=16 * 9, near_pool=60, **bff), 0.0, 16
    if which == "shared_direction":                          # unrelated cosines around 0.5: a longer part before the test
        return wl.llama8b_bff(n_req=6, tokens=16 * 220, layers=20, kv_heads=2, prefix_tokens=16 * 5, near_pool=60, **bff), 1.0, 16
    if which == "no_test":                                   # unrelated cosines around 0.85 against thr 0.9: full length
        return wl.llama8b_bff(n_req=6, tokens=16 * 220, layers=20, kv_heads=2, prefix_tokens=16 * 5, near_pool=60, **bff), 2.35, 64
    if which == "dense":                                     # most tiles hold more related pairs than are finished one by one
        return wl.zipf_bff(n_req=8, tokens=32 * 150, layers=12, kv_heads=2, pool=150, t=32, d=64, thr=0.9), 0.0, 64
    if which == "pair_list_full":                            # 2.4 open pairs per left block, the list holds 1.6: in the panel kernel
        return wl.llama8b_bff(n_req=2, tokens=16 * 1300, layers=8, kv_heads=2, prefix_tokens=0, near_pool=560, near_frac=1.0, **bff), 0.0, 64
    if which == "pair_list_full_long":                       # the same behind a test that comes too late for the panel kernel: in the ring kernel
        return wl.llama8b_bff(n_req=2, tokens=16 * 1300, layers=8, kv_heads=2, prefix_tokens=0, near_pool=560, near_frac=1.0, **bff), 1.3, 64
    if which == "f32":
        return wl.mixed(n_req=9, min_tokens=600, max_tokens=3000, chunk_tokens=512, layers=2, kv_heads=2, pool=64, dtype=torch.float32, seed=78, **bff), 0.0, 16
    raise AssertionError(which)


@pytest.mark.parametrize("rule", ["argmax", "first_row"])
@pytest.mark.parametrize("which", ["white", "shared_direction", "no_test", "dense", "pair_list_full", "pair_list_full_long", "f32"])
def test_tree_with_early_rejection_matches_oracle(oracle, which, rule):
    kb = gu.load_binding()
    rec, common, cap = _case(which)
    print("early", which, rule, "G", rec.G, "n", rec.n, "r", rec.r, flush=True)
    mat = wl.materialise(rec, DEV, phys_perm=True)
    if common:
        gen = torch.Generator(device=DEV)
        gen.manual_seed(5)
        for g in range(rec.G):
            mat["K"][g] = (mat["K"][g].float() + common * torch.randn(rec.r, generator=gen, device=DEV)).to(rec.dtype)
    pick = [0, rec.G - 1]
    host = ([wl.to_numpy_pool(mat["K"][g]) for g in pick], [wl.to_numpy_pool(mat["V"][g]) for g in pick],
            [mat["bt"][g].cpu().numpy().copy() for g in pick])
    alone = kb.Cache(mat["K"], mat["V"], mat["bt"], rec.t, rec.d)
    kb.block_norms(kb.Context(DEV), alone)
    torch.cuda.synchronize()
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat, cand_cap=cap, rule=rule)
    assert torch.equal(cache.orig_norm_k, alone.orig_norm_k)          # bit for bit: tails written or not
    res = gu.oracle_fuse(oracle, rec, host, rule=rule)
    gu.check_ambiguity(res, which)
    for r, g in zip(res, pick):
        gu.compare_group(r, cache, g, rec.dtype == torch.float32, which)
    # the path that the case is for was taken
    slices, open_pairs, room = kb.early_counts(ctx, plan)
    row = rec.r * mat["K"].element_size() // 64
    print("slices", sorted(set(slices.tolist())), "of", row, "open pairs", open_pairs.tolist(), "room", room, "fused", stats.fused, flush=True)
    assert room > 0
    if which == "no_test":                           # (the choice is a group's own: a few groups do test)
        assert np.mean(slices == row) > 0.8 and np.all(slices[pick] == row)
    else:
        assert np.all((slices >= 2) & (slices <= row * 3 // 4)) and open_pairs.any()
    if which == "shared_direction":
        assert np.median(slices) > row / 4           # unrelated white blocks need less at this threshold
    if which == "white":
        assert np.median(slices) < row / 4
    if which == "dense":
        assert open_pairs.sum() < stats.fused        # a pair that fused and was not left open comes from a tile at full length
    assert (open_pairs.max() > room) == which.startswith("pair_list_full")
    if which == "pair_list_full_long":
        assert np.all(slices > 11)                   # kPanelSlices
    per_group = kb.group_counters(ctx, plan)
    assert per_group[pick, 0].tolist() == [int(r.stats[1]) for r in res]
    assert per_group[pick, 1].tolist() == [int(r.stats[2]) for r in res]
    assert stats.fused > 0 and int(cache.refcount.sum()) == rec.G * rec.n and bool((cache.remap >= -1).all())
    if which != "no_test":
        assert np.all(per_group[:, 3] == 0)
