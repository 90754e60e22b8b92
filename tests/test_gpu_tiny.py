"""A whole tree call in one launch (csrc/tiny.hip) at the edges of what it takes: sets of no and of one block, blocks of a few lanes
and of a lane's full share, pools larger than the table, many members per target, tables with errors.  Exactly the oracle's tables,
pools, counts, scales and norms."""
import numpy as np
import pytest
import torch

from paper_2601_03067_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _recipe(counts, t, d, dtype, bases, groups):
    """Leaves of the given sizes, one per unit; every block one of `bases` blocks with noise, or (0) a block of its own"""
    n = int(sum(counts))
    rng = np.random.default_rng(n * 31 + t * d)
    src = rng.integers(0, bases, n) if bases else np.full(n, -1)
    start = np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.int32)
    cnt = np.asarray(counts, np.int32)
    return wl.Recipe("tiny", 8, groups, 1, 1, t, d, dtype, 0.9, src.astype(np.int64), np.full(n, 0.03, np.float32),
                     max(bases, 1), start, cnt, cnt * t, start, cnt, np.arange(len(counts) + 1, dtype=np.int32))


# (leaf sizes, tokens per block, head size, dtype, bases, groups, unused blocks of the pool)
CASES = [([1, 1], 16, 64, torch.bfloat16, 1, 1, 0),                      # one pair
         ([0, 3, 0, 0, 5, 1], 16, 32, torch.float32, 3, 2, 3),           # empty sets on either side
         ([8, 8, 8, 8], 16, 64, torch.float32, 9, 2, 0),                 # a lane's full share in binary32 (two partial sums)
         ([6, 7, 5], 16, 128, torch.bfloat16, 4, 3, 5),                  # ... and in bfloat16: half the wavefronts
         ([9, 2, 13], 1, 64, torch.bfloat16, 5, 2, 1),                   # 8 lanes hold a block
         ([7, 4, 6], 16, 72, torch.bfloat16, 6, 2, 96),                  # a block that ends within a lane's share; the largest pool
         ([1] * 64, 4, 64, torch.float32, 7, 2, 64),                     # the most entries, six heights, up to ten members a target
         ([2] * 9 + [12], 16, 64, torch.bfloat16, 1, 300, 0),            # one target takes everything
         ([4, 8, 3], 16, 64, torch.float32, 0, 1, 0),                    # nothing fuses
         ([5], 16, 64, torch.bfloat16, 2, 1, 4),                         # no height
         ([8, 8, 8, 9], 16, 64, torch.float32, 9, 2, 0),                 # the most keys of 4096 bytes that stay in LDS ...
         ([8, 8, 8, 9], 16, 64, torch.float32, 9, 2, 1),                 # ... and one more
         ([11, 9, 13], 16, 128, torch.bfloat16, 7, 2, 0),                # the same in bfloat16
         ([11, 9, 13], 16, 128, torch.bfloat16, 7, 2, 1)]


def _inputs(rec, spare):
    mat = wl.materialise(rec, DEV, phys_perm=True)
    if spare:                                                           # blocks that no entry points at, among the others
        gen = torch.Generator(device=DEV)
        gen.manual_seed(3)
        P = rec.n + spare
        at = torch.stack([torch.randperm(P, generator=gen, device=DEV)[:rec.n] for _ in range(rec.G)])
        for name in ("K", "V"):
            big = torch.randn(rec.G, P, rec.r, generator=gen, device=DEV).to(rec.dtype)
            for g in range(rec.G):
                big[g][at[g]] = mat[name][g]
            mat[name] = big
        mat["bt"] = torch.stack([at[g][mat["bt"][g].long()] for g in range(rec.G)]).to(torch.int32).contiguous()
    if rec.n > 5:
        mat["K"][:, int(mat["bt"][0, 4])] = 0                           # a zero block, in one group an entry's
    return mat


def _left_behind(plan):
    """What the view of the last height promises after a call: sets, assignments, candidate counts, the diagnostic's zeros"""
    kb = gu.load_binding()
    c, v = plan.cache, plan.view(plan.n_heights - 1)
    get = lambda ptr, shape, dtype: kb.device_array(ptr, int(np.prod(shape)), dtype, DEV).reshape(shape)
    out = {"set_ids": get(v.set_ids, (c.G, c.n), np.int32), "set_cnt": get(v.set_cnt, (c.G, v.n_slots), np.int32),
           "cand_cnt": get(v.cand_cnt, (c.G, v.r_stride), np.int32), "best_packed": get(v.best_packed, (c.G, v.r_stride), np.uint64)}
    assign = get(v.assign, (c.G, v.r_stride), np.int32)
    r_slot, r_base = get(v.r_slot, (v.n_nodes,), np.int32), get(v.r_base, (v.n_nodes,), np.int32)
    out["assign"] = [assign[g, b:b + out["set_cnt"][g, s]].tolist() for g in range(c.G) for s, b in zip(r_slot, r_base)]
    return out


def _steps_behind(ctx, plan, thr):
    """The single steps of the last height once more, on what the call left"""
    kb = gu.load_binding()
    c, last = plan.cache, plan.n_heights - 1
    dense = torch.full((c.G, max(int(plan.view(last).total_s), 1)), -2.0, device=DEV)
    kb.similarity(ctx, plan, last, thr, dense_s=dense)
    kb.assign(ctx, plan, last, thr)
    left = _left_behind(plan)
    kb.merge(ctx, plan, last)
    torch.cuda.synchronize()
    return dense, left


def _same(left, want):
    for name in want:
        assert left[name] == want[name] if name == "assign" else np.array_equal(left[name], want[name]), name


@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_tree_matches_oracle(oracle, case):
    counts, t, d, dtype, bases, groups, spare = case
    print("tiny", case, flush=True)
    rec = _recipe(counts, t, d, dtype, bases, groups)
    mat = _inputs(rec, spare)
    host = gu.host_copy(mat)
    cache, plan, stats, ctx = gu.gpu_fuse(rec, mat)
    res = gu.oracle_fuse(oracle, rec, host)
    gu.check_ambiguity(res, str(case))
    for g, r in enumerate(res):
        gu.compare_group(r, cache, g, dtype == torch.float32, str(case))
    assert stats.fused == sum(int(r.stats[1]) for r in res) and stats.near_threshold == sum(int(r.stats[2]) for r in res)
    # launch by launch (stages are timed there) on the same inputs: the same bits, and the same counts of what the screen leaves open
    again = {"K": torch.from_numpy(np.stack(host[0]).view(np.int16 if dtype == torch.bfloat16 else np.float32)).to(DEV).view(dtype),
             "V": torch.from_numpy(np.stack(host[1]).view(np.int16 if dtype == torch.bfloat16 else np.float32)).to(DEV).view(dtype),
             "bt": torch.from_numpy(np.stack(host[2])).to(DEV)}
    other, staged, st, ctx2 = gu.gpu_fuse(rec, again, timing=True)
    assert st.ms_norms > 0 and st.ms_rewrite > 0 and stats.ms_total == 0
    for name in ("K", "V", "bt", "scale_k", "scale_v", "norm_k", "norm_v", "orig_norm_k", "orig_norm_v", "refcount", "remap", "n_free", "n_phys"):
        assert torch.equal(getattr(cache, name), getattr(other, name)), name
    for name in ("fused", "near_threshold", "refined", "cand_overflow", "merge_targets", "physical_blocks"):
        assert getattr(stats, name) == getattr(st, name), name
    if plan.n_heights:
        _same(_left_behind(plan), _left_behind(staged))
        print("single steps behind the call", flush=True)
        kb, before = gu.load_binding(), cache.K.clone()
        kb.merge(ctx, plan, plan.n_heights - 1)                         # no target waits for it
        assert torch.equal(cache.K, before)
        (dense, left), (dense2, want) = _steps_behind(ctx, plan, rec.thr), _steps_behind(ctx2, staged, rec.thr)
        assert torch.equal(dense, dense2)
        for name in ("set_ids", "set_cnt", "assign"):
            assert left[name] == want[name] if name == "assign" else np.array_equal(left[name], want[name]), name
        assert torch.equal(cache.K, other.K) and torch.equal(cache.V, other.V)


@pytest.mark.parametrize("fault,text", [("outside", "outside"), ("shared", "not injective"), ("range", "norm")])
def test_faulty_tables_are_reported(fault, text):
    rec = _recipe([3, 4], 16, 64, torch.float32, 3, 2)
    mat = _inputs(rec, 2)
    if fault == "outside":
        mat["bt"][1, 2] = rec.n + 2
    elif fault == "shared":
        mat["bt"][0, 1] = mat["bt"][0, 5]
    else:
        mat["K"][0, int(mat["bt"][0, 6])] *= 2.0 ** 60
    with pytest.raises(Exception, match=text):
        gu.gpu_fuse(rec, mat)
