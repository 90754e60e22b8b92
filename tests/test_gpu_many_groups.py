"""More nodes, groups or requests than the widest workgroups of a kernel have launches for (a launch has fewer than 2^32 threads
along one axis): the narrower variants take over, and the results are those that the inputs were made for."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
R = 64                                # the shortest blocks: 128 bytes


def _fuse(G, leaves):
    """G groups of sum(leaves) blocks.  Every second block is an exact copy of the one before it, all others point their own
    way; -> the fused cache and the statistics."""
    from paper_2601_03067_amd import binding as kb
    n = sum(leaves)
    print("groups", G, "leaves", len(leaves), "blocks", n, flush=True)
    # one-hot blocks with signs: block pair m of a group is +-e_(m mod R) on top of a length of its own, so that pairs of
    # different m are orthogonal, opposite, or (beyond 2 R pairs) the same direction
    m = torch.arange(n, device=DEV) // 2
    K1 = torch.zeros(n, R, device=DEV, dtype=torch.bfloat16)
    K1[torch.arange(n, device=DEV), m % R] = torch.where((m // R) % 2 == 0, 1.0, -1.0).to(torch.bfloat16)
    K = K1.repeat(G, 1, 1).view(G, n, R)
    bt = torch.arange(n, device=DEV, dtype=torch.int32).repeat(G, 1)
    ctx = kb.Context(DEV)
    cache = kb.Cache(K, K.clone(), bt, 1, R)
    start = np.concatenate([[0], np.cumsum(leaves)[:-1]]).astype(np.int32)
    plan = kb.Plan(ctx, cache, kb.tree_spec(start, np.array(leaves, np.int32), np.arange(len(leaves) + 1, dtype=np.int32)), cand_cap=16)
    stats = kb.fuse_tree(ctx, plan, 0.9)
    torch.cuda.synchronize()
    return cache, stats


def _kept(leaves):
    """Blocks that survive in a group: a right block fuses where the left set holds its direction."""
    n = sum(leaves)
    way = (np.arange(n) // 2) % (2 * R)

    def over(sets):
        if len(sets) == 1:
            return sets[0]
        a, b = over(sets[:len(sets) // 2]), over(sets[len(sets) // 2:])
        return np.concatenate([a, b[~np.isin(b, a)]])

    return len(over(np.split(way, np.cumsum(leaves)[:-1])))


def _check(cache, stats, leaves):
    G, n = cache.bt.shape
    kept = _kept(leaves)
    assert stats.physical_blocks == G * kept and stats.fused == G * (n - kept)
    for x in (cache.bt, cache.refcount, cache.scale_k, cache.remap):
        assert bool((x == x[0]).all())
    assert bool((cache.n_phys == kept).all()) and bool((cache.n_free == n - kept).all())
    assert bool((cache.free_list[:, :n - kept] == cache.free_list[0, :n - kept]).all())
    # every block still points its own way, with its own length
    m = torch.arange(n, device=DEV) // 2
    own = cache.K.view(G, n, R)[0][cache.bt[0].long(), m % R].float() * cache.scale_k[0]
    assert torch.equal(own, torch.where((m // R) % 2 == 0, 1.0, -1.0))


def test_more_one_tile_nodes_than_wide_workgroups():
    """8 392 704 nodes of one 32 x 32 tile: 512 threads each would be more than a launch has."""
    leaves = [1] * 4098
    _check(*_fuse(4096, leaves), leaves)


def test_more_large_nodes_than_the_widest_bookkeeping():
    """4 196 352 nodes, one in 2049 of them with a set too large for LDS: 1024 threads each would be more than a launch has."""
    leaves = [1100] + [1] * 4097
    _check(*_fuse(2048, leaves), leaves)


def test_more_groups_than_the_widest_lists():
    """4 194 400 groups of two blocks: the free lists of the table rewrite have more threads than a launch holds with 1024 a group,
    and more workgroups of 256 than it takes at once."""
    leaves = [1, 1]
    _check(*_fuse(4194400, leaves), leaves)


def test_shared_decode_of_more_heads_than_merging_wavefronts():
    """67 110 400 query heads: the merge with a wavefront each would take more threads than a launch has."""
    from paper_2601_03067_amd import binding as kb
    B, rep, t, d, shared, rest = 4194400, 16, 16, 64, 4, 5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(4)
    K = torch.randn(1, shared + 2, t * d, generator=gen, device=DEV).to(torch.bfloat16)
    V = torch.randn(1, shared + 2, t * d, generator=gen, device=DEV).to(torch.bfloat16)
    cache = kb.Cache(K, V, torch.arange(shared + 2, device=DEV, dtype=torch.int32)[None].contiguous(), t, d)
    cache.identity_scales()
    # three in ten requests have the shared blocks and five tokens more (two partial states), the others five tokens
    ctx_len = np.where(np.arange(B) % 10 < 3, shared * t + rest, rest).astype(np.int32)
    start = np.where(ctx_len == rest, shared + 1, 0).astype(np.int32)
    ctx = kb.Context(DEV)
    plan = kb.SharedDecodePlan(ctx, cache, 1, start, ctx_len, rep, min_cluster_blocks=shared)
    assert 4 * (plan.info.items_cluster + plan.info.items_residual) > 5 * B
    print("plan built", flush=True)
    q = torch.randn(1, B, rep, d, generator=gen, device=DEV, dtype=torch.bfloat16)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device=DEV)
    kb.paged_decode_attn_shared(ctx, cache, plan, q, out=out)
    for c in (shared * t + rest, rest):
        pick = torch.from_numpy(np.nonzero(ctx_len == c)[0][::997]).to(DEV)
        first = 0 if c > rest else (shared + 1) * t
        k, v = K.view(-1, d)[first:first + c].double(), V.view(-1, d)[first:first + c].double()
        ref = torch.softmax(q[0, pick].double() @ k.T / d ** 0.5, -1) @ v
        # logits below 15, values below 6: as in test_gpu_decode_bf16.py
        assert float((out[0, pick].double() - ref).abs().max()) < 1.2e-5
    assert bool(torch.isfinite(out).all())
