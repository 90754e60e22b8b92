"""Shared-block decode: blocks of one to four pieces, tails that leave whole pieces empty, more partial
states per request than a wavefront has lanes, padded head counts, against attention in binary64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (block size, head dim, KV heads, query heads per KV head, least blocks of a cluster, blocks of the longest request, layers);
# from 4096 query heads on the partial states are merged by a wavefront per head, 8 states at a time in rounds of 64; plans of
# little more than one state per request have a merge of their own (the cases with 1 or 2 blocks, and those without clusters)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("t,d,heads,rep,least,blocks,layers",
                         [(16, 128, 2, 4, 1, 75, 2), (16, 64, 1, 1, 1, 70, 2), (32, 128, 1, 8, 2, 20, 2), (48, 64, 2, 3, 1, 9, 2),
                          (64, 128, 1, 16, 1, 7, 2), (16, 128, 1, 2, 4, 1, 300), (16, 128, 2, 4, 1, 75, 57), (16, 64, 1, 16, 1, 75, 29),
                          (16, 128, 1, 16, 1, 20, 29), (32, 64, 2, 3, 1, 37, 76),
                          (16, 64, 2, 4, 1, 2, 2), (16, 128, 1, 2, 9, 4, 2), (64, 64, 1, 4, 1, 1, 2), (16, 128, 2, 5, 9, 5, 2)])
def test_against_binary64(t, d, heads, rep, least, blocks, layers, dtype):
    from paper_2601_03067_amd import binding as kb
    print("shared decode", t, d, heads, rep, least, blocks, layers, dtype, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(t + d + blocks)
    B, groups = 9, layers * heads
    # request b takes stored block j in the set j if bit b of j is set (request 0: of all), so that the sets of requests that
    # share a block differ from block to block; every other block is its own
    ids, nxt = [], 2 * blocks
    for b in range(B):
        mine = []
        for j in range(blocks):
            if b == 0 or (j >> (b - 1)) & 1:
                mine.append(j)
            elif j % 3 == 0:
                mine.append(nxt)
                nxt += 1
        ids.append(mine)
    ids[B - 1] = []                                                              # an empty request
    ctx_len = np.array([max(0, len(m) * t - (5 * i + (t - 3 if i == 2 else 0)) % t) for i, m in enumerate(ids)], np.int32)
    start = np.concatenate([[0], np.cumsum([len(m) for m in ids])[:-1]]).astype(np.int32)
    bt = torch.tensor(sum(ids, []), dtype=torch.int32, device=DEV).repeat(groups, 1).contiguous()
    n, P = bt.shape[1], nxt
    K = torch.randn(groups, P, t * d, generator=gen, device=DEV).to(dtype)
    V = torch.randn(groups, P, t * d, generator=gen, device=DEV).to(dtype)
    cache = kb.Cache(K, V, bt, t, d)
    cache.scale_k.copy_(0.5 + torch.rand(groups, n, generator=gen, device=DEV))
    cache.scale_v.copy_(0.5 + torch.rand(groups, n, generator=gen, device=DEV))
    q = torch.randn(layers, B, heads * rep, d, generator=gen, device=DEV).to(dtype)
    ctx = kb.Context(DEV)
    plan = kb.SharedDecodePlan(ctx, cache, heads, start, ctx_len, heads * rep, min_cluster_blocks=least)
    out = kb.paged_decode_attn_shared(ctx, cache, plan, q)
    torch.cuda.synchronize()
    assert B * heads * rep * layers >= 4096 or layers == 2                        # (the last four: items of one and two steps, and one piece more)
    if blocks == 75:
        assert plan.info.clusters > 64 * groups                                  # request 0 is in all: more slots than lanes,
    elif layers > 2 and blocks > 1:
        assert 8 * groups < plan.info.clusters < 56 * groups                     # or more than one read of 8 in a round
    ref = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    for g in range(groups):
        li, h = divmod(g, heads)
        for b in range(B):
            c = int(ctx_len[b])
            if c == 0:
                continue
            x = slice(int(start[b]), int(start[b]) + (c + t - 1) // t)
            p = bt[g, x].long()
            k = (K[g][p].double().view(-1, t, d) * cache.scale_k[g, x, None, None].double()).reshape(-1, d)[:c]
            v = (V[g][p].double().view(-1, t, d) * cache.scale_v[g, x, None, None].double()).reshape(-1, d)[:c]
            hs = slice(h * rep, (h + 1) * rep)
            ref[li, b, hs] = torch.softmax((q[li, b, hs].double() @ k.T) / d ** 0.5, -1) @ v
    # as for the paged kernel: binary32 roundings of logits below 10 move an output, values below 6, by 1.2e-5 at most
    assert float((out.double() - ref).abs().max()) < 1.2e-5
