"""Chunked prefill: the kernel for few queries, whose wavefronts share the context out among them, and the staged kernel for
many, on either side of the line between them, at ragged query counts and contexts, against attention in binary64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _reference(cache, t, d, heads, layers, q, q_begin, sm_scale=None):
    _, nq, Hq, _ = q.shape
    rep, ctx = Hq // heads, q_begin + nq
    out = torch.empty(q.shape, dtype=torch.float64, device=DEV)
    nb = (ctx + t - 1) // t
    hidden = torch.arange(ctx, device=DEV)[None, :] > torch.arange(q_begin, ctx, device=DEV)[:, None]
    for g in range(layers * heads):
        li, h = divmod(g, heads)
        x = cache.bt[g, :nb].long()
        k = (cache.K[g][x].double().view(nb, t, d) * cache.scale_k[g, :nb, None, None].double()).reshape(-1, d)[:ctx]
        v = (cache.V[g][x].double().view(nb, t, d) * cache.scale_v[g, :nb, None, None].double()).reshape(-1, d)[:ctx]
        for j in range(h * rep, (h + 1) * rep):
            z = (q[li, :, j].double() @ k.T) * (d ** -0.5 if sm_scale is None else sm_scale)
            out[li, :, j] = torch.softmax(z.masked_fill(hidden, float("-inf")), -1) @ v
    return out


# (layers, heads, rep, t, d, chunk begin, first query after it, queries); staged kernel's workgroups in the comment
CASES = [(1, 1, 1, 16, 64, 0, 0, 1),             # one token, nothing before it
         (1, 2, 4, 16, 128, 0, 0, 33),           # the chunk only: 31 rows of one piece, then one more
         (1, 2, 4, 16, 128, 32, 3, 5),           # 2 blocks before the chunk: fewer tiles than wavefronts
         (2, 1, 16, 48, 64, 48 * 9, 17, 2),      # three pieces per block, two positions per workgroup
         (1, 3, 3, 32, 128, 1024, 0, 100),       # heads padded from 3 to 4
         (3, 8, 4, 16, 128, 512, 0, 256),        # 192, three rounds of split workgroups: the context is too short for them
         (3, 8, 4, 16, 128, 512, 0, 257),        # 216: the staged kernel, one row in its last workgroup
         (4, 8, 16, 32, 64, 96, 31, 57),         # 256, staged
         (3, 8, 4, 16, 128, 2048, 0, 256),       # 192: the last grid of the split kernel, a context long enough with or without reuse
         (4, 8, 4, 16, 128, 160, 5, 128),        # 128, two rounds: staged with reuse, split without
         (4, 8, 4, 16, 64, 160, 5, 128)]         # the same heads of 64 elements: one round, split


def _compare(case, reuse, sm_scale=None, signed_scales=False):
    from paper_2601_03067_amd import binding as kb
    layers, heads, rep, t, d, begin, skip, nq = case
    print("prefill", case, "reuse", reuse, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11 + nq)
    q_begin, groups = begin + skip, layers * heads
    n = (q_begin + nq + t - 1) // t
    P = n + 2
    K = torch.randn(groups, P, t * d, generator=gen, device=DEV).to(torch.bfloat16)
    V = torch.randn(groups, P, t * d, generator=gen, device=DEV).to(torch.bfloat16)
    # blocks before the chunk share stored blocks (up to about four to one), those of the chunk are their own
    bt = torch.arange(n, device=DEV, dtype=torch.int32).repeat(groups, 1)
    if begin:
        bt[:, :begin // t] = torch.randint(0, max(1, begin // t // 2), (groups, begin // t), generator=gen, device=DEV, dtype=torch.int32)
    tail = (q_begin + nq) % t
    if tail:                                     # rows after the last query may hold anything
        K.view(groups, P, t, d)[:, n - 1, tail:] = float("nan")
        V.view(groups, P, t, d)[:, n - 1, tail:] = float("nan")
    cache = kb.Cache(K, V, bt.contiguous(), t, d)
    cache.scale_k.copy_(0.5 + torch.rand(groups, n, generator=gen, device=DEV))
    cache.scale_v.copy_(0.5 + torch.rand(groups, n, generator=gen, device=DEV))
    if signed_scales:
        cache.scale_k[:, ::3] *= -1.0
    ctx = kb.Context(DEV)
    q = torch.randn(layers, nq, heads * rep, d, generator=gen, device=DEV).to(torch.bfloat16)
    plan = kb.PrefillPlan(ctx, cache, heads, heads * rep, 0, begin, q_begin, q_begin + nq, reuse=reuse)
    out = kb.prefill_attn(ctx, cache, plan, q, sm_scale=sm_scale)
    ref = _reference(cache, t, d, heads, layers, q, q_begin, sm_scale)
    # The weights are kept as a bfloat16 head and remainder, 2^-17 of their size at most (half a unit of the ninth bit of the
    # ninth), and values are below 1.5 * 6: 7e-5 for a row that is a single weight, on top of 1.2e-5 of binary32 roundings of
    # logits below 15.
    err = float((out.double() - ref).abs().max())
    assert err < 8.2e-5, err


@pytest.mark.parametrize("reuse", [True, False])
@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_against_binary64(case, reuse):
    _compare(case, reuse)


@pytest.mark.parametrize("sm_scale", [-0.1, 0.0])
@pytest.mark.parametrize("signed_scales", [False, True])
@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_softmax_scale_of_either_sign(case, signed_scales, sm_scale):
    """Logits times a scale that is not positive: the largest ones are then the smallest products (of either sign, with scales
    of either sign); rows that see nothing of a tile are among them.  Logits stay below those of the test above."""
    _compare(case, True, sm_scale=sm_scale, signed_scales=signed_scales)


# Grids of the staged kernel beyond two workgroups per compute unit, head size 128, where its registers are for three wavefronts per
# SIMD; the last one is on the other side of that line.
STAGED = [(18, 8, 4, 16, 128, 64, 5, 129),       # 720: a workgroup of one position, six rows of the last piece hidden
          (21, 8, 1, 32, 128, 0, 0, 513),        # 840: nothing before the chunk, both pieces of the last tile
          (9, 8, 16, 48, 128, 96, 7, 65),        # 648: three pieces per block, two positions per wavefront
          (18, 8, 4, 16, 128, 16, 1, 100)]       # 576, most of it the chunk itself


@pytest.mark.parametrize("reuse", [True, False])
@pytest.mark.parametrize("case", STAGED, ids=[str(i) for i in range(len(STAGED))])
def test_large_grids_against_binary64(case, reuse):
    _compare(case, reuse)


# Walks of one to four tiles in the staged kernel with room for two tiles on their way (193 to 512 workgroups): fewer than are asked for
# before the first is multiplied, as many, one and two more.
SHORT = [(28, 8, 4, 16, 128, 0, 0, 1),           # 224 workgroups, half a tile
         (28, 8, 4, 16, 128, 0, 0, 32),          # one
         (28, 8, 4, 16, 128, 0, 9, 33),          # 448; one and a half, two of the last piece's rows hidden
         (28, 8, 4, 16, 128, 32, 3, 45),         # up to two and a half
         (21, 8, 2, 16, 128, 0, 44, 65)]         # 336; four, a workgroup of one position


@pytest.mark.parametrize("reuse", [True, False])
@pytest.mark.parametrize("case", SHORT, ids=[str(i) for i in range(len(SHORT))])
def test_short_walks_against_binary64(case, reuse):
    _compare(case, reuse)


# Groups of (layer, KV head) in whole eights and some left over, or fewer than eight, dealt out to the XCDs; either kernel
GROUPS = [(11, 1, 4, 16, 128, 512, 0, 700),      # 242 workgroups of the staged kernel
          (5, 5, 1, 16, 128, 160, 7, 900),       # 200
          (13, 1, 4, 16, 64, 96, 0, 600),        # 247
          (3, 1, 16, 32, 64, 64, 3, 600),        # 225 of three groups
          (3, 5, 4, 16, 64, 256, 5, 40),         # split
          (19, 1, 2, 16, 128, 2048, 0, 20),
          (7, 1, 8, 48, 128, 96, 1, 30)]


@pytest.mark.parametrize("reuse", [True, False])
@pytest.mark.parametrize("case", GROUPS, ids=[str(i) for i in range(len(GROUPS))])
def test_groups_dealt_out_to_the_xcds(case, reuse):
    _compare(case, reuse)
