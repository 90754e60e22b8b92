"""Paged decode over bfloat16 pools, both products on the matrix cores: edges of the 16-token pieces, of the pairs a
wavefront takes and of the splits, every head count, against attention in binary64; the same inputs over all-head blocks,
which the vector-ALU kernel takes."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# every way a request can end inside, at and just past a piece, a pair of pieces, a round of four wavefronts, a split
CONTEXTS = [0, 1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 127, 128, 129, 255, 300, 1000]


def _setup(t, d, heads, seed, layers=2, all_heads=False, contexts=CONTEXTS, dtype=torch.bfloat16):
    from paper_2601_03067_amd import binding as kb
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    blocks = [(c + t - 1) // t for c in contexts]
    n, groups, width = sum(blocks), layers * (1 if all_heads else heads), d * (heads if all_heads else 1)
    P = n + 3
    K = torch.randn(groups, P, t * width, generator=gen, device=DEV).to(dtype)
    V = torch.randn(groups, P, t * width, generator=gen, device=DEV).to(dtype)
    bt = torch.randint(0, P, (groups, n), generator=gen, device=DEV, dtype=torch.int32)       # shared blocks among them
    cache = kb.Cache(K, V, bt, t, width)
    cache.scale_k.copy_(0.5 + torch.rand(groups, n, generator=gen, device=DEV))
    cache.scale_v.copy_(0.5 + torch.rand(groups, n, generator=gen, device=DEV))
    start = np.concatenate([[0], np.cumsum(blocks)[:-1]]).astype(np.int32)
    return kb, cache, start, max(blocks), gen


def _call(kb, cache, heads, q, start, max_blocks, all_heads, contexts=CONTEXTS):
    ctx = kb.Context(DEV)
    rs = torch.from_numpy(start).to(DEV)
    cl = torch.tensor(contexts, dtype=torch.int32, device=DEV)
    step = kb.paged_decode_attn_all_heads if all_heads else kb.paged_decode_attn
    out = step(ctx, cache, heads, q, rs, cl, max_blocks)
    torch.cuda.synchronize()
    return out.cpu().double()


def _reference(cache, t, d, heads, q, start, all_heads, contexts=CONTEXTS):
    layers, B, Hq, _ = q.shape
    rep = Hq // heads
    out = torch.zeros(q.shape, dtype=torch.float64)
    qc, K, V, bt = q.cpu().double(), cache.K.cpu().double(), cache.V.cpu().double(), cache.bt.cpu().long()
    sk, sv = cache.scale_k.cpu().double(), cache.scale_v.cpu().double()
    for li in range(layers):
        for h in range(heads):
            g, w, s = (li, heads, h) if all_heads else (li * heads + h, 1, 0)
            for b, c in enumerate(contexts):
                if c == 0:
                    continue
                x = slice(int(start[b]), int(start[b]) + (c + t - 1) // t)
                k = (K[g, bt[g, x]].view(-1, t, w, d)[:, :, s] * sk[g, x, None, None]).reshape(-1, d)[:c]
                v = (V[g, bt[g, x]].view(-1, t, w, d)[:, :, s] * sv[g, x, None, None]).reshape(-1, d)[:c]
                p = torch.softmax(qc[li, b, h * rep:(h + 1) * rep] @ k.T / d ** 0.5, -1)
                out[li, b, h * rep:(h + 1) * rep] = p @ v
    return out


@pytest.mark.parametrize("t,d,heads,rep,all_heads", [(16, 128, 2, 4, False), (16, 64, 3, 1, False), (32, 128, 2, 8, False),
                                                     (48, 64, 1, 3, False), (16, 128, 1, 16, False), (64, 128, 2, 7, False),
                                                     (16, 128, 2, 4, True), (32, 64, 4, 2, True), (48, 128, 2, 16, True)])
def test_against_binary64(t, d, heads, rep, all_heads):
    kb, cache, start, max_blocks, gen = _setup(t, d, heads, 7 * t + d + rep, all_heads=all_heads)
    q = torch.randn(2, len(CONTEXTS), heads * rep, d, generator=gen, device=DEV).to(torch.bfloat16)
    ref = _reference(cache, t, d, heads, q, start, all_heads)
    out = _call(kb, cache, heads, q, start, max_blocks, all_heads)
    # A logit of this input is at most 10 (|q| |k| / sqrt(d) = sqrt(d), times a scale below 1.5, and the largest of a thousand
    # normal draws at 4 of 1.5 standard deviations): its binary32 roundings move a weight by 10 * 3 * 2^-24 = 2e-6, and
    # outputs, sums of values below 6 with weights that add to one, by 1.2e-5 at most.
    assert float((out - ref).abs().max()) < 1.2e-5
    assert float(out[:, CONTEXTS.index(0)].abs().max()) == 0.0


@pytest.mark.parametrize("dtype,t", [(torch.bfloat16, 16), (torch.float32, 16), (torch.bfloat16, 32)])
@pytest.mark.parametrize("layers,heads,requests", [(1, 8, 1), (1, 8, 5), (2, 4, 3), (3, 3, 4), (11, 1, 2), (1, 2, 7), (4, 1, 6), (1, 1, 40),
                                                   (3, 5, 140), (11, 1, 100)])
def test_workgroups_dealt_out_to_the_xcds(layers, heads, requests, dtype, t):
    """Contexts from 1024 tokens on: every (layer, request, KV head, split) is done once, for whole eights of groups, what is left of
    them, one split of many requests, and two of more than 512 (layer, request, KV head) triples."""
    d = 64
    contexts = [1100 - 37 * b % 1090 for b in range(requests)]
    kb, cache, start, max_blocks, gen = _setup(t, d, heads, 3 + requests, layers, contexts=contexts, dtype=dtype)
    q = torch.randn(layers, requests, heads * 2, d, generator=gen, device=DEV).to(dtype)
    ref = _reference(cache, t, d, heads, q, start, False, contexts)
    out = _call(kb, cache, heads, q, start, max_blocks, False, contexts)
    assert float((out - ref).abs().max()) < 1.2e-5                         # the same bound as above


@pytest.mark.parametrize("layers,heads,requests", [(1, 8, 5), (2, 4, 260)])
def test_a_length_beyond_max_blocks_stays_inside(layers, heads, requests):
    """Lengths on the device that have outgrown max_blocks (several splits, and one): nothing behind the workspace is written, and the
    requests that max_blocks covers are what they are without the others."""
    t, d = 16, 64
    contexts = [1100 - 37 * b % 1090 for b in range(requests)]
    contexts[requests // 2] = contexts[-1] = 2500
    kb, cache, start, _, gen = _setup(t, d, heads, 17, layers, contexts=contexts)
    max_blocks = (1100 + t - 1) // t
    q = torch.randn(layers, requests, heads * 2, d, generator=gen, device=DEV).to(torch.bfloat16)
    nbytes = kb.decode_workspace_bytes(layers, requests, heads * 2, heads, d, max_blocks)
    ws = torch.full((nbytes + (1 << 20),), 0xA5, dtype=torch.uint8, device=DEV)
    rs, cl = torch.from_numpy(start).to(DEV), torch.tensor(contexts, dtype=torch.int32, device=DEV)
    out = kb.paged_decode_attn(kb.Context(DEV), cache, heads, q, rs, cl, max_blocks, workspace=ws)
    assert bool((ws[nbytes:] == 0xA5).all())
    covered = [b for b in range(requests) if contexts[b] <= 1100]
    ref = _reference(cache, t, d, heads, q, start, False, contexts)
    assert float((out.cpu().double() - ref)[:, covered].abs().max()) < 1.2e-5  # the bound of test_against_binary64


def test_rows_past_the_context_and_infinite_values():
    t, d, heads, rep = 32, 128, 2, 4
    kb, cache, start, max_blocks, gen = _setup(t, d, heads, 5)
    n = cache.bt.shape[1]
    cache.bt.copy_(torch.arange(n, dtype=torch.int32, device=DEV))         # one block each, so that tails can be spoilt
    q = torch.randn(2, len(CONTEXTS), heads * rep, d, generator=gen, device=DEV).to(torch.bfloat16)
    clean = _call(kb, cache, heads, q, start, max_blocks, False)
    K, V = cache.K.view(4, -1, t, d), cache.V.view(4, -1, t, d)
    for b, c in enumerate(CONTEXTS):
        if c % t:
            K[:, int(start[b]) + c // t, c % t:] = float("nan")
            V[:, int(start[b]) + c // t, c % t:] = float("nan")
    assert torch.equal(_call(kb, cache, heads, q, start, max_blocks, False), clean)
    # one infinite value inside a context: that column of that request is infinite for every head, all else is finite
    b = CONTEXTS.index(300)
    V[:, int(start[b]) + 3, 5, 77] = float("-inf")
    out = _call(kb, cache, heads, q, start, max_blocks, False)
    assert bool((out[:, b, :, 77] == float("-inf")).all())
    keep = torch.ones_like(out, dtype=torch.bool)
    keep[:, b, :, 77] = False
    assert float((out[keep] - clean[keep]).abs().max()) < 1.2e-5           # the same bound as above


def test_all_heads_result_is_kept():
    """Blocks over all heads whose scales do not belong to their rows: logits of several hundred, where binary32 leaves an
    entry open by 1e-5 and more.  The result is pinned to that of the vector-ALU kernel (golden/decode_all_heads.npy: this
    call, taken when that kernel was the only one), to the bounds that perf/cases.py states for the entry point."""
    from paper_2601_03067_amd import binding as kb
    t, d, heads, rep, ctx = 16, 64, 4, 2, [700, 37, 433]
    rng = np.random.default_rng(11)
    blocks = [(c + t - 1) // t for c in ctx]
    n = sum(blocks)

    def integers(most, *shape):
        return rng.integers(-most, most + 1, shape).astype(np.float32)

    def to_gpu(x):
        return torch.from_numpy(x).to(DEV).to(torch.bfloat16)

    # keys share a direction, so that many of the large logits of a row lie close together
    K = to_gpu((integers(112, 1, 1, t * heads * d) + integers(15, 1, n, t * heads * d)) / 32)
    V, q = to_gpu(integers(127, 1, n, t * heads * d) / 32), to_gpu(integers(127, 1, len(ctx), heads * rep, d) / 64)
    cache = kb.Cache(K, V, torch.from_numpy(rng.permutation(n).astype(np.int32)[None]).to(DEV), t, d * heads)
    fused = torch.from_numpy(rng.integers(0, 4, (1, n)) < 3).to(DEV)
    cache.scale_k.copy_(torch.where(fused, 45.0 + 0.125 * torch.arange(n, device=DEV), 1.0))
    cache.scale_v.copy_(torch.where(fused, 44.0 - 0.125 * torch.arange(n, device=DEV), 1.0))
    rs = torch.tensor([sum(blocks[:b]) for b in range(len(ctx))], dtype=torch.int32, device=DEV)
    cl = torch.tensor(ctx, dtype=torch.int32, device=DEV)
    out = kb.paged_decode_attn_all_heads(kb.Context(DEV), cache, heads, q, rs, cl, max(blocks)).cpu().numpy().astype(np.float64)
    ref = np.load(os.path.join(os.path.dirname(__file__), "golden", "decode_all_heads.npy")).astype(np.float64)
    size = np.maximum(np.abs(ref), np.sqrt((ref ** 2).mean()))
    assert float(np.linalg.norm(out - ref) / np.linalg.norm(ref)) <= 1.2e-6
    assert float((np.abs(out - ref) / size).max()) <= 8e-6


@pytest.mark.parametrize("step", ["paged", "static", "all_heads", "shared"])
def test_logits_of_minus_infinity(step):
    """A token with an infinite key element may give a logit of -inf: it has no weight, and the row is that of the others."""
    from paper_2601_03067_amd import binding as kb
    t, d, heads, rep = 16, 128, 2, 4
    all_heads = step == "all_heads"
    _, cache, start, max_blocks, gen = _setup(t, d, heads, 9, all_heads=all_heads)
    n = cache.bt.shape[1]
    cache.bt.copy_(torch.arange(n, dtype=torch.int32, device=DEV))
    b, other = CONTEXTS.index(1000), CONTEXTS.index(300)
    cache.bt[:, int(start[other]):int(start[other]) + 12] = cache.bt[:, int(start[b]):int(start[b]) + 12]     # shared by two
    cache.scale_k[:, ::3] = 1.0                                                # the scale of a block that was not fused
    cache.scale_v[:, ::3] = 1.0
    q = torch.randn(2, len(CONTEXTS), heads * rep, d, generator=gen, device=DEV).to(torch.bfloat16)
    q[..., 7] = q[..., 7].abs() + 0.5
    q[..., 90] = -q[..., 90].abs() - 0.5
    K = cache.K.view(cache.K.shape[0], -1, t, heads if all_heads else 1, d)
    K[:, ::2, 5, :, 7] = float("-inf")                                         # one token of every other block
    K[:, 1::5, 11, :, 90] = float("inf")                                       # q < 0 there
    ctx = kb.Context(DEV)
    rs, cl = torch.from_numpy(start).to(DEV), torch.tensor(CONTEXTS, dtype=torch.int32, device=DEV)
    if step == "shared":
        plan = kb.SharedDecodePlan(ctx, cache, heads, start, np.array(CONTEXTS, np.int32), heads * rep, min_cluster_blocks=1)
        assert plan.info.clusters > 0
        out = kb.paged_decode_attn_shared(ctx, cache, plan, q)
    elif step == "static":
        out = torch.empty(q.shape, dtype=torch.float32, device=DEV)
        kb.paged_decode_attn_static(ctx, cache, heads, q, rs, cl, max_blocks, out)
    else:
        out = (kb.paged_decode_attn_all_heads if all_heads else kb.paged_decode_attn)(ctx, cache, heads, q, rs, cl, max_blocks)
    ref = _reference(cache, t, d, heads, q, start, all_heads)
    assert bool(torch.isfinite(ref).all())
    assert float((out.cpu().double() - ref).abs().max()) < 1.2e-5              # the bound of test_against_binary64


@pytest.mark.parametrize("d,scale", [(128, 45.25), (64, 31.7), (128, 300.1)])
def test_weights_of_large_logits(d, scale):
    """Logits of several hundred: the scale's rounding, 2^-24 of it, would move a weight by 1e-5.  The queries pick single key
    elements, so that the products themselves are exact and the weights alone are tested."""
    t, heads, rep = 16, 2, 4
    kb, cache, start, max_blocks, gen = _setup(t, d, heads, 3 * d)
    q = torch.zeros(2, len(CONTEXTS), heads * rep, d, device=DEV)
    q.scatter_(-1, torch.randint(0, d, q.shape[:-1] + (1,), generator=gen, device=DEV), 1.0)
    # logits up to 255 / 16 * scale / sqrt(d), in steps that leave several tokens with a share of the weight
    cache.K.copy_(240 / 16 + torch.randint(0, 16, cache.K.shape, generator=gen, device=DEV) / 16)
    cache.scale_k.copy_(scale * (1.0 + torch.rand(cache.scale_k.shape, generator=gen, device=DEV) / 512))
    q = q.to(torch.bfloat16)
    # against the library's own softmax scale, a binary32
    ref = _reference(cache, t, d, heads, q.double() * (float(np.float32(1.0 / d ** 0.5)) * d ** 0.5), start, False)
    out = _call(kb, cache, heads, q, start, max_blocks, False)
    # Two roundings of the exponent's argument x move a weight 2^-x by x 2^-x ln 2 * 2^-23 <= 0.37 * 2^-23 of the largest
    # one, exp2, the sums of weights and of products and the division by a unit (2^-24) each: below 5 units of the values.
    assert float((out - ref).abs().max()) < 5 * 2.0 ** -24 * float(cache.V.float().abs().max())


# longest contexts of one and of two steps (workgroups of one and two wavefronts), and one token more
@pytest.mark.parametrize("t,d,rep,longest", [(16, 128, 1, 16), (16, 128, 4, 32), (32, 64, 16, 32), (16, 64, 2, 33), (48, 128, 3, 48),
                                             (16, 128, 8, 64), (64, 64, 4, 64), (16, 128, 4, 65)])
def test_short_contexts(t, d, rep, longest):
    heads, contexts = 2, [0, 1, 15, longest // 2, longest - 1, longest]
    kb, cache, start, max_blocks, gen = _setup(t, d, heads, t + longest, contexts=contexts)
    cache.bt.copy_(torch.arange(cache.bt.shape[1], dtype=torch.int32, device=DEV))
    V = cache.V.view(cache.V.shape[0], -1, t, d)
    q = torch.randn(2, len(contexts), heads * rep, d, generator=gen, device=DEV).to(torch.bfloat16)
    ref = _reference(cache, t, d, heads, q, start, False, contexts)
    out = _call(kb, cache, heads, q, start, max_blocks, False, contexts)
    assert float((out - ref).abs().max()) < 1.2e-5               # the bound of test_against_binary64
    # an infinite value: that column of that request, and no other
    b = len(contexts) - 1
    V[:, int(start[b]) + (longest - 1) // t, (longest - 1) % t, 3] = float("inf")
    spoilt = _call(kb, cache, heads, q, start, max_blocks, False, contexts)
    assert bool((spoilt[:, b, :, 3] == float("inf")).all())
    spoilt[:, b, :, 3] = out[:, b, :, 3]
    assert float((spoilt - out).abs().max()) < 1.2e-5


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,heads,rep,B", [(128, 8, 1, 32), (64, 8, 3, 33), (128, 8, 16, 32), (64, 16, 4, 31)])
def test_two_splits_of_many_requests(d, heads, rep, B, dtype):
    """Two splits each, 512 (layer, request, KV head) triples and a few more or fewer: both merges of the splits' states."""
    from paper_2601_03067_amd import binding as kb
    t, layers = 16, 2
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B + rep)
    contexts = [(37 * b) % 209 for b in range(B - 1)] + [208]             # 13 blocks: two splits of 7
    blocks = [(c + t - 1) // t for c in contexts]
    n = sum(blocks)
    K = torch.randn(layers * heads, n, t * d, generator=gen, device=DEV).to(dtype)
    V = torch.randn(layers * heads, n, t * d, generator=gen, device=DEV).to(dtype)
    bt = torch.randperm(n, generator=gen, device=DEV).to(torch.int32).repeat(layers * heads, 1).contiguous()
    cache = kb.Cache(K, V, bt, t, d)
    cache.scale_k.copy_(0.5 + torch.rand(bt.shape, generator=gen, device=DEV))
    cache.scale_v.copy_(0.5 + torch.rand(bt.shape, generator=gen, device=DEV))
    q = torch.randn(layers, B, heads * rep, d, generator=gen, device=DEV).to(dtype)
    start = np.concatenate([[0], np.cumsum(blocks)[:-1]]).astype(np.int32)
    out = _call(kb, cache, heads, q, start, max(blocks), False, contexts)
    ref = _reference(cache, t, d, heads, q, start, False, contexts)
    assert float((out - ref).abs().max()) < 1.2e-5                        # the bound of test_against_binary64
