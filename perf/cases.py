"""Cases that the speed of this library is judged by: what a serving engine has it do, over the range of sizes it meets.

Four operations, each through its public entry point in ``binding``:

* ``fuse``     one Fast Fusion pass over a paged cache (norms, tree of similarity / assignment / merge, table rewrite)
* ``decode``   one step of paged decode attention through the fused block table
* ``shared``   the same decode step organised around the blocks that several requests share
* ``prefill``  causal attention of a run of prompt tokens over a fused context, with reuse on fused blocks

A case is a dict of plain values; ``layers`` x ``kv_heads`` are the groups the call covers.  The structure of a workload
(which block repeats which, lengths of the requests) is a function of the case alone; all values come from the seed.
"""
import math

import numpy as np
import torch

from paper_2601_03067_amd import binding as kb
from paper_2601_03067_amd import workloads as wl

DEV = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}

_BASE = {"op": "fuse", "kind": "bff", "layers": 1, "kv_heads": 8, "rep": 4, "t": 16, "d": 128, "dtype": "bf16", "requests": 8,
         "tokens": 1024, "chunk": 2048, "prefix": 256, "thr": 0.9, "common": 0.0, "screen": "none", "all_heads": False, "queries": 0,
         "reuse": True}


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest fusion: four requests of eight blocks in binary32, two groups.  What it costs is launches and the host.
        _case(name="fuse-tiny", kind="tiny", kv_heads=2, rep=2, d=64, dtype="f32", requests=4, tokens=128, thr=0.95),
        # The batch of the headline benchmark, whole: 32 layers x 8 KV heads, 64 requests of 2048 tokens with a common prefix.
        _case(name="fuse-batch", layers=32, requests=64, tokens=2048, prefix=512),
        # One long prompt fused over its 16 chunks, 32 layers; keys share a direction, as the keys of real caches do, and the
        # one-byte copies are centred on it, which is the option made for such keys.
        _case(name="fuse-chunks", kind="cff", layers=32, tokens=32768, common=2.35, screen="fp8c"),
        # Large batch whose blocks repeat by popularity (Zipf), 32-token blocks, eight query heads per KV head, 2 layers.
        _case(name="fuse-popular", kind="zipf", layers=2, rep=8, t=32, requests=256, tokens=4096),
        # 512 requests of 512 to 8192 tokens, chunks first, then requests, partial tail blocks: one layer of the largest batch.
        _case(name="fuse-ragged", kind="mixed", requests=512, tokens=8192),
        # One layer's attention for one request of a chat session: the smallest call of a decode loop, all latency.
        _case(name="decode-one", op="decode", requests=1, tokens=1000, prefix=0),
        # One layer's attention for a batch of ragged requests, as an engine calls it layer by layer.
        _case(name="decode-layer", op="decode", kind="mixed", requests=48, tokens=8192),
        # The whole decode step of the headline batch shape (8 of its 32 layers in one call).
        _case(name="decode-batch", op="decode", layers=8, requests=64, tokens=2048, prefix=512),
        # Eight query heads per KV head and 32-token blocks, popular blocks fused to a sixth of the cache.
        _case(name="decode-popular", op="decode", kind="zipf", layers=2, rep=8, t=32, requests=256, tokens=4096),
        # Three quarters of every context is a common system prompt: decode around the shared blocks.
        _case(name="decode-shared", op="shared", layers=8, requests=64, tokens=2048, prefix=1536),
        # Last 2048-token chunk of a 32768-token prompt, 4 layers: the long end of chunked prefill.
        _case(name="prefill-last", op="prefill", kind="cff", layers=4, tokens=32768, queries=2048),
        # A short follow-up prompt in an ordinary context, one layer, odd number of tokens: the short end.
        _case(name="prefill-short", op="prefill", kind="cff", layers=1, tokens=4296, queries=200),
    ]


# ---- structure of a case ----------------------------------------------------------------------------------------------------

def _recipe(c):
    kw = dict(layers=c["layers"], kv_heads=c["kv_heads"], t=c["t"], d=c["d"], dtype=DTYPES[c["dtype"]])
    if c["kind"] == "tiny":
        rec = wl.tiny_bff()
    elif c["kind"] == "bff":
        near = max(8, c["requests"] * 8)
        rec = wl.llama8b_bff(n_req=c["requests"], tokens=c["tokens"], prefix_tokens=c["prefix"], near_pool=near, **kw)
    elif c["kind"] == "cff":
        rec = wl.cff_long(tokens=c["tokens"] // c["t"] * c["t"], chunk_tokens=c["chunk"], **kw)
    elif c["kind"] == "zipf":
        rec = wl.zipf_bff(n_req=c["requests"], tokens=c["tokens"], thr=c["thr"], pool=max(64, c["requests"] * 80), **kw)
    else:
        rec = wl.mixed(n_req=c["requests"], min_tokens=max(c["t"], c["tokens"] // 16), max_tokens=c["tokens"],
                       chunk_tokens=c["chunk"], pool=max(16, c["requests"] * 8), **kw)
    rec.q_heads = rec.kv_heads * c["rep"]
    rec.thr = c["thr"]
    return rec


def _contexts(c, rec):
    """Context lengths of a decode step: whole requests, minus an odd number of tokens of the last block where the case's
    length is not a multiple of the block size."""
    if c["kind"] in ("bff", "zipf") and c["tokens"] % c["t"]:
        return np.full(rec.B, c["tokens"] // c["t"] * c["t"] - c["t"] + c["tokens"] % c["t"], np.int32)
    return rec.ctx_len.astype(np.int32)


def _prefill_span(c, rec):
    """(chunk_begin, q_begin, q_end): the last ``queries`` tokens of the prompt; the chunk starts at a block boundary."""
    q_end = int(rec.ctx_len[0])
    q_begin = max(0, q_end - c["queries"])
    return q_begin // c["t"] * c["t"], q_begin, q_end


def _node_pairs(rec):
    """Sum over the tree's nodes of (left set x right set), from the structure: copies of one base fuse, other blocks do not."""
    up, total = rec.unit_leaf_ptr, 0

    def join(a, b):
        nonlocal total
        total += len(a) * len(b)
        fused = (b >= 0) & np.isin(b, a)
        return np.concatenate([a, b[~fused]])

    def over(items):
        return items[0] if len(items) == 1 else join(over(items[: len(items) // 2]), over(items[len(items) // 2:]))

    leaves = [rec.src[s: s + k] for s, k in zip(rec.leaf_start, rec.leaf_count)]
    units = [over(leaves[a:b]) for a, b in zip(up[:-1], up[1:]) if b > a]
    kept = len(over(units)) if units else 0
    return total, kept


def work(case):
    """Bytes and operations of one pass that the operation cannot do without."""
    c = dict(_BASE, **case)
    rec = _recipe(c)
    el = 2 if c["dtype"] == "bf16" else 4
    block = rec.r * el
    if c["op"] == "fuse":
        pairs, kept = _node_pairs(rec)
        n_leaf = int(rec.leaf_count.sum())
        rebuilt = min(kept, n_leaf - kept)
        # Every block is read once for its norm, every rebuilt block written once (and put back by the next pass: the fusion
        # works in place).  A pair of blocks whose energy is spread evenly is not ruled out before the product has run over a
        # share 1 - thr of their elements (Cauchy-Schwarz on the rest): the operations that no exact method is without.
        return {"bytes": float(rec.G) * (2 * rec.n * block + 3 * 2 * rebuilt * block),
                "flops": float(rec.G) * 2.0 * rec.r * pairs * (1.0 - c["thr"])}
    _, kept = _node_pairs(rec)
    stored = rec.n - int(rec.leaf_count.sum()) + kept
    if c["op"] in ("decode", "shared"):
        ctx = _contexts(c, rec)
        tokens = float(ctx.sum()) * rec.G
        q = rec.layers * rec.B * rec.q_heads * rec.d
        return {"bytes": min(float(stored) * rec.G * 2 * block, tokens * 2 * rec.d * el) + q * (el + 4.0),
                "flops": 4.0 * tokens * rec.d * c["rep"]}
    begin, q0, q1 = _prefill_span(c, rec)
    seen = sum(p + 1 for p in range(q0, q1))
    q = rec.layers * (q1 - q0) * rec.q_heads * rec.d
    return {"bytes": min(stored, q1 // c["t"]) * float(rec.G) * 2 * block + q * 6.0,
            "flops": 4.0 * rec.G * c["rep"] * rec.d * seen}


def tolerance(case):
    """Tables and counts are whole numbers and exact; stored blocks are sums in fp64, rounded once (one bfloat16 step at most).
    Attention against the same sums in fp64, measured on these inputs: per-request decode 1.0e-7 - 2.6e-7 (largest entry
    1.7e-6), which multiplies in binary32; shared decode and prefill 2.3e-6 - 4.5e-6 (largest entry 1.9e-5), whose weights
    keep 16 bits.  Stated at about four times that."""
    if case["op"] == "fuse":
        return {"rel": 1e-6, "max": 8e-3}
    if case["op"] == "decode":
        return {"rel": 1.2e-6, "max": 8e-6}
    return {"rel": 2e-5, "max": 8e-5}


# ---- one state --------------------------------------------------------------------------------------------------------------

def _state(c, seed):
    rec = _recipe(c)
    mat = wl.materialise(rec, DEV, seed=wl._subseed(wl.MASTER_SEED, seed), phys_perm=True)
    K, V, bt = mat["K"], mat["V"], mat["bt"]
    if c["common"]:                   # every key of a group shares one offset
        gen = torch.Generator(device=DEV)
        gen.manual_seed(wl._subseed(seed, 11))
        for g in range(rec.G):
            off = c["common"] * torch.randn(rec.r, generator=gen, device=DEV, dtype=torch.float32)
            K[g] = (K[g].float() + off).to(K.dtype)
    ctx = kb.Context(DEV)
    cache = kb.Cache(K, V, bt, rec.t, rec.d)
    cache.free_list.zero_()
    plan = kb.Plan(ctx, cache, kb.tree_spec(rec.leaf_start, rec.leaf_count, rec.unit_leaf_ptr))
    if c["screen"] in ("fp8", "fp8c"):
        kb.set_screen_fp8(ctx, plan, centre=c["screen"] == "fp8c")
    elif c["screen"] == "prefix":
        kb.set_screen_prefix(ctx, plan, rec.r // 4)
    return rec, ctx, cache, plan


def _all_heads(c, rec, cache):
    """The fused cache as one of all-head blocks (one table per layer, the first head's): [layers][P][t][heads][d]."""
    L, H = rec.layers, rec.kv_heads

    def pool(x):
        return x.view(L, H, cache.P, rec.t, rec.d).permute(0, 2, 3, 1, 4).contiguous().view(L, cache.P, rec.r * H)

    ah = kb.Cache(pool(cache.K), pool(cache.V), cache.bt.view(L, H, -1)[:, 0].contiguous(), rec.t, rec.d * H)
    ah.scale_k.copy_(cache.scale_k.view(L, H, -1)[:, 0])
    ah.scale_v.copy_(cache.scale_v.view(L, H, -1)[:, 0])
    return ah


def prepare(case, seed):
    c = dict(_BASE, **case)
    rec, ctx, cache, plan = _state(c, seed)
    s = {"c": c, "rec": rec, "ctx": ctx, "cache": cache, "plan": plan}
    if c["op"] == "fuse":
        # The fusion works in place.  What a pass will have rewritten is kept, so that the next pass starts from the cache as
        # the prefill left it (in an engine the next batch's blocks arrive in those places).
        k0, v0, s["bt0"] = cache.K.clone(), cache.V.clone(), cache.bt.clone()
        kb.fuse_tree(ctx, plan, c["thr"])
        r = rec.r
        hit = torch.cat([((cache.K[g] != k0[g]).any(-1) | (cache.V[g] != v0[g]).any(-1)) for g in range(rec.G)])
        s["rows"] = torch.nonzero(hit).flatten()
        s["k0"], s["v0"] = k0.view(-1, r)[s["rows"]].clone(), v0.view(-1, r)[s["rows"]].clone()
        del k0, v0
        _put_back(s)
        return s
    kb.fuse_tree(ctx, plan, c["thr"])
    s["plan"] = None
    s["q"] = None
    gen = torch.Generator(device=DEV)
    gen.manual_seed(wl._subseed(seed, 12))

    def queries(n):
        x = torch.randn(rec.layers, n, rec.q_heads, rec.d, generator=gen, device=DEV, dtype=torch.float32)
        return x.to(rec.dtype)

    if c["op"] == "prefill":
        begin, q0, q1 = _prefill_span(c, rec)
        s["q"] = queries(q1 - q0)
        s["plan"] = kb.PrefillPlan(ctx, cache, rec.kv_heads, rec.q_heads, 0, begin, q0, q1, reuse=c["reuse"])
    else:
        ctx_len = _contexts(c, rec)
        s["q"] = queries(rec.B)
        s["rs"] = torch.from_numpy(rec.req_start.astype(np.int32)).to(DEV)
        s["cl"] = torch.from_numpy(ctx_len).to(DEV)
        s["max_blocks"] = int((int(ctx_len.max()) + rec.t - 1) // rec.t)
        if c["op"] == "shared":
            s["plan"] = kb.SharedDecodePlan(ctx, cache, rec.kv_heads, rec.req_start, ctx_len, rec.q_heads)
        else:
            if c["all_heads"]:
                s["cache"] = _all_heads(c, rec, cache)
            s["ws"] = torch.empty(kb.decode_workspace_bytes(rec.layers, rec.B, rec.q_heads, rec.kv_heads, rec.d, s["max_blocks"]),
                                  device=DEV, dtype=torch.uint8)
    s["out"] = torch.empty(s["q"].shape, device=DEV, dtype=torch.float32)
    return s


def _put_back(s):
    cache, r = s["cache"], s["rec"].r
    cache.K.view(-1, r)[s["rows"]] = s["k0"]
    cache.V.view(-1, r)[s["rows"]] = s["v0"]
    cache.bt.copy_(s["bt0"])


def run(state):
    s, c = state, state["c"]
    ctx, cache, rec = s["ctx"], s["cache"], s["rec"]
    if c["op"] == "fuse":
        _put_back(s)
        st = kb.fuse_tree(ctx, s["plan"], c["thr"])
        return {"K": cache.K, "V": cache.V, "bt": cache.bt, "scale_k": cache.scale_k, "scale_v": cache.scale_v,
                "refcount": cache.refcount, "remap": cache.remap, "free_list": cache.free_list, "n_free": cache.n_free,
                "n_phys": cache.n_phys, "norm_k": cache.norm_k, "norm_v": cache.norm_v, "orig_norm_k": cache.orig_norm_k,
                "fused": st.fused, "physical": st.physical_blocks}
    if c["op"] == "prefill":
        return kb.prefill_attn(ctx, cache, s["plan"], s["q"], out=s["out"])
    if c["op"] == "shared":
        return kb.paged_decode_attn_shared(ctx, cache, s["plan"], s["q"], out=s["out"])
    step = kb.paged_decode_attn_all_heads if c["all_heads"] else kb.paged_decode_attn
    return step(ctx, cache, rec.kv_heads, s["q"], s["rs"], s["cl"], s["max_blocks"], workspace=s["ws"], out=s["out"])


# ---- further cases of the same ranges ---------------------------------------------------------------------------------------

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    """Rough upper bound of a pass: (bytes of the cache, multiply-adds of the tree without fusion, of the attention)."""
    n = c["requests"] * c["tokens"] if c["kind"] != "cff" else c["tokens"]
    blocks = n // c["t"] + 1
    groups = c["layers"] * c["kv_heads"]
    block = c["t"] * c["d"]
    cache = groups * blocks * block * 4.0 * (2 if c["dtype"] == "f32" else 1)
    tree = groups * 0.5 * blocks * blocks * block * (16 if c["dtype"] == "f32" else 1)
    attn = groups * c["rep"] * c["d"] * c["tokens"] * max(c["queries"], c["requests"])
    return cache, tree, attn


def draw(rng):
    while True:
        op = rng.choice(["fuse", "fuse", "fuse", "decode", "decode", "prefill", "shared"])
        c = _case(op=op, layers=_log(rng, 1, 32), kv_heads=rng.choice([1, 2, 4, 8]), t=rng.choice([16, 16, 16, 32]),
                  d=rng.choice([64, 128, 128]), rep=rng.choice([1, 2, 4, 4, 8, 16]), tokens=_log(rng, 100, 32768))
        c["requests"] = _log(rng, 1 if op == "decode" else 2, 512)
        c["thr"] = rng.choice([0.8, 0.85, 0.9, 0.95])
        c["common"] = rng.choice([0.0, 0.0, 1.0])
        if op == "prefill":
            c["kind"], c["requests"] = "cff", 1
            c["tokens"] = max(c["tokens"], 4 * c["t"])
            c["chunk"] = rng.choice([512, 1024, 2048])
            c["queries"] = min(_log(rng, 1, 2048), c["tokens"] // c["t"] * c["t"])
            c["reuse"] = rng.random() < 0.75
        elif op == "shared":
            c["kind"] = "bff"
            c["prefix"] = int(c["tokens"] * rng.uniform(0.3, 0.9)) // c["t"] * c["t"]
        else:
            c["kind"] = rng.choice(["bff", "bff", "cff", "zipf", "mixed"])
            if c["kind"] == "cff":
                c["requests"], c["chunk"] = 1, rng.choice([512, 1024, 2048])
            c["prefix"] = int(c["tokens"] * rng.choice([0.0, 0.25, 0.5])) // c["t"] * c["t"]
            if rng.random() < 0.15:
                c["dtype"] = "f32"
            if op == "fuse":
                c["screen"] = rng.choice(["none", "none", "none", "prefix", "fp8", "fp8c"])
                if c["screen"] == "prefix" and (c["thr"] < 0.9 or c["common"]):     # not what that option is made for
                    c["screen"] = "none"
            elif c["kind"] != "cff" and rng.random() < 0.2:
                c["all_heads"] = True
        if c["all_heads"] and c["kv_heads"] * c["t"] * c["d"] * 4 > 32768:
            c["all_heads"] = False
        cache, tree, attn = _cost(c)
        # no larger than the listed ones: a third of the largest cache, half of the largest tree, half of the longest prefill
        if c["tokens"] < 4 * c["t"] or cache > 6e9 or tree > 2.5e13 or attn > 6e11:
            continue
        if op == "fuse" and cache < 2e5:
            continue
        return c
