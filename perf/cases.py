"""Performance cases of the verification step: what a serving program calls per
decoding step, from one sequence to a full card's batch.

A case is one call (for tree acceptance: the acceptance and the KV move that
follows it) through the package's public entry points, with the inputs, the
output buffers and the workspace that a serving loop keeps between steps.
Lengths belong to the case (drawn from its ``lens`` number), so that its work
is fixed; their order over the batch and all values come from the seed.

Kinds: "chain" (verify_attn), "tree" (verify_attn_tree), "paged"
(verify_attn_paged over a shuffled pool, chain or tree drafts), "accept"
(accept_greedy) and "accept_tree" (accept_greedy_tree + compact_accepted_kv).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2508_21706_amd as sm
from paper_2508_21706_amd import workloads as wl

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CODES = {"f32": sm.binding.SPECMOE_F32, "bf16": sm.binding.SPECMOE_BF16, "f16": sm.binding.SPECMOE_F16}
ELT = {"f32": 4, "bf16": 2, "f16": 2}


def _attn(name, kind, B, Hq, Hkv, D, dtype, ctx_lo, ctx_hi, chunk_lo, chunk_hi, lens, page=0, tree=False):
    case = dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, D=D, dtype=dtype, ctx_lo=ctx_lo, ctx_hi=ctx_hi, chunk_lo=chunk_lo,
                chunk_hi=chunk_hi, lens=lens, page=page, tree=tree)
    return dict(case, name=name) if name else case


def _accept(name, kind, B, C, V, dtype, chunk_lo, lens):
    case = dict(kind=kind, B=B, C=C, V=V, dtype=dtype, chunk_lo=chunk_lo, lens=lens)
    return dict(case, name=name) if name else case


def listed():
    return [
        # a toy model or a unit test's call: all latency
        _attn("attn_tiny_f32", "chain", 2, 4, 1, 64, "f32", 128, 200, 4, 4, 1),
        # an interactive server with few users: Mixtral-8x7B's layer shape
        # (32 query and 8 KV heads of 128), drafts of 5
        _attn("attn_b4", "chain", 4, 32, 8, 128, "bf16", 512, 2048, 5, 5, 2),
        # the ordinary batch of the same model
        _attn("attn_b64", "chain", 64, 32, 8, 128, "bf16", 512, 2048, 5, 5, 3),
        # the same with 16-token tree drafts
        _attn("attn_tree_b64", "tree", 64, 32, 8, 128, "bf16", 512, 2048, 16, 16, 4, tree=True),
        # the same with an FP16 cache in 16-token pages
        _attn("attn_paged_f16_b64", "paged", 64, 32, 8, 128, "f16", 512, 2048, 5, 5, 5, page=16),
        # ragged contexts and chunks, seven query heads per KV head
        _attn("attn_ragged_b128", "chain", 128, 28, 4, 128, "bf16", 256, 4096, 1, 16, 6),
        # the throughput end: a card full of sequences, drafts of 8
        _attn("attn_b256", "chain", 256, 32, 8, 128, "bf16", 1024, 4096, 8, 8, 7),
        # long documents
        _attn("attn_long_b32", "chain", 32, 32, 8, 128, "bf16", 16384, 32768, 4, 4, 8),
        # the draft model's own decode step: multi-head, one token
        _attn("attn_draft_b64", "chain", 64, 32, 32, 128, "bf16", 512, 2048, 1, 1, 9),
        # the acceptance step after the b64 and b256 verifications
        _accept("accept_b64", "accept", 64, 5, 32000, "bf16", 5, 10),
        _accept("accept_b256", "accept", 256, 8, 32000, "bf16", 8, 11),
        # and after the tree verification, with the move of the accepted
        # path's K/V rows
        _accept("accept_tree_b64", "accept_tree", 64, 16, 32000, "bf16", 16, 12),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


# (query heads, KV heads, head dim)
SHAPES = [(32, 8, 128), (32, 8, 128), (28, 4, 128), (32, 32, 128), (8, 1, 128), (4, 1, 64), (12, 4, 64), (16, 8, 64)]
KV_BYTES = 2.5e9       # valid K and V rows of one drawn call, at most (below the largest listed case)
CACHE_BYTES = 4.6e9    # K and V caches of one drawn state, at most
LOGIT_BYTES = 1.3e8    # logits of one drawn acceptance step, at most
KV_BYTES_F32 = 2.5e8   # fp32 caches are for small models


def draw(rng):
    lens = rng.randrange(1000, 1 << 30)
    if rng.random() < 0.3:
        kind = rng.choice(["accept", "accept", "accept_tree"])
        dtype = "bf16" if rng.random() < 0.75 else "f32"
        C = _log_int(rng, 1 if kind == "accept" else 2, 24)
        V = rng.choice([32000, 32000, 8 * _log_int(rng, 125, 19000)])
        B = min(_log_int(rng, 1, 256), max(1, int(LOGIT_BYTES / (C * V * ELT[dtype]))))
        return _accept("", kind, B, C, V, dtype, rng.choice([C, C, max(1, C // 3)]), lens)
    Hq, Hkv, D = rng.choice(SHAPES)
    g = Hq // Hkv
    dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f16", "f32"])
    kind = rng.choice(["chain", "chain", "chain", "tree", "paged", "paged"])
    tree = kind == "tree" or (kind == "paged" and rng.random() < 0.3)
    chunk_hi = min(_log_int(rng, 1, 32 if tree else 16), 128 // g)
    chunk_lo = rng.choice([chunk_hi, chunk_hi, max(1, chunk_hi // 4)])
    ctx_hi = _log_int(rng, 64, 32768)
    ctx_lo = max(1, int(ctx_hi * rng.uniform(0.1, 1.0)))
    row = 2 * Hkv * D * ELT[dtype]   # K and V bytes of one token
    cap = KV_BYTES_F32 if dtype == "f32" else KV_BYTES
    S = wl.round_up(ctx_hi + chunk_hi, 256)
    most = max(1, min(int(cap / (row * (ctx_hi + chunk_hi))), int(CACHE_BYTES / (row * S))))
    return _attn("", kind, min(_log_int(rng, 1, 256), most), Hq, Hkv, D, dtype, ctx_lo, ctx_hi, chunk_lo, chunk_hi,
                 lens, page=rng.choice([16, 16, 64, 128]) if kind == "paged" else 0, tree=tree)


def _lengths(case):
    """Context and chunk lengths of the case, before the seed orders them."""
    rng = np.random.default_rng([case["lens"], 1])
    B = case["B"]
    if "ctx_lo" in case:
        ctx = rng.integers(case["ctx_lo"], case["ctx_hi"] + 1, size=B)
        chunk = rng.integers(case["chunk_lo"], case["chunk_hi"] + 1, size=B)
    else:
        ctx = rng.integers(512, 2049, size=B)
        chunk = rng.integers(case["chunk_lo"], case["C"] + 1, size=B)
    return ctx.astype(np.int32), chunk.astype(np.int32)


def _ordered(case, seed):
    ctx, chunk = _lengths(case)
    order = np.random.default_rng([seed, 2]).permutation(case["B"])
    return ctx[order], chunk[order]


def _cache_rows(case):
    return wl.round_up(case["ctx_hi"] + case["chunk_hi"], 256)


def _attn_state(case, seed, dev):
    ctx, chunk = _ordered(case, seed)
    gen = torch.Generator(device=dev).manual_seed(seed)
    dt = DTYPES[case["dtype"]]
    B, Hq, Hkv, D, C, S = case["B"], case["Hq"], case["Hkv"], case["D"], case["chunk_hi"], _cache_rows(case)
    st = dict(kind=case["kind"], scale=1.0 / math.sqrt(D))
    st["q"] = torch.randn((B, C, Hq, D), generator=gen, device=dev, dtype=dt)
    if case["page"]:
        n = B * (S // case["page"])
        shape = (n + 8, Hkv, case["page"], D)   # a pool with a few pages free
        table = np.random.default_rng([seed, 5]).permutation(n + 8)[:n].astype(np.int32)
        st["table"] = torch.from_numpy(table.reshape(B, -1)).to(dev)
    else:
        shape = (B, Hkv, S, D)
    st["k"] = torch.randn(shape, generator=gen, device=dev, dtype=dt)
    st["v"] = torch.randn(shape, generator=gen, device=dev, dtype=dt)
    st["ctx"], st["chunk"] = torch.from_numpy(ctx).to(dev), torch.from_numpy(chunk).to(dev)
    st["mask"] = None
    if case["tree"]:
        st["mask"] = torch.from_numpy(wl.tree_draft_masks(seed, chunk, C).view(np.int64)).to(dev)
    st["out"] = torch.empty((B, C, Hq, D), dtype=torch.float32, device=dev)
    st["lse"] = torch.empty((B, C, Hq), dtype=torch.float32, device=dev)
    st["ws"] = sm.alloc_workspace(sm.make_desc(B, Hq, Hkv, D, C, S, CODES[case["dtype"]]), dev)
    return st


def _accept_state(case, seed, dev):
    """Logits with one clear winner per row, drafts that match it with
    probability 0.7 (a tree's: their parent's winner)."""
    ctx, chunk = _ordered(case, seed)
    gen = torch.Generator(device=dev).manual_seed(seed)
    rng = np.random.default_rng([seed, 4])
    B, C, V = case["B"], case["C"], case["V"]
    st = dict(kind=case["kind"])
    logits = torch.randn((B, C, V), generator=gen, device=dev, dtype=DTYPES[case["dtype"]])
    won = rng.integers(0, V, size=(B, C))
    logits.scatter_(2, torch.from_numpy(won).to(dev).unsqueeze(2), 8.0)
    st["logits"] = logits
    parent = np.broadcast_to(np.maximum(np.arange(C) - 1, 0), (B, C))
    if case["kind"] == "accept_tree":
        words = wl.tree_draft_masks(seed, chunk, C)
        above = words & ~(np.uint64(1) << np.arange(C, dtype=np.uint64))[None, :]
        # the parent is the highest ancestor
        parent = np.array([[int(w).bit_length() - 1 if w else 0 for w in row] for row in above])
        st["mask"] = torch.from_numpy(words.view(np.int64)).to(dev)
        S = wl.round_up(2048 + C, 256)
        st["k"] = torch.randn((B, 8, S, 128), generator=gen, device=dev, dtype=torch.bfloat16)
        st["v"] = torch.randn((B, 8, S, 128), generator=gen, device=dev, dtype=torch.bfloat16)
    tokens = np.where(rng.random((B, C)) < 0.7, np.take_along_axis(won, parent, 1), rng.integers(0, V, size=(B, C)))
    tokens[:, 0] = rng.integers(0, V, size=B)
    st["tokens"] = torch.from_numpy(tokens.astype(np.int32)).to(dev)
    st["ctx"], st["chunk"] = torch.from_numpy(ctx).to(dev), torch.from_numpy(chunk).to(dev)
    st["out"] = {"argmax": torch.empty((B, C), dtype=torch.int32, device=dev)}
    for key in ("accepted", "next_token", "new_ctx_lens"):
        st["out"][key] = torch.empty((B,), dtype=torch.int32, device=dev)
    if case["kind"] == "accept_tree":
        st["out"]["path"] = torch.empty((B,), dtype=torch.int64, device=dev)
    st["ws"] = sm.alloc_accept_workspace(sm.accept_desc(B, C, V, CODES[case["dtype"]]), dev)
    return st


def prepare(case, seed):
    dev = torch.device("cuda:0")
    return (_accept_state if case["kind"].startswith("accept") else _attn_state)(case, seed, dev)


def run(st):
    kind = st["kind"]
    if kind == "chain":
        return sm.verify_attn(st["q"], st["k"], st["v"], st["ctx"], st["chunk"], st["scale"], out=st["out"],
                              lse=st["lse"], workspace=st["ws"])
    if kind == "tree":
        return sm.verify_attn_tree(st["q"], st["k"], st["v"], st["ctx"], st["chunk"], st["mask"], st["scale"],
                                   out=st["out"], lse=st["lse"], workspace=st["ws"])
    if kind == "paged":
        return sm.verify_attn_paged(st["q"], st["k"], st["v"], st["table"], st["ctx"], st["chunk"], st["scale"],
                                    draft_mask=st["mask"], out=st["out"], lse=st["lse"], workspace=st["ws"])
    if kind == "accept":
        return sm.accept_greedy(st["logits"], st["tokens"], st["ctx"], st["chunk"], out=st["out"],
                                workspace=st["ws"])
    res = sm.accept_greedy_tree(st["logits"], st["tokens"], st["mask"], st["ctx"], st["chunk"], out=st["out"],
                                workspace=st["ws"])
    sm.compact_accepted_kv(st["k"], st["v"], st["ctx"], res["path"])
    return dict(res, k=st["k"], v=st["v"])


def work(case):
    ctx, chunk = (x.astype(np.int64) for x in _lengths(case))
    B, elt = case["B"], ELT[case["dtype"]]
    if case["kind"].startswith("accept"):
        # the valid rows' logits, tokens (and mask words), lengths and outputs;
        # the few K/V rows that a tree's path moves are left out
        rows, tree = int(chunk.sum()), case["kind"] == "accept_tree"
        return {"bytes": rows * case["V"] * elt + rows * (12 if tree else 4) + B * 8 + B * case["C"] * 4
                + B * (20 if tree else 12), "flops": 0}
    Hq, Hkv, D, C = case["Hq"], case["Hkv"], case["D"], case["chunk_hi"]
    T = ctx + chunk
    kv = 2 * int(T.sum()) * Hkv * D * elt
    q = int(chunk.sum()) * Hq * D * elt
    out = B * C * Hq * (D + 1) * 4   # the padding rows are written too
    return {"bytes": kv + q + out, "flops": 4 * Hq * D * int((chunk * T).sum())}


def tolerance(case):
    if case["kind"].startswith("accept"):
        return "exact"   # whole numbers, and rows moved as they are
    # 16-bit inputs: the probabilities are rounded to the inputs' type before
    # the product with V (bf16 8, f16 11 significant bits), which leaves the
    # outputs 1.6e-3 and 2e-4 from 64-bit ones; fp32 sums are up to 6e-7 off.
    # Four times that, and for single values the usual multiple of it.
    return {"f32": {"rel": 2.5e-6}, "f16": {"rel": 8e-4}, "bf16": {"rel": 6.5e-3}}[case["dtype"]]


def exact(case, seed):
    if case["kind"].startswith("accept"):
        return None
    st = prepare(case, seed)
    B, C, Hq, D = st["q"].shape
    Hkv, g = case["Hkv"], case["Hq"] // case["Hkv"]
    dev = st["q"].device
    out = torch.zeros((B, C, Hq, D), dtype=torch.float64, device=dev)
    lse = torch.full((B, C, Hq), -math.inf, dtype=torch.float64, device=dev)
    ctx, chunk = st["ctx"].tolist(), st["chunk"].tolist()
    for b in range(B):
        l, c = ctx[b], chunk[b]
        T = l + c
        if case["page"]:
            pages = st["table"][b].long()[: -(-T // case["page"])]
            k, v = (st[n][pages].transpose(0, 1).reshape(Hkv, -1, D)[:, :T].double() for n in ("k", "v"))
        else:
            k, v = (st[n][b, :, :T].double() for n in ("k", "v"))
        hidden = torch.ones((c, T), dtype=torch.bool, device=dev).triu(l + 1)
        if case["tree"]:
            hidden[:, l:] = (st["mask"][b, :c, None] >> torch.arange(c, device=dev)) & 1 == 0
        q = st["q"][b, :c].double().reshape(c, Hkv, g, D).permute(1, 0, 2, 3).reshape(Hkv, c * g, D)
        s = torch.matmul(q, k.transpose(1, 2).contiguous()) * st["scale"]
        s.masked_fill_(hidden.repeat_interleave(g, 0), -math.inf)
        z = torch.logsumexp(s, -1)
        o = torch.matmul(torch.exp(s - z[..., None]), v.contiguous())
        out[b, :c] = o.reshape(Hkv, c, g, D).permute(1, 0, 2, 3).reshape(c, Hq, D)
        lse[b, :c] = z.reshape(Hkv, c, g).permute(1, 0, 2).reshape(c, Hq)
    return out, lse
