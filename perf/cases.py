"""Performance cases of the draft-to-verify round.

Each case is one call, or one round of calls, as a serving program makes them
through the package's public entry points: inputs, outputs and workspaces are
in device memory before the pass and are kept from one pass to the next.

Shapes are those of the synthetic workloads (vocabulary 151936, 32 query and
8 KV heads of dimension 128, blocks of 16 or 32 positions, budgets 8 to 512,
1 to 32 sequences) and, for drawn cases, the ranges around them.
"""
import ctypes
import heapq
import math

import numpy as np
import torch

import paper_2607_22634_amd as P

DEV = "cuda"
VOCAB = 151936
MODES = {"best": P.PRESTO_TREE_BEST_FIRST, "beam": P.PRESTO_TREE_BEAM}


def _dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _esize(name):
    return 2 if name == "bf16" else 4


# ---------------------------------------------------------------------------
# the cases

def _topk(rows, k, dtype, entropy=False, vocab=VOCAB, pad=0):
    return dict(kind="topk", rows=rows, k=k, dtype=dtype, entropy=entropy, vocab=vocab, pad=pad)


def _tree(batch, depth, k, budget, mode="best", width=0, lam=0.2):
    return dict(kind="tree", batch=batch, depth=depth, k=k, budget=budget, mode=mode, width=width, lam=lam)


def _attn(batch, nodes, lo, hi, dtype="bf16", hq=32, hkv=8, dim=128, hint=False, slots=False):
    return dict(kind="attn", batch=batch, nodes=nodes, ctx_lo=lo, ctx_hi=hi, dtype=dtype, hq=hq, hkv=hkv,
                dim=dim, hint=hint, slots=slots)


def _accept(batch, nodes, depth, dtype="bf16", vocab=VOCAB):
    return dict(kind="accept", batch=batch, nodes=nodes, depth=depth, dtype=dtype, vocab=vocab)


def _round(dtype, depth, vocab, k, budget, hq, hkv, dim, ctx):
    return dict(kind="round", dtype=dtype, depth=depth, vocab=vocab, k=k, budget=budget, hq=hq, hkv=hkv, dim=dim,
                ctx=ctx)


def listed():
    return [
        # the smallest round (a toy model in fp32, as one debugs with): every
        # call is launch latency
        dict(name="round-tiny-f32", **_round("f32", 4, 1024, 2, 8, 2, 1, 64, 128)),
        # interactive decoding of one sequence: a whole round of one target
        # layer and its bookkeeping
        dict(name="round-single", **_round("bf16", 16, VOCAB, 4, 64, 32, 8, 128, 4096)),
        # drafter head output of 32 sequences with blocks of 32 positions:
        # the paper's k = 10 and the entropy-adaptive weight
        dict(name="topk-batch", **_topk(1024, 10, "bf16", entropy=True)),
        # between two rounds of self-speculation, one sequence: the slot block
        # of the last accepted node, its candidates (fp32 head), the trigram
        # lattice, the next tree and its flattened input layout
        dict(name="selfspec-next", kind="next", dtype="f32", nodes=65, slots=14, vocab=VOCAB, k=4, budget=64,
             trigrams=1 << 20),
        # tree search of one sequence (latency of the round)
        dict(name="tree-single", **_tree(1, 16, 4, 64)),
        # tree search of a serving batch, long blocks, marginal-only scores
        dict(name="tree-batch", **_tree(32, 32, 4, 128, lam=0.0)),
        # large trees
        dict(name="tree-large", **_tree(4, 16, 8, 256)),
        # the paper's default policy (beam of 10, k = 10) at its largest budget
        dict(name="tree-beam", **_tree(1, 16, 10, 512, mode="beam", width=10)),
        # a serving batch with ragged contexts in slotted caches
        dict(name="attn-serving", **_attn(16, 33, 1024, 8192, hint=True, slots=True)),
        # long contexts and large trees
        dict(name="attn-large", **_attn(4, 257, 32768, 32768)),
        # an fp32 target layer
        dict(name="attn-f32", **_attn(2, 33, 2048, 2048, dtype="f32")),
        # acceptance over a serving batch
        dict(name="accept-batch", **_accept(32, 129, 32)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["topk", "tree", "tree", "attn", "attn", "accept", "round"])
    if kind == "topk":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        vocab = rng.choice([VOCAB, VOCAB, _log_int(rng, 1000, 200000)])
        rows = _log_int(rng, 1, 1024 if dtype == "bf16" else 512)
        return _topk(min(rows, 1024 * VOCAB // vocab), rng.randint(1, 16), dtype, rng.random() < 0.4, vocab,
                     rng.choice([0, 0, rng.randint(1, 40)]))
    if kind == "tree":
        k, mode = rng.choice([2, 3, 4, 4, 5, 8, 10]), rng.choice(["best", "best", "beam"])
        depth = rng.randint(12, 32) if k <= 7 else rng.randint(8, 28)
        budget = _log_int(rng, 8, 600)
        return _tree(_log_int(rng, 1, 32), depth, k, budget, mode, rng.randint(4, 25) if mode == "beam" else 0,
                     rng.choice([0.0, 0.2, 0.2, 0.5]))
    if kind == "attn":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        hq, hkv = rng.choice([(32, 8), (32, 8), (8, 8), (16, 2), (40, 8)])
        nodes = _log_int(rng, 8, 300) if dtype == "bf16" else _log_int(rng, 8, 40)
        batch = _log_int(rng, 1, 32) if dtype == "bf16" else rng.randint(1, 2)
        hi = _log_int(rng, 100, 33000) if dtype == "bf16" else _log_int(rng, 100, 2048)
        while batch > 1 and batch * hi > 4 * 32768:
            batch -= 1
        if batch * nodes * hi > 4 * 257 * 32768:
            nodes = 4 * 257 * 32768 // (batch * hi)
        ragged = rng.random() < 0.5
        return _attn(batch, nodes, max(1, hi // 8) if ragged else hi, hi, dtype, hq, hkv, rng.choice([64, 128, 128]),
                     hint=ragged and rng.random() < 0.7, slots=rng.random() < 0.5)
    if kind == "accept":
        nodes = _log_int(rng, 8, 400)
        return _accept(max(1, min(_log_int(rng, 1, 32), 4128 // nodes)), nodes, rng.randint(8, 32),
                       rng.choice(["bf16", "bf16", "f32"]) if nodes < 130 else "bf16",
                       rng.choice([VOCAB, _log_int(rng, 1000, VOCAB)]))
    return _round("bf16", rng.randint(12, 20), rng.choice([32000, 32003, VOCAB]), rng.choice([3, 4, 8]),
                  _log_int(rng, 16, 200), 32, 8, 128, _log_int(rng, 200, 8000))


# ---------------------------------------------------------------------------
# inputs, from the seed alone and without the package

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _logits(g, rows, vocab, dtype, pad=0):
    """Head outputs: N(0, 4^2) with one to three raised tokens per row."""
    x = torch.empty(rows, vocab + pad, dtype=_dtype(dtype), device=DEV)
    for r in range(0, rows, 256):
        n = min(256, rows - r)
        y = torch.randn(n, vocab + pad, generator=g, device=DEV) * 4
        at = torch.randint(0, vocab, (n, 3), generator=g, device=DEV)
        y.scatter_(1, at, 14 + 8 * torch.rand(n, 3, generator=g, device=DEV))
        x[r:r + n] = y.to(x.dtype)
    return x[:, :vocab]


def _random_tree(rng, n_max, nodes, max_depth, vocab):
    """Parents (before their children), depths, tokens (distinct among
    siblings) and ancestor bits of one random draft tree."""
    parent = np.full(n_max, -1, np.int32)
    depth = np.full(n_max, -1, np.int32)
    token = np.full(n_max, -1, np.int32)
    words = (n_max + 63) // 64
    anc = np.zeros((n_max, words), np.uint64)
    depth[0], token[0] = 0, rng.integers(0, vocab)
    anc[0, 0] = 1
    taken = [set() for _ in range(n_max)]
    for n in range(1, nodes):
        p = int(rng.integers(max(0, n - 12), n))
        while depth[p] >= max_depth:
            p = int(parent[p])
        t = int(rng.integers(0, vocab))
        while t in taken[p]:
            t = int(rng.integers(0, vocab))
        taken[p].add(t)
        parent[n], depth[n], token[n] = p, depth[p] + 1, t
        anc[n] = anc[p]
        anc[n, n // 64] |= np.uint64(1) << np.uint64(n % 64)
    return parent, depth, token, anc


def _dev(a):
    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.int64) if a.dtype == np.uint64 else a).to(DEV)


def _candidates(g, batch, depth, k, vocab=VOCAB):
    """A top-k table as a drafter with one clear and some near choices per
    position gives it: bf16 logits (so that equal values are common) against
    a normaliser above them."""
    z = (14 + 4 * torch.rand(batch, depth, k, generator=g, device=DEV)).to(torch.bfloat16).float()
    z[:, :, 0] += 2 * torch.rand(batch, depth, generator=g, device=DEV).to(torch.bfloat16).float()
    z = z.sort(dim=-1, descending=True).values
    lse = torch.logsumexp(z, -1, keepdim=True) + 0.5 * torch.rand(batch, depth, 1, generator=g, device=DEV)
    ids = torch.argsort(torch.rand(batch, depth, 8 * k, generator=g, device=DEV), dim=-1)[..., :k]
    ids = (ids * (vocab // (8 * k))).to(torch.int32)
    return ids.contiguous(), (z - lse).contiguous()


def _lattice(g, batch, depth, k, floor=True):
    u = torch.log(1e-3 + (1 - 1e-3) * torch.rand(batch, depth, k, k, k, generator=g, device=DEV))
    if floor:
        miss = torch.rand(batch, depth, k, k, k, generator=g, device=DEV) < 0.5
        u = torch.where(miss, torch.full_like(u, math.log(1e-4)), u)
    return u.contiguous()


def _attn_inputs(g, rng, c):
    b, n, hq, hkv, d = c["batch"], c["nodes"], c["hq"], c["hkv"], c["dim"]
    ctx = rng.integers(c["ctx_lo"], c["ctx_hi"] + 1, b).astype(np.int32)
    if c["slots"]:  # every sequence's slot has room for what it will append
        start = np.concatenate([[0], np.cumsum(ctx + 40)[:-1]]).astype(np.int32)
        rows, off = int((ctx + 40).sum()), np.stack([start, ctx], 1)
    else:
        start = np.concatenate([[0], np.cumsum(ctx)[:-1]]).astype(np.int32)
        rows, off = int(ctx.sum()), np.concatenate([[0], np.cumsum(ctx)]).astype(np.int32)
    t = _dtype(c["dtype"])
    new = lambda *s: torch.randn(*s, generator=g, device=DEV).to(t)  # noqa: E731
    trees = [_random_tree(rng, n, n if i % 3 else max(1, n - i % 2 * (n // 4)), 31, VOCAB) for i in range(b)]
    live = np.array([(tr[1] >= 0).sum() for tr in trees], np.int32)
    return dict(q=new(b, n, hq, d), kc=new(rows, hkv, d), vc=new(rows, hkv, d), kt=new(b, n, hkv, d),
                vt=new(b, n, hkv, d), off=_dev(off), start=start, ctx=ctx, live=live, n_nodes=_dev(live),
                anc=_dev(np.stack([tr[3] for tr in trees])), anc_np=[tr[3] for tr in trees])


def _accept_inputs(g, rng, c):
    b, n, vocab = c["batch"], c["nodes"], c["vocab"]
    trees = [_random_tree(rng, n, n, c["depth"], vocab) for _ in range(b)]
    logits = _logits(g, b * n, vocab, c["dtype"])
    # the target agrees with the draft at most nodes: a node's best token is
    # that of its first child
    at_r, at_t = [], []
    for s, (parent, _, token, _) in enumerate(trees):
        seen = set()
        for m in range(1, n):
            p = int(parent[m])
            if p not in seen and rng.random() < 0.8:
                at_r.append(s * n + p)
                at_t.append(int(token[m]))
            seen.add(p)
    logits[torch.tensor(at_r, device=DEV), torch.tensor(at_t, device=DEV)] = 30.0
    i32 = lambda j: _dev(np.stack([t[j] for t in trees]))  # noqa: E731
    return dict(logits=logits.view(b, n, vocab), parent=i32(0), token=i32(2), trees=trees,
                n_nodes=torch.full((b,), n, dtype=torch.int32, device=DEV))


def _round_inputs(g, rng, c):
    """One sequence: a drafter block, a dense prefix signal, one layer's
    queries, keys and values, the cache with room to append, and the target's
    logits (the drafter's rows with noise: the n-th node, for the first nodes
    mostly a chain, agrees with the n-th position)."""
    d, n, vocab, t = c["depth"], c["budget"] + 1, c["vocab"], _dtype(c["dtype"])
    new = lambda *s: torch.randn(*s, generator=g, device=DEV).to(t)  # noqa: E731
    drafter = _logits(g, d, vocab, c["dtype"])
    rows = torch.arange(n, device=DEV).clamp(max=d - 1)
    target = torch.cat([(drafter[rows[i:i + 64]].float() + torch.randn(min(64, n - i), vocab, generator=g, device=DEV))
                        .to(t) for i in range(0, n, 64)])
    rows = c["ctx"] + d + 8
    return dict(drafter=drafter, rho=_lattice(g, 1, d, c["k"], floor=False),
                lam=torch.full((d,), 0.2, device=DEV), root=_dev(rng.integers(0, vocab, 1).astype(np.int32)),
                q=new(1, n, c["hq"], c["dim"]), kc=new(rows, c["hkv"], c["dim"]), vc=new(rows, c["hkv"], c["dim"]),
                kt=new(1, n, c["hkv"], c["dim"]), vt=new(1, n, c["hkv"], c["dim"]), target=target.view(1, n, vocab),
                ctx0=_dev(np.array([[0, c["ctx"]]], np.int32)), cap=_dev(np.array([rows], np.int32)))


def _next_inputs(g, rng, c):
    """After acceptance in self-speculation: the accepted path, the slot
    logits of every node, and a trigram table of which about half of the
    trigrams of the next block are known."""
    n, s, vocab, k = c["nodes"], c["slots"], c["vocab"], c["k"]
    parent, depth, token, _ = _random_tree(rng, n, n, 16, vocab)
    last = int(rng.integers(n // 2, n))
    path = [last]
    while path[0] > 0:
        path.insert(0, int(parent[path[0]]))
    logits = _logits(g, n * s, vocab, c["dtype"])
    cand = logits[last * s + 1:last * s + s].float().topk(k).indices.cpu().numpy()
    prev, root = int(rng.integers(0, vocab)), int(rng.integers(0, vocab))
    known = {}
    rows = [[prev], [root]] + [list(r) for r in cand]
    for j in range(2, len(rows)):
        for a in rows[j - 2]:
            for b in rows[j - 1]:
                for t in rows[j]:
                    if rng.random() < 0.5:
                        known[(int(a), int(b), int(t))] = 1
    tri = np.concatenate([np.array(list(known), np.int64).reshape(-1, 3), rng.integers(0, vocab, (c["trigrams"], 3))])
    tri = np.unique(tri, axis=0)
    val = np.log(rng.uniform(1e-3, 1.0, len(tri))).astype(np.float32)
    full = np.full((1, 17), -1, np.int32)
    full[0, :len(path)] = path
    return dict(path=_dev(full), accept_len=_dev(np.array([len(path) - 1], np.int32)), logits=logits, last=last,
                prev=_dev(np.array([prev], np.int32)), root=_dev(np.array([root], np.int32)), tri=tri, val=val,
                lam=torch.full((s - 1,), 0.2, device=DEV), root_pos=_dev(np.array([4096], np.int32)))


def _inputs(c, seed):
    g, rng = _gen(seed), np.random.default_rng([seed, 1])
    if c["kind"] == "topk":
        return dict(logits=_logits(g, c["rows"], c["vocab"], c["dtype"], c["pad"]))
    if c["kind"] == "tree":
        ids, lp = _candidates(g, c["batch"], c["depth"], c["k"])
        rho = _lattice(g, c["batch"], c["depth"], c["k"]) if c["lam"] else None
        return dict(ids=ids, lp=lp, rho=rho, lam=torch.full((c["depth"],), c["lam"], device=DEV),
                    root=_dev(rng.integers(0, VOCAB, c["batch"]).astype(np.int32)))
    return {"attn": _attn_inputs, "accept": _accept_inputs, "round": _round_inputs, "next": _next_inputs}[c["kind"]](
        g, rng, c)


# ---------------------------------------------------------------------------
# what a program keeps: outputs and workspaces

def _i32(*shape):
    return torch.empty(*shape, dtype=torch.int32, device=DEV)


def _f32(*shape):
    return torch.empty(*shape, dtype=torch.float32, device=DEV)


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device=DEV)


def _topk_out(rows, k):
    return dict(ids=_i32(rows, k), logprob=_f32(rows, k), lse=_f32(rows))


def _tree_out(batch, budget):
    n = budget + 1
    return dict(n_nodes=_i32(batch), parent=_i32(batch, n), token=_i32(batch, n), depth=_i32(batch, n),
                rank=_i32(batch, n), score=_f32(batch, n),
                anc=torch.empty(batch, n, (n + 63) // 64, dtype=torch.int64, device=DEV))


def _accept_out(batch, n, depth):
    return dict(accept_len=_i32(batch), path=_i32(batch, depth + 1), bonus=_i32(batch), target_argmax=_i32(batch, n))


def _attn_ws(q, hkv, max_ctx, layout, total):
    b, n, hq, d = q.shape
    desc = P.AttnDesc(b, n, hq, hkv, d, max_ctx, d ** -0.5,
                      P.PRESTO_DT_BF16 if q.dtype == torch.bfloat16 else P.PRESTO_DT_F32, layout, total)
    return _bytes(P.lib().presto_tree_attention_workspace(ctypes.byref(desc)))


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    s["case"] = c
    kind = c["kind"]
    if kind == "topk":
        s["out"] = _topk_out(c["rows"], c["k"])
        s["ws"] = P.topk_workspace(c["rows"], c["vocab"], c["k"], DEV)
        s["entropy"] = _f32(c["rows"]) if c["entropy"] else None
        s["lam"] = _f32(c["rows"]) if c["entropy"] else None
    elif kind == "tree":
        s["out"] = _tree_out(c["batch"], c["budget"])
    elif kind == "attn":
        s["layout"] = P.PRESTO_CTX_SLOTS if c["slots"] else P.PRESTO_CTX_PACKED
        s["max_ctx"], s["total"] = int(s["ctx"].max()), int(s["ctx"].sum()) if c["hint"] else 0
        s["out"] = torch.empty_like(s["q"])
        s["ws"] = _attn_ws(s["q"], c["hkv"], s["max_ctx"], s["layout"], s["total"])
    elif kind == "accept":
        s["out"] = _accept_out(c["batch"], c["nodes"], c["depth"])
        s["ws"] = _bytes(P.lib().presto_accept_workspace(c["batch"], c["nodes"], c["vocab"]))
    elif kind == "round":
        n = c["budget"] + 1
        s["topk"], s["topk_ws"] = _topk_out(c["depth"], c["k"]), P.topk_workspace(c["depth"], c["vocab"], c["k"], DEV)
        s["tree"], s["att"] = _tree_out(1, c["budget"]), torch.empty_like(s["q"])
        s["att_ws"] = _attn_ws(s["q"], c["hkv"], c["ctx"], P.PRESTO_CTX_SLOTS, c["ctx"])
        s["acc"], s["ctx"] = _accept_out(1, n, c["depth"]), torch.empty_like(s["ctx0"])
        s["acc_ws"] = _bytes(P.lib().presto_accept_workspace(1, n, c["vocab"]))
        s["flags"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    else:
        cap = 64
        while cap < 2 * len(s["tri"]):
            cap *= 2
        s["cap"], s["table"] = cap, _bytes(P.presto_ngram_table_bytes(cap))
        P.presto_ngram_clear(s["table"], cap)
        t = _dev(s["tri"].astype(np.int32))
        P.presto_ngram_insert(s["table"], cap, t[:, 0].contiguous(), t[:, 1].contiguous(), t[:, 2].contiguous(),
                              _dev(s["val"]))
        rows, k = c["slots"] - 1, c["k"]
        s["sel"] = torch.empty(1, rows, dtype=torch.int64, device=DEV)
        s["topk"], s["topk_ws"] = _topk_out(rows, k), P.topk_workspace(rows, c["vocab"], k, DEV)
        s["rho"], s["tree"] = _f32(1, rows, k, k, k), _tree_out(1, c["budget"])
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "topk":
        out = P.presto_topk(s["logits"], c["k"], entropy=s["entropy"], workspace=s["ws"], **s["out"])
        if c["entropy"]:
            return (*out, P.presto_entropy_lambda(s["entropy"], 0.6, 2.0, out=s["lam"]))
        return out
    if kind == "tree":
        return P.presto_build_tree(s["ids"], s["lp"], s["rho"], s["lam"], s["root"], c["depth"], c["k"], c["budget"],
                                   mode=MODES[c["mode"]], beam_width=c["width"], out=s["out"])
    if kind == "attn":
        return P.presto_tree_attention(s["q"], s["kc"], s["vc"], s["off"], s["kt"], s["vt"], s["anc"], s["n_nodes"],
                                       s["max_ctx"], out=s["out"], workspace=s["ws"], ctx_layout=s["layout"],
                                       total_ctx=s["total"])
    if kind == "accept":
        return P.presto_accept(s["logits"], s["parent"], s["token"], s["n_nodes"], c["depth"], out=s["out"],
                               workspace=s["ws"])
    if kind == "round":
        s["ctx"].copy_(s["ctx0"])  # the scheduler's record of the sequence
        ids, lp, lse = P.presto_topk(s["drafter"], c["k"], flags=s["flags"], workspace=s["topk_ws"], **s["topk"])
        tree = P.presto_build_tree(ids, lp, s["rho"], s["lam"], s["root"], c["depth"], c["k"], c["budget"],
                                   out=s["tree"])
        att = P.presto_tree_attention(s["q"], s["kc"], s["vc"], s["ctx"], s["kt"], s["vt"], tree["anc"],
                                      tree["n_nodes"], c["ctx"], out=s["att"], workspace=s["att_ws"],
                                      ctx_layout=P.PRESTO_CTX_SLOTS, total_ctx=c["ctx"])
        acc = P.presto_accept(s["target"], tree["parent"], tree["token"], tree["n_nodes"], c["depth"], out=s["acc"],
                              flags=s["flags"], workspace=s["acc_ws"])
        P.presto_commit_kv(s["kt"], s["vt"], acc["path"], acc["accept_len"], s["kc"], s["vc"], s["ctx"], s["cap"],
                           flags=s["flags"])
        return dict(ids=ids, logprob=lp, lse=lse, attention=att, k_cache=s["kc"], v_cache=s["vc"], ctx=s["ctx"],
                    flags=s["flags"], **{"tree_" + k: v for k, v in tree.items()}, **acc)
    sel = P.presto_select_slots(s["path"], s["accept_len"], c["nodes"], c["slots"], 1, out=s["sel"])
    ids, lp, lse = P.presto_topk_rows(s["logits"], sel.view(-1), c["k"], workspace=s["topk_ws"], **s["topk"])
    rows = c["slots"] - 1
    rho = P.presto_ngram_gather(s["table"], s["cap"], math.log(1e-4), ids, s["prev"], s["root"], rows, c["k"],
                                out=s["rho"])
    tree = P.presto_build_tree(ids, lp, rho, s["lam"], s["root"], rows, c["k"], c["budget"], out=s["tree"])
    flat = P.presto_flatten_slots(tree["depth"], tree["anc"], tree["n_nodes"], s["root_pos"], c["slots"])
    return dict(sel=sel, ids=ids, logprob=lp, lse=lse, rho=rho, **{"tree_" + k: v for k, v in tree.items()},
                **{"flat_" + k: v for k, v in flat.items()})


# ---------------------------------------------------------------------------
# what a pass cannot do without

def _topk_work(rows, vocab, k, e):
    return rows * vocab * e + rows * (8 * k + 4)


def _tree_work(batch, depth, k, budget, rho):
    n = budget + 1
    return batch * (depth * k * 8 + (depth * k ** 3 * 4 if rho else 0) + n * (20 + 8 * ((n + 63) // 64)))


def _attn_work(ctx, live, hq, hkv, d, e):
    """Bytes and flops of sequences with `ctx` keys and `live` nodes each."""
    b = sum(hkv * (c + n) * d * 2 * e + n * hq * d * 2 * e for c, n in zip(ctx, live))
    return b, sum(n * hq * 4 * d * (c + 6) for c, n in zip(ctx, live))


def work(case):
    c = case
    e = _esize(c["dtype"]) if "dtype" in c else 0
    if c["kind"] == "topk":
        return dict(bytes=_topk_work(c["rows"], c["vocab"], c["k"], e), flops=3 * c["rows"] * c["vocab"])
    if c["kind"] == "tree":
        return dict(bytes=_tree_work(c["batch"], c["depth"], c["k"], c["budget"], c["lam"] != 0),
                    flops=3 * c["batch"] * c["budget"] * c["k"])
    if c["kind"] == "attn":
        b = c["batch"]
        live = [c["nodes"] if i % 3 else c["nodes"] - i % 2 * (c["nodes"] // 4) for i in range(b)]
        by, fl = _attn_work([(c["ctx_lo"] + c["ctx_hi"]) / 2] * b, live, c["hq"], c["hkv"], c["dim"], e)
        return dict(bytes=int(by), flops=int(fl))
    if c["kind"] == "accept":
        return dict(bytes=c["batch"] * c["nodes"] * (c["vocab"] * e + 12), flops=c["batch"] * c["nodes"] * c["vocab"])
    if c["kind"] == "round":
        n = c["budget"] + 1
        by, fl = _attn_work([c["ctx"]], [n], c["hq"], c["hkv"], c["dim"], e)
        by += _topk_work(c["depth"], c["vocab"], c["k"], e) + _tree_work(1, c["depth"], c["k"], c["budget"], True)
        return dict(bytes=by + n * c["vocab"] * e, flops=fl + (3 * c["depth"] + n) * c["vocab"])
    rows, r = c["slots"] - 1, c["nodes"] * (1 + c["slots"])
    return dict(bytes=_topk_work(rows, c["vocab"], c["k"], e) + _tree_work(1, rows, c["k"], c["budget"], True) +
                rows * c["k"] ** 3 * 16 + r * (4 + 8 * ((r + 63) // 64)), flops=3 * rows * c["vocab"])


def tolerance(case):
    kind = case["kind"]
    if kind in ("tree", "accept"):
        return "exact"  # whole numbers, and fp32 scores whose order of operations is fixed
    if kind in ("topk", "next"):
        return {"rel": 5e-7, "max": 5e-6}  # fp32 sums over the vocabulary in another order
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 4e-5}
    return {"rel": 1.3e-2, "max": 0.08}  # bf16 queries, probabilities and split partials


# ---------------------------------------------------------------------------
# the same in 64 bits, without the package

def _exact_topk(x, k, entropy):
    ids, lp, lse, ent = [], [], [], []
    for r in range(0, x.shape[0], 32):
        z = x[r:r + 32].double()
        v, i = z.sort(dim=-1, descending=True, stable=True)
        i, v = i[:, :k], v[:, :k]
        m = v[:, :1]
        e = (z - m).exp()
        s = e.sum(-1, keepdim=True)
        ids.append(i.to(torch.int32))
        lp.append(v - m - s.log())
        lse.append((m + s.log())[:, 0])
        if entropy:
            ent.append((s.log() - (e * (z - m)).sum(-1, keepdim=True) / s)[:, 0])
    return [torch.cat(t) for t in (ids, lp, lse) + ((ent,) if entropy else ())]


def _scores(lp, rho, lam, row, c2, c1):
    """fp32 token scores of a context, rounded as the score is defined."""
    if rho is None:
        return lp[row]
    return lp[row] + lam[row] * rho[row, c2, c1]


def _children(lp, rho, lam, depth, path, S):
    """(S, rank path) of every child of a node."""
    row = len(path)
    if row >= depth:
        return []
    s = _scores(lp, rho, lam, row, path[-2] if row >= 2 else 0, path[-1] if row >= 1 else 0)
    return [(np.float32(S + s[r]), path + (r,)) for r in range(len(s))]


def _best_first(lp, rho, lam, depth, budget):
    heap, out = [], []
    push = lambda kids: [heapq.heappush(heap, (-float(S), p, S)) for S, p in kids]  # noqa: E731
    push(_children(lp, rho, lam, depth, (), np.float32(0)))
    while heap and len(out) < budget:
        _, p, S = heapq.heappop(heap)
        out.append((S, p))
        push(_children(lp, rho, lam, depth, p, S))
    return out


def _beam_search(lp, rho, lam, depth, budget, width):
    order = lambda x: (-float(x[0]), x[1])  # noqa: E731
    kept, beam = [], [(np.float32(0), ())]
    for _ in range(depth):
        if len(kept) >= budget:
            break
        kids = [ch for S, p in beam for ch in _children(lp, rho, lam, depth, p, S)]
        kept += kids
        beam = sorted(kids, key=order)[:width]
    return sorted(kept, key=order)[:budget]


def _tree_rows(nodes, ids, root, budget):
    """The flattened tree of nodes [(S, rank path)] in order."""
    n, w = budget + 1, (budget + 64) // 64
    o = dict(n_nodes=np.int32(len(nodes) + 1), parent=np.full(n, -1, np.int32), token=np.full(n, -1, np.int32),
             depth=np.full(n, -1, np.int32), rank=np.full(n, -1, np.int32), score=np.full(n, -np.inf, np.float32),
             anc=np.zeros((n, w), np.uint64))
    o["token"][0], o["depth"][0], o["score"][0], o["anc"][0, 0] = root, 0, 0, 1
    at = {(): 0}
    for i, (S, p) in enumerate(nodes, 1):
        at[p] = i
        q = at[p[:-1]]
        o["parent"][i], o["token"][i], o["depth"][i], o["rank"][i], o["score"][i] = q, ids[len(p) - 1, p[-1]], len(p), p[-1], S
        o["anc"][i] = o["anc"][q]
        o["anc"][i, i // 64] |= np.uint64(1) << np.uint64(i % 64)
    return o


def _exact_tree(ids, lp, rho, lam, root, c):
    ids, lp, lam, root = (t.cpu().numpy() for t in (ids, lp, lam, root))
    rho = None if rho is None else rho.cpu().numpy()
    rows = []
    for b in range(len(root)):
        a = (lp[b], None if rho is None else rho[b], lam, c["depth"], c["budget"])
        nodes = _beam_search(*a, c["width"]) if c.get("mode") == "beam" else _best_first(*a)
        rows.append(_tree_rows(nodes, ids[b], root[b], c["budget"]))
    out = {k: np.stack([r[k] for r in rows]) for k in rows[0]}
    out["anc"] = out["anc"].view(np.int64)
    return out


def _exact_attn(q, kc, vc, kt, vt, start, ctx, live, anc, hkv):
    b, n, hq, d = q.shape
    out = torch.zeros(b, n, hq, d, dtype=torch.float64, device=DEV)
    for s in range(b):
        m, lo, hi = int(live[s]), int(start[s]), int(start[s]) + int(ctx[s])
        bits = torch.zeros(m, m, dtype=torch.bool)
        for i in range(m):
            for w in range(anc[s].shape[1]):
                x = int(anc[s][i, w])
                for j in range(64 * w, min(m, 64 * w + 64)):
                    bits[i, j] = bool(x >> (j % 64) & 1)
        mask = torch.cat([torch.ones(m, hi - lo, dtype=torch.bool), bits], 1).to(DEV)
        for g in range(hkv):
            K = torch.cat([kc[lo:hi, g], kt[s, :m, g]]).double()
            V = torch.cat([vc[lo:hi, g], vt[s, :m, g]]).double()
            for h in range(g * hq // hkv, (g + 1) * hq // hkv):
                x = (q[s, :m, h].double() @ K.t()) * d ** -0.5
                out[s, :m, h] = x.masked_fill(~mask, -math.inf).softmax(-1) @ V
    return out


def _argmax(x):
    """The lowest id of each row's largest value."""
    m = x.float().max(-1, keepdim=True).values
    return (x.float() == m).to(torch.uint8).argmax(-1).to(torch.int32)


def _walk(a, parent, token, depth):
    path = [0]
    while True:
        kids = [m for m in range(len(parent)) if parent[m] == path[-1] and token[m] == a[path[-1]]]
        if not kids:
            break
        path.append(kids[0])
    full = np.full(depth + 1, -1, np.int32)
    full[:len(path)] = path
    return np.int32(len(path) - 1), full, np.int32(a[path[-1]])


def _exact_accept(logits, parent, token, depth):
    b, n, vocab = logits.shape
    a = torch.cat([_argmax(logits[s]) for s in range(b)]).view(b, n).cpu().numpy()
    walks = [_walk(a[s], parent[s], token[s], depth) for s in range(b)]
    return dict(accept_len=np.array([w[0] for w in walks]), path=np.stack([w[1] for w in walks]),
                bonus=np.array([w[2] for w in walks]), target_argmax=a)


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    kind = c["kind"]
    if kind == "topk":
        out = _exact_topk(s["logits"], c["k"], c["entropy"])
        return (*out, 0.6 * out[3] / (out[3] + 2.0)) if c["entropy"] else tuple(out)
    if kind == "tree":
        return _exact_tree(s["ids"], s["lp"], s["rho"], s["lam"], s["root"], c)
    if kind == "attn":
        return _exact_attn(s["q"], s["kc"], s["vc"], s["kt"], s["vt"], s["start"], s["ctx"], s["live"], s["anc_np"],
                           c["hkv"])
    if kind == "accept":
        return _exact_accept(s["logits"], [t[0] for t in s["trees"]], [t[2] for t in s["trees"]], c["depth"])
    if kind == "round":
        ids, lp, lse = _exact_topk(s["drafter"], c["k"], False)
        tree = _exact_tree(ids[None], lp.float()[None], s["rho"], s["lam"], s["root"], c)
        att = _exact_attn(s["q"], s["kc"], s["vc"], s["kt"], s["vt"], [0], [c["ctx"]], tree["n_nodes"],
                          tree["anc"].view(np.uint64), c["hkv"])
        acc = _exact_accept(s["target"], tree["parent"], tree["token"], c["depth"])
        used = acc["path"][0][:int(acc["accept_len"][0]) + 1]
        for cache, rows in ((s["kc"], s["kt"]), (s["vc"], s["vt"])):
            cache[c["ctx"]:c["ctx"] + len(used)] = rows[0, torch.from_numpy(used).long().to(DEV)]
        ctx = np.array([[0, c["ctx"] + len(used)]], np.int32)
        return dict(ids=ids, logprob=lp, lse=lse, attention=att, k_cache=s["kc"], v_cache=s["vc"], ctx=ctx,
                    flags=np.zeros(1, np.int32), **{"tree_" + k: v for k, v in tree.items()}, **acc)
    rows, n, sl, k = c["slots"] - 1, c["nodes"], c["slots"], c["k"]
    sel = s["last"] * sl + 1 + np.arange(rows)
    ids, lp, lse = _exact_topk(s["logits"][torch.from_numpy(sel).to(DEV)], k, False)
    known = {tuple(t): v for t, v in zip(s["tri"].tolist(), s["val"])}
    cand = [[int(s["prev"])], [int(s["root"])]] + ids.cpu().numpy().tolist()
    floor = np.float32(math.log(1e-4))
    rho = np.empty((1, rows, k, k, k), np.float32)
    for j in range(rows):
        for a in range(k):
            for b in range(k):
                t2 = cand[j][a] if j >= 2 else cand[j][0]
                t1 = cand[j + 1][b] if j >= 1 else cand[j + 1][0]
                for r in range(k):
                    rho[0, j, a, b, r] = known.get((t2, t1, cand[j + 2][r]), floor)
    tree = _exact_tree(ids[None], lp.float()[None], torch.from_numpy(rho), s["lam"], s["root"],
                       dict(depth=rows, budget=c["budget"]))
    tn, r = c["budget"] + 1, (c["budget"] + 1) * (1 + sl)
    pos, anc = np.full((1, r), -1, np.int32), np.zeros((1, r, (r + 63) // 64), np.uint64)
    for i in range(int(tree["n_nodes"][0])):
        up = [m for m in range(tn) if int(tree["anc"].view(np.uint64)[0, i, m // 64]) >> (m % 64) & 1]
        for j in range(1 + sl):
            row = i * (1 + sl) + j
            pos[0, row] = 4096 + tree["depth"][0, i] + j
            for col in [m * (1 + sl) for m in up] + ([i * (1 + sl) + q for q in range(1, 1 + sl)] if j else []):
                anc[0, row, col // 64] |= np.uint64(1) << np.uint64(col % 64)
    return dict(sel=sel[None].astype(np.int64), ids=ids, logprob=lp, lse=lse, rho=rho,
                **{"tree_" + k_: v for k_, v in tree.items()}, flat_pos=pos, flat_anc=anc.view(np.int64),
                flat_n_rows=(tree["n_nodes"] * (1 + sl)).astype(np.int32))
