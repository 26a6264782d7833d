"""GPU parity of presto_tree_attention against the oracle.

Per (b, n, h) row: ||o - o_ref||_2 <= tol * ||o_ref||_2 with tol = 2e-2 for
bf16 (matrix cores, fp32 accumulation, bf16 probabilities) and 1e-4 for the
fp32 path; padding rows must be exactly zero.  The small workloads are
compared in full, the large ones on sampled rows that the oracle computes
one by one, in the launch configuration the bench uses.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_22634_amd as P
import synthetic as sy
from brute import anc_from_parent
from gpu_util import attn_data, oracle_tree, round_data, to_dev, to_host, tree_to_dev, tree_to_host

pytestmark = pytest.mark.gpu


def _tree_for(cfg):
    """The oracle's tree of the workload, on the device (both sides use it)."""
    w, _ = round_data(cfg)
    return w, tree_to_dev(oracle_tree(cfg))


def _run(w, att, tree_dev, total_ctx=0):
    return P.presto_tree_attention(
        to_dev(att["q"], w.dtype), to_dev(att["k_cache"], w.dtype), to_dev(att["v_cache"], w.dtype),
        to_dev(att["ctx_offsets"]), to_dev(att["k_tree"], w.dtype), to_dev(att["v_tree"], w.dtype),
        tree_dev["anc"], tree_dev["n_nodes"], int(np.diff(att["ctx_offsets"]).max()), w.scale,
        total_ctx=total_ctx)


def _row_errors(got, ref):
    num = np.linalg.norm(got - ref, axis=-1)
    den = np.linalg.norm(ref, axis=-1)
    return num / np.maximum(den, 1e-30)


@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_attention_matches_oracle_full(cfg):
    w, tree = _tree_for(cfg)
    _, att = attn_data(cfg)
    print(f"attn cfg={cfg} full compare", flush=True)
    out = _run(w, att, tree)
    torch.cuda.synchronize()
    th = tree_to_host(tree)
    ref = oracle.tree_attention(w.dtype, att["q"], att["k_cache"], att["v_cache"],
                                att["ctx_offsets"], att["k_tree"], att["v_tree"], th["anc"],
                                th["n_nodes"], w.scale)
    got = sy.as_f32(to_host(out), w.dtype).astype(np.float64)
    reff = sy.as_f32(ref, w.dtype).astype(np.float64)
    tol = 2e-2 if w.dtype == "bf16" else 1e-4
    for s in range(w.batch):
        nn = int(th["n_nodes"][s])
        err = _row_errors(got[s, :nn], reff[s, :nn])
        assert err.max() <= tol, (s, err.max())
        assert not got[s, nn:].any()


@pytest.mark.parametrize("cfg", [4, 5])
def test_attention_matches_oracle_sampled(cfg):
    w, tree = _tree_for(cfg)
    _, att = attn_data(cfg)
    print(f"attn cfg={cfg} sampled compare", flush=True)
    out = _run(w, att, tree)
    torch.cuda.synchronize()
    th = tree_to_host(tree)
    rng = np.random.default_rng(cfg)
    rows = []
    for s in range(w.batch):
        nn = int(th["n_nodes"][s])
        nodes = {0, nn - 1} | set(rng.integers(0, nn, size=6).tolist())
        for n in nodes:
            for h in rng.choice(w.hq, size=4, replace=False):
                rows.append((s, n, int(h)))
    rows = np.array(rows, np.int32)
    ref = oracle.tree_attention_rows(w.dtype, att["q"], att["k_cache"], att["v_cache"],
                                     att["ctx_offsets"], att["k_tree"], att["v_tree"], th["anc"],
                                     th["n_nodes"], rows, w.scale)
    got = sy.as_f32(to_host(out), w.dtype)[rows[:, 0], rows[:, 1], rows[:, 2]].astype(np.float64)
    err = _row_errors(got, ref)
    assert err.max() <= 2e-2, err.max()


def _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes):
    offs = np.zeros(b + 1, np.int32)
    offs[1:] = np.cumsum(ctx)
    f = lambda *s: sy.cast(rng.standard_normal(s, dtype=np.float32), dtype)
    att = {"q": f(b, N, hq, d), "k_cache": f(max(int(offs[-1]), 1), hkv, d),
           "v_cache": f(max(int(offs[-1]), 1), hkv, d), "ctx_offsets": offs,
           "k_tree": f(b, N, hkv, d), "v_tree": f(b, N, hkv, d)}
    anc = anc_from_parent(parent, n_nodes, N)
    return att, anc


@pytest.mark.parametrize("dtype,hq,hkv,d", [("bf16", 32, 8, 128), ("bf16", 8, 8, 64),
                                            ("bf16", 16, 2, 128), ("f32", 4, 2, 128)])
def test_attention_edges(dtype, hq, hkv, d):
    rng = np.random.default_rng([hq, hkv, d])
    b, N = 5, 70
    ctx = np.array([0, 1, 63, 64, 3000], np.int32)
    parent = np.full((b, N), -1, np.int32)
    n_nodes = np.array([1, 70, 37, 2, 70], np.int32)
    for s in range(b):
        for n in range(1, int(n_nodes[s])):
            parent[s, n] = n - 1 if s == 3 else rng.integers(0, n)  # chain or random tree
    att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)
    w = sy.workload(1).with_(dtype=dtype, head_dim=d)
    scale = 1 / np.sqrt(d)
    out = P.presto_tree_attention(
        to_dev(att["q"], dtype), to_dev(att["k_cache"], dtype), to_dev(att["v_cache"], dtype),
        to_dev(att["ctx_offsets"]), to_dev(att["k_tree"], dtype), to_dev(att["v_tree"], dtype),
        to_dev(anc), to_dev(n_nodes), int(ctx.max()), scale)
    torch.cuda.synchronize()
    ref = oracle.tree_attention(dtype, att["q"], att["k_cache"], att["v_cache"],
                                att["ctx_offsets"], att["k_tree"], att["v_tree"], anc, n_nodes,
                                scale)
    got = sy.as_f32(to_host(out), dtype).astype(np.float64)
    reff = sy.as_f32(ref, dtype).astype(np.float64)
    tol = 2e-2 if dtype == "bf16" else 1e-4
    for s in range(b):
        nn = int(n_nodes[s])
        assert _row_errors(got[s, :nn], reff[s, :nn]).max() <= tol
        assert not got[s, nn:].any()


def test_attention_is_deterministic():
    w, tree = _tree_for(2)
    _, att = attn_data(2)
    a = to_host(_run(w, att, tree))
    b = to_host(_run(w, att, tree))
    np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("hint", ["actual", "tiny", "half", "uniform"])
def test_attention_ragged_total_ctx_hint(hint):
    """Ragged contexts (workload 3): the total-context hint only changes how
    the context is split and dealt to workgroups, never the result; a hint
    below the real total (down to 1) or at batch x max_ctx (no compaction)
    must match the oracle just the same."""
    w, tree = _tree_for(3)
    _, att = attn_data(3)
    ctx = np.diff(att["ctx_offsets"]).astype(np.int64)
    total = {"actual": int(ctx.sum()), "tiny": 1, "half": int(ctx.sum()) // 2,
             "uniform": int(w.batch * ctx.max())}[hint]
    print(f"attn ragged hint={hint} total_ctx={total}", flush=True)
    out = _run(w, att, tree, total_ctx=total)
    torch.cuda.synchronize()
    th = tree_to_host(tree)
    ref = oracle.tree_attention(w.dtype, att["q"], att["k_cache"], att["v_cache"],
                                att["ctx_offsets"], att["k_tree"], att["v_tree"], th["anc"],
                                th["n_nodes"], w.scale)
    got = sy.as_f32(to_host(out), w.dtype).astype(np.float64)
    reff = sy.as_f32(ref, w.dtype).astype(np.float64)
    for s in range(w.batch):
        nn = int(th["n_nodes"][s])
        err = _row_errors(got[s, :nn], reff[s, :nn])
        assert err.max() <= 2e-2, (s, err.max())
        assert not got[s, nn:].any()


@pytest.mark.parametrize("layout", ["packed", "slots"])
def test_attention_many_ragged_sequences_compact(layout):
    """More sequences than a wave has lanes (70), ragged contexts including
    empty ones, with the total-context hint: the workgroups' pair search runs
    over several 64-sequence groups.  The slots layout leaves gaps of large
    values between the sequences' cache rows, which must never be read."""
    rng = np.random.default_rng(77 if layout == "packed" else 78)
    b, N, hq, hkv, d, dtype = 70, 9, 8, 2, 64, "bf16"
    ctx = rng.integers(0, 600, b).astype(np.int32)
    ctx[[3, 40]] = 0
    ctx[65] = 3000
    parent = np.full((b, N), -1, np.int32)
    n_nodes = rng.integers(1, N + 1, b).astype(np.int32)
    for s in range(b):
        for n in range(1, int(n_nodes[s])):
            parent[s, n] = rng.integers(0, n)
    att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)
    scale = 1 / np.sqrt(d)
    total = int(ctx.sum())
    kc, vc, offs = att["k_cache"], att["v_cache"], att["ctx_offsets"]
    ctx_arg, lay = offs, P.PRESTO_CTX_PACKED
    if layout == "slots":
        gap = 5
        start = (offs[:-1] + gap * np.arange(1, b + 1)).astype(np.int32)
        rows = int(start[-1] + ctx[-1]) + gap
        big = sy.cast(np.full((rows, hkv, d), 300.0, np.float32), dtype)
        ks, vs = big.copy(), big.copy()
        for s in range(b):
            ks[start[s]:start[s] + ctx[s]] = kc[offs[s]:offs[s + 1]]
            vs[start[s]:start[s] + ctx[s]] = vc[offs[s]:offs[s + 1]]
        kc_dev, vc_dev = to_dev(ks, dtype), to_dev(vs, dtype)
        ctx_arg, lay = np.stack([start, ctx], axis=1).astype(np.int32), P.PRESTO_CTX_SLOTS
    else:
        kc_dev, vc_dev = to_dev(kc, dtype), to_dev(vc, dtype)
    print(f"attn compact layout={layout} batch={b} total_ctx={total}", flush=True)
    out = P.presto_tree_attention(
        to_dev(att["q"], dtype), kc_dev, vc_dev, to_dev(ctx_arg), to_dev(att["k_tree"], dtype),
        to_dev(att["v_tree"], dtype), to_dev(anc), to_dev(n_nodes), int(ctx.max()), scale,
        ctx_layout=lay, total_ctx=total)
    torch.cuda.synchronize()
    ref = oracle.tree_attention(dtype, att["q"], kc, vc, offs, att["k_tree"], att["v_tree"], anc,
                                n_nodes, scale)
    got = sy.as_f32(to_host(out), dtype).astype(np.float64)
    reff = sy.as_f32(ref, dtype).astype(np.float64)
    for s in range(b):
        nn = int(n_nodes[s])
        assert _row_errors(got[s, :nn], reff[s, :nn]).max() <= 2e-2, s
        assert not got[s, nn:].any()


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 128), (6, 2, 64), (32, 8, 128), (5, 5, 64)])
@pytest.mark.parametrize("how", ["split", "no_workspace", "unaligned"])
def test_attention_f32_blocks(hq, hkv, d, how):
    """fp32: query rows around a 32-row block, contexts around a 32-key block
    and around the four waves' share of a split, dead row blocks, no room for
    split partials, and tensors that are only 4-byte aligned."""
    rng = np.random.default_rng([hq, hkv, d, len(how)])
    N, dtype = 65, "f32"
    ctx = np.array([0, 1, 31, 32, 33, 127, 128, 129, 1500], np.int32)
    n_nodes = np.array([1, 65, 8, 32, 31, 33, 64, 3, 65], np.int32)
    b = len(ctx)
    parent = np.full((b, N), -1, np.int32)
    for s in range(b):
        for n in range(1, int(n_nodes[s])):
            parent[s, n] = rng.integers(max(0, n - 5), n)
    att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)

    def dev(a):
        if how != "unaligned":
            return to_dev(a, dtype)
        flat = torch.zeros(a.size + 1, dtype=torch.float32, device="cuda")
        flat[1:] = to_dev(a, dtype).reshape(-1)
        return flat[1:].view(a.shape)

    kw = {"workspace": torch.empty(4, dtype=torch.uint8, device="cuda")} if how == "no_workspace" else {}
    print(f"attn f32 hq={hq} hkv={hkv} d={d} {how}", flush=True)
    out = P.presto_tree_attention(dev(att["q"]), dev(att["k_cache"]), dev(att["v_cache"]),
                                  to_dev(att["ctx_offsets"]), dev(att["k_tree"]), dev(att["v_tree"]),
                                  to_dev(anc), to_dev(n_nodes), int(ctx.max()), d ** -0.5, **kw)
    torch.cuda.synchronize()
    ref = oracle.tree_attention(dtype, att["q"], att["k_cache"], att["v_cache"], att["ctx_offsets"],
                                att["k_tree"], att["v_tree"], anc, n_nodes, d ** -0.5)
    got, reff = to_host(out).astype(np.float64), ref.astype(np.float64)
    for s in range(b):
        nn = int(n_nodes[s])
        # sums of up to 1565 fp32 terms and dot products of d terms, each
        # within about sqrt(d) 2^-24 of its magnitude: a few 1e-6
        assert _row_errors(got[s, :nn], reff[s, :nn]).max() <= 1e-5, s
        assert not got[s, nn:].any()


@pytest.mark.parametrize("hq,hkv,d,N", [(32, 8, 128, 65), (32, 8, 128, 68), (32, 8, 128, 69), (8, 2, 64, 129),
                                        (4, 2, 128, 136), (16, 2, 128, 34), (10, 2, 128, 52), (8, 2, 128, 257),
                                        (2, 2, 128, 257), (4, 2, 64, 1023)])
@pytest.mark.parametrize("b", [1, 3])
def test_attention_rows_past_a_full_tile(hq, hkv, d, N, b):
    """1 .. 16 query rows past a multiple of 256 (and just past 16, and with one
    head per KV head) in tiles of their own, which these short contexts get:
    whole trees, trees that end inside the last rows, at the full tile's edge
    and before it, contexts around a 64-key tile and a 16-key group, with one
    split and with many."""
    rng = np.random.default_rng([hq, hkv, d, N, b])
    G, dtype = hq // hkv, "bf16"
    full = (G * N // 256) * 256 // G  # nodes whose rows lie in full tiles
    over = min(full + 1, N)
    for ctx, live in (([0, 15, 16], [N, full, over]), ([4000, 65, 1], [over, N, 3]),
                      ([63, 130, 700], [N, N, full])):
        ctx, n_nodes = np.array(ctx[:b], np.int32), np.array(live[:b], np.int32)
        parent = np.full((b, N), -1, np.int32)
        for s in range(b):
            for n in range(1, int(n_nodes[s])):
                parent[s, n] = rng.integers(max(0, n - 9), n)
        att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)
        print(f"attn tail hq={hq} hkv={hkv} d={d} N={N} ctx={ctx.tolist()} live={n_nodes.tolist()}", flush=True)
        out = P.presto_tree_attention(
            to_dev(att["q"], dtype), to_dev(att["k_cache"], dtype), to_dev(att["v_cache"], dtype),
            to_dev(att["ctx_offsets"]), to_dev(att["k_tree"], dtype), to_dev(att["v_tree"], dtype),
            to_dev(anc), to_dev(n_nodes), int(ctx.max()), d ** -0.5)
        torch.cuda.synchronize()
        ref = oracle.tree_attention(dtype, att["q"], att["k_cache"], att["v_cache"], att["ctx_offsets"],
                                    att["k_tree"], att["v_tree"], anc, n_nodes, d ** -0.5)
        got = sy.as_f32(to_host(out), dtype).astype(np.float64)
        reff = sy.as_f32(ref, dtype).astype(np.float64)
        for s in range(b):
            nn = int(n_nodes[s])
            assert _row_errors(got[s, :nn], reff[s, :nn]).max() <= 2e-2, s
            assert not got[s, nn:].any()


@pytest.mark.parametrize("G,N", [(4, 33), (4, 69), (2, 40), (1, 300), (8, 16)])
def test_attention_padding_rows_without_a_merge(G, N):
    """Contexts short enough for one split: nobody but the attention kernel
    itself clears the rows of padding nodes, whichever 32-row block they
    start in (the waves of a row tile's dead blocks help with its last live
    one)."""
    rng = np.random.default_rng([G, N])
    hkv, d, dtype = 2, 128, "bf16"
    live = np.unique([1, 2, N // 4, N // 3, N // 2, N - 9, N - 1, N]).astype(np.int32)
    b = len(live)
    ctx = rng.integers(0, 40, b).astype(np.int32)
    parent = np.full((b, N), -1, np.int32)
    for s in range(b):
        for n in range(1, int(live[s])):
            parent[s, n] = rng.integers(max(0, n - 5), n)
    att, anc = _edge_inputs(rng, b, N, G * hkv, hkv, d, ctx, dtype, parent, live)
    out = torch.full((b, N, G * hkv, d), 7.0, dtype=torch.bfloat16, device="cuda")
    print(f"attn padding G={G} N={N} live={live.tolist()}", flush=True)
    P.presto_tree_attention(to_dev(att["q"], dtype), to_dev(att["k_cache"], dtype), to_dev(att["v_cache"], dtype),
                            to_dev(att["ctx_offsets"]), to_dev(att["k_tree"], dtype), to_dev(att["v_tree"], dtype),
                            to_dev(anc), to_dev(live), int(ctx.max()), d ** -0.5, out=out)
    torch.cuda.synchronize()
    ref = oracle.tree_attention(dtype, att["q"], att["k_cache"], att["v_cache"], att["ctx_offsets"],
                                att["k_tree"], att["v_tree"], anc, live, d ** -0.5)
    got = sy.as_f32(to_host(out), dtype).astype(np.float64)
    reff = sy.as_f32(ref, dtype).astype(np.float64)
    for s in range(b):
        assert _row_errors(got[s, :live[s]], reff[s, :live[s]]).max() <= 2e-2, s
        assert not got[s, live[s]:].any(), s


def _attend(att, anc, n_nodes, ctx, d, dtype, **kw):
    out = P.presto_tree_attention(
        to_dev(att["q"], dtype), to_dev(att["k_cache"], dtype), to_dev(att["v_cache"], dtype),
        to_dev(att["ctx_offsets"]), to_dev(att["k_tree"], dtype), to_dev(att["v_tree"], dtype),
        to_dev(anc), to_dev(n_nodes), int(ctx.max()), d ** -0.5, **kw)
    torch.cuda.synchronize()
    ref = oracle.tree_attention(dtype, att["q"], att["k_cache"], att["v_cache"], att["ctx_offsets"],
                                att["k_tree"], att["v_tree"], anc, n_nodes, d ** -0.5)
    return sy.as_f32(to_host(out), dtype).astype(np.float64), sy.as_f32(ref, dtype).astype(np.float64)


def _not_numbers(dtype, shape):
    """NaN and infinities of both signs, as storage values."""
    x = np.resize(np.array([np.nan, np.inf, -np.inf], np.float32), shape)
    return x if dtype == "f32" else (np.ascontiguousarray(x).view(np.uint32) >> 16).astype(np.uint16)


@pytest.mark.parametrize("dtype,hq,hkv,d,N,ctx", [
    ("f32", 4, 2, 128, 40, [0, 5, 20]), ("f32", 4, 2, 64, 40, [0, 5, 700]), ("f32", 32, 8, 128, 40, [0, 5, 1500]),
    ("bf16", 8, 2, 128, 40, [0, 5, 20]), ("bf16", 8, 2, 128, 65, [0, 5, 20]), ("bf16", 8, 2, 64, 68, [0, 5, 9000]),
    ("bf16", 8, 8, 128, 40, [0, 5, 4000])])
def test_attention_queries_that_are_not_numbers(dtype, hq, hkv, d, N, ctx):
    """A query of a padding node may hold anything (uninitialised memory): its
    row is zeros.  A live node's query that is NaN gives NaN in its own rows,
    and in no other, however the context is split and merged."""
    rng = np.random.default_rng([hq, hkv, d, N])
    ctx = np.array(ctx, np.int32)
    n_nodes = np.array([N - 3, 7, N], np.int32)
    b = len(ctx)
    parent = np.full((b, N), -1, np.int32)
    for s in range(b):
        for n in range(1, int(n_nodes[s])):
            parent[s, n] = rng.integers(max(0, n - 5), n)
    att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)
    for s in range(b):
        nn = int(n_nodes[s])
        att["q"][s, nn:] = _not_numbers(dtype, att["q"][s, nn:].shape)
        att["q"][s, 1] = _not_numbers(dtype, (1,))[0]
        att["q"][s, nn - 1] = _not_numbers(dtype, (1,))[0]
    print(f"attn NaN queries {dtype} hq={hq} hkv={hkv} d={d} N={N} ctx={ctx.tolist()}", flush=True)
    kw = {"workspace": torch.empty(4, dtype=torch.uint8, device="cuda")} if dtype == "f32" and N == 40 and d == 64 else {}
    got, ref = _attend(att, anc, n_nodes, ctx, d, dtype, **kw)
    tol = 2e-2 if dtype == "bf16" else 1e-5
    for s in range(b):
        nn = int(n_nodes[s])
        bad = [1, nn - 1]
        good = [n for n in range(nn) if n not in bad]
        assert (got[s, nn:] == 0).all(), s
        assert np.isnan(got[s, bad]).all(), s
        assert _row_errors(got[s, good], ref[s, good]).max() <= tol, s


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 128), (6, 2, 64), (32, 8, 128)])
@pytest.mark.parametrize("split", [True, False])
def test_attention_f32_branches_are_isolated(hq, hkv, d, split):
    """fp32: a tree node whose K or V is not a number reaches its descendants
    only; every other row is what it would be without it."""
    rng = np.random.default_rng([hq, hkv, d])
    N, dtype = 70, "f32"
    ctx = np.array([0, 31, 64, 1300], np.int32)
    n_nodes = np.array([70, 40, 69, 70], np.int32)
    b = len(ctx)
    parent = np.full((b, N), -1, np.int32)
    for s in range(b):
        for n in range(1, int(n_nodes[s])):
            parent[s, n] = (n - 1) // 3
    att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)
    for s in range(b):
        for n in (5, 33, int(n_nodes[s]) - 1):
            att["v_tree"][s, n, :, n % 7::9] = _not_numbers(dtype, (hkv, len(range(n % 7, d, 9))))
        att["k_tree"][s, 11, :, 3] = np.nan
    print(f"attn f32 isolation hq={hq} hkv={hkv} d={d} split={split}", flush=True)
    kw = {} if split else {"workspace": torch.empty(4, dtype=torch.uint8, device="cuda")}
    got, ref = _attend(att, anc, n_nodes, ctx, d, dtype, **kw)
    for s in range(b):
        nn = int(n_nodes[s])
        fin = np.isfinite(ref[s, :nn])
        np.testing.assert_array_equal(np.isfinite(got[s, :nn]), fin, err_msg=str(s))
        assert not fin.all() and fin.any()
        # the errors of the numbers alone, against their rows' size
        assert _row_errors(np.where(fin, got[s, :nn], 0), np.where(fin, ref[s, :nn], 0)).max() <= 1e-5, s
        assert not got[s, nn:].any()


@pytest.mark.parametrize("hq,hkv,d,N,b,max_ctx,total", [
    (8, 2, 128, 129, 17, 4000, 27200),   # shares: three balanced row tiles, 42 shares
    (16, 16, 64, 257, 12, 8000, 28800),  # shares: one head per KV head, a second tile of one row
    (8, 8, 128, 257, 40, 2000, 40000),   # shares: several short sequences in each
    (4, 4, 64, 300, 9, 8000, 28800),     # shares: two tiles of 160 rows
    (16, 2, 128, 130, 9, 8000, 28800),   # shares: eight heads per KV head, five tiles
    (12, 6, 64, 600, 8, 20000, 96000),  # shares: two rounds of full tiles
    (8, 2, 128, 129, 9, 1500, 5400),     # pairs
    (4, 4, 64, 300, 9, 1500, 5400),      # pairs
    (16, 2, 128, 130, 5, 4000, 8000),    # pairs
    (8, 2, 64, 65, 70, 4000, 28),        # pairs: more sequences than a wave has lanes
    (8, 2, 128, 129, 5, 300, 600),       # the longest context's grid
    (8, 4, 64, 129, 6, 1500, 3600),      # pairs: two heads per KV head, a second tile of two rows
    (16, 2, 128, 130, 17, 300, 2040),    # unsplit
])
def test_attention_ragged_schedules(hq, hkv, d, N, b, max_ctx, total):
    """The schedules of a ragged batch with a total-context hint, with several
    row tiles per KV head: trees whose live rows end in the first tile (dead
    tiles), in a later one and at a tile's last row, empty and one-key
    contexts beside long ones, and bounds and hints far from the contexts (a
    hint only schedules), so that shares end among a sequence's first tiles."""
    rng = np.random.default_rng([hq, hkv, d, N, b])
    G, dtype = hq // hkv, "bf16"
    ctx = rng.integers(0, 250, b).astype(np.int32)
    ctx[:3] = [0, 1, min(max_ctx, 900)]
    n_nodes = rng.integers(1, N + 1, b).astype(np.int32)
    n_nodes[:4] = [N, 2, N, min(N, 256 // G)]
    parent = np.full((b, N), -1, np.int32)
    for s in range(b):
        for n in range(1, int(n_nodes[s])):
            parent[s, n] = rng.integers(max(0, n - 7), n)
    att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)
    print(f"attn schedules hq={hq} hkv={hkv} d={d} N={N} b={b} max_ctx={max_ctx} total={total}", flush=True)
    outs = [torch.full((b, N, hq, d), x, dtype=torch.bfloat16, device="cuda") for x in (7.0, -3.0)]
    for out in outs:
        P.presto_tree_attention(
            to_dev(att["q"], dtype), to_dev(att["k_cache"], dtype), to_dev(att["v_cache"], dtype),
            to_dev(att["ctx_offsets"]), to_dev(att["k_tree"], dtype), to_dev(att["v_tree"], dtype),
            to_dev(anc), to_dev(n_nodes), max_ctx, d ** -0.5, total_ctx=total, out=out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))  # bit for bit
    ref = oracle.tree_attention(dtype, att["q"], att["k_cache"], att["v_cache"], att["ctx_offsets"],
                                att["k_tree"], att["v_tree"], anc, n_nodes, d ** -0.5)
    got = sy.as_f32(to_host(out), dtype).astype(np.float64)
    reff = sy.as_f32(ref, dtype).astype(np.float64)
    for s in range(b):
        nn = int(n_nodes[s])
        assert _row_errors(got[s, :nn], reff[s, :nn]).max() <= 2e-2, s
        assert not got[s, nn:].any(), s


@pytest.mark.parametrize("hq,hkv,d,N,b,max_ctx,split_len", [
    (32, 8, 128, 65, 3, 60000, 6016),   # four rows past a full tile
    (32, 8, 128, 68, 3, 60000, 6016),   # sixteen
    (8, 2, 64, 129, 3, 60000, 2880),    # the second of two full tiles takes them
    (4, 2, 128, 136, 3, 60000, 1472),   # two heads per KV head
    (16, 2, 128, 34, 3, 60000, 1472),   # eight
    (10, 2, 128, 52, 3, 60000, 1472),   # five: a node on both sides of the tile's edge
    (8, 2, 128, 257, 3, 60000, 6080),   # five ancestor words
    (8, 2, 128, 129, 64, 100, 0),       # not split
    (32, 8, 64, 65, 32, 200, 0),        # not split
])
def test_attention_rows_that_ride_along(hq, hkv, d, N, b, max_ctx, split_len):
    """1 .. 16 query rows past a multiple of 256 that the last full tile takes
    along (long or many sequences; a bound on the context far above the
    contexts gives the long ones' plan): whole trees, trees that end inside the
    tail's rows, at the tile's edge and before it; contexts around a 64-key
    tile, a 16-key group and a split's end, with one part and with several."""
    rng = np.random.default_rng([hq, hkv, d, N, b])
    G, dtype = hq // hkv, "bf16"
    full = (G * N // 256) * 256 // G  # nodes whose rows lie in full tiles
    over = min(full + 1, N)
    if split_len:
        sets = [([0, 15, 16], [N, full, over]), ([split_len + 70, 65, 1], [over, N, 3]),
                ([2 * split_len - 20, split_len - N, split_len - 1], [N, N, N])]
    else:
        sets = [(rng.integers(0, max_ctx, b), rng.choice([N, N, N, full, over, over - 1, 1, N // 2], b))]
    for ctx, live in sets:
        ctx, n_nodes = np.array(ctx, np.int32), np.array(live, np.int32)
        parent = np.full((b, N), -1, np.int32)
        for s in range(b):
            for n in range(1, int(n_nodes[s])):
                parent[s, n] = rng.integers(max(0, n - 9), n)
        att, anc = _edge_inputs(rng, b, N, hq, hkv, d, ctx, dtype, parent, n_nodes)
        for s in range(b):  # queries of padding nodes are whatever memory held
            att["q"][s, n_nodes[s]:] = _not_numbers(dtype, att["q"][s, n_nodes[s]:].shape)
        print(f"attn along hq={hq} hkv={hkv} d={d} N={N} b={b} ctx={ctx[:3].tolist()} live={n_nodes[:3].tolist()}",
              flush=True)
        outs = [torch.full((b, N, hq, d), x, dtype=torch.bfloat16, device="cuda") for x in (7.0, -3.0)]
        for out in outs:
            P.presto_tree_attention(
                to_dev(att["q"], dtype), to_dev(att["k_cache"], dtype), to_dev(att["v_cache"], dtype),
                to_dev(att["ctx_offsets"]), to_dev(att["k_tree"], dtype), to_dev(att["v_tree"], dtype),
                to_dev(anc), to_dev(n_nodes), max_ctx, d ** -0.5, out=out)
        torch.cuda.synchronize()
        assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))  # bit for bit
        ref = oracle.tree_attention(dtype, att["q"], att["k_cache"], att["v_cache"], att["ctx_offsets"],
                                    att["k_tree"], att["v_tree"], anc, n_nodes, d ** -0.5)
        got = sy.as_f32(to_host(out), dtype).astype(np.float64)
        reff = sy.as_f32(ref, dtype).astype(np.float64)
        for s in range(b):
            nn = int(n_nodes[s])
            assert _row_errors(got[s, :nn], reff[s, :nn]).max() <= 2e-2, s
            assert (got[s, nn:] == 0).all(), s
