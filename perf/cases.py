"""Timed cases of tree attention: the calls a training or serving program makes.

A case names an entry point ("kind"), the heads, head dimension and dtype, and
the range its document pages are drawn from.  A page is the packed sample
``[prefix | layout stream | content branches]``; its structure is drawn from
the case's own ``tree`` number, the tensors' values from the seed.

    forward   tree_attn_fwd on packed K/V, every token a query
    backward  tree_attn_bwd of that forward
    decode    one decode step over a paged cache, its schedule copied by the
              call (branch_decode) or resident in the workspace
              (branch_decode_resident)
    session   content streams opened, prefilled in one step and closed
    relayout  cache_from_rows: row-layout blocks into the paged layouts
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_06146_amd as pa

DEVICE = "cuda"
BLOCK = 16


def _case(name, kind, hq, hkv, d, dtype, pages, prefix, stream, branches, length, tree=0, **more):
    """``prefix``, ``stream`` and ``branches`` are (low, high) bounds;
    ``length`` = (low, high) draws branch lengths uniformly, (low, high,
    median) from a lognormal distribution (sigma 0.5) clipped to them."""
    c = {"name": name, "kind": kind, "hq": hq, "hkv": hkv, "d": d, "dtype": dtype, "pages": pages,
         "prefix_lo": prefix[0], "prefix_hi": prefix[1], "stream_lo": stream[0], "stream_hi": stream[1],
         "branch_lo": branches[0], "branch_hi": branches[1], "len_lo": length[0], "len_hi": length[1],
         "len_median": length[2] if len(length) > 2 else 0, "tree": tree}
    c.update(more)
    return c


def listed():
    return [
        # A unit-sized page in fp32, as a numerics check or a debug run calls it: latency and one launch.
        _case("forward_tiny_f32", "forward", 4, 1, 64, "f32", 1, (256, 256), (64, 64), (4, 4), (32, 32)),
        # One page's sample on its own: branch creation while serving, or a training micro-batch of one.
        _case("forward_page_bf16", "forward", 16, 2, 128, "bf16", 1, (1537, 1537), (203, 203), (21, 21), (4, 1024, 80)),
        # A training micro-batch: eight ragged pages packed without padding (43k tokens).
        _case("forward_8pages_bf16", "forward", 16, 2, 128, "bf16", 8, (1024, 4096), (128, 512), (8, 48), (4, 1024, 80)),
        # A micro-batch of a model with 64-wide heads, seven query heads per KV head.
        _case("forward_4pages_d64", "forward", 28, 4, 64, "bf16", 4, (1024, 4096), (128, 512), (8, 48), (4, 1024, 80)),
        # The gradients of the two bf16 forwards above.
        _case("backward_page_bf16", "backward", 16, 2, 128, "bf16", 1, (1537, 1537), (203, 203), (21, 21), (4, 1024, 80)),
        _case("backward_8pages_bf16", "backward", 16, 2, 128, "bf16", 8, (1024, 4096), (128, 512), (8, 48), (4, 1024, 80)),
        # One page being decoded by itself: a step is a chain of latencies.
        _case("decode_page_bf16", "decode", 16, 2, 128, "bf16", 1, (2048, 2048), (256, 256), (16, 16), (16, 256), resident=False, new=0),
        # A full serving batch: 64 pages, every branch one token; the schedule is uploaded once for all layers.
        _case("decode_64pages_bf16", "decode", 16, 2, 128, "bf16", 64, (3072, 3072), (256, 256), (24, 24), (1, 1024), resident=True, new=0),
        # A dense page in the middle of decoding: 96 live branches and 32 just opened ones of 8 tokens.
        _case("decode_dense_mixed", "decode", 28, 4, 128, "bf16", 1, (8192, 8192), (1024, 1024), (96, 96), (64, 2048), resident=False, new=32),
        # A step of a few pages held in fp32, as a precision check of a served model runs it.
        _case("decode_4pages_f32", "decode", 16, 2, 128, "f32", 4, (1024, 1024), (128, 128), (16, 16), (16, 256), resident=False, new=0),
        # The step driver when layout streams close regions: new content streams prefill their first 8 tokens.
        _case("session_forks_bf16", "session", 16, 2, 128, "bf16", 8, (1024, 1024), (256, 256), (8, 8), (8, 8)),
        # A row-layout cache of 262k tokens taken over.
        {"name": "relayout_bf16", "kind": "relayout", "hkv": 2, "d": 128, "dtype": "bf16", "blocks": 16384},
    ]


def _spread(rng, lo, hi):
    """A whole number, even over the logarithm of lo .. hi."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)) - 0.5 / hi))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "backward", "backward", "decode", "decode", "decode", "session", "relayout"])
    hq, hkv = rng.choice([(16, 2), (16, 2), (28, 4), (4, 1)])
    d = rng.choice([64, 128, 128])
    tree = rng.randrange(1 << 30)
    if kind == "relayout":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        return {"kind": kind, "hkv": hkv, "d": d, "dtype": dtype, "blocks": _spread(rng, 16, 16384)}
    if kind in ("forward", "backward"):
        f32 = kind == "forward" and rng.random() < 0.3
        pages = 1 if f32 else _spread(rng, 1, 8)
        p = _spread(rng, 256, 1024 if f32 else 3072)
        s = _spread(rng, 32, 384)
        n = _spread(rng, 4, 16 if f32 else 40)
        c = _case("", kind, hq, hkv, d, "f32" if f32 else "bf16", pages, (max(1, p * 2 // 3), p * 4 // 3), (max(1, s * 2 // 3), s * 4 // 3),
                  (max(1, n * 2 // 3), n * 4 // 3), (4, 1024, _spread(rng, 30, 120)), tree)
        while c["pages"] > 1 and work(c)["flops"] > 4e11 * (2 if kind == "backward" else 1):
            c["pages"] -= 1
    elif kind == "session":
        c = _case("", kind, hq, hkv, d, "bf16", _spread(rng, 1, 16), (256, _spread(rng, 256, 2048)), (64, 256), (2, _spread(rng, 2, 16)), (1, 8), tree)
    else:
        f32 = rng.random() < 0.25
        p = _spread(rng, 256, 1024 if f32 else 8192)
        n = _spread(rng, 2, 16 if f32 else 96)
        c = _case("", kind, hq, hkv, d, "f32" if f32 else "bf16", _spread(rng, 1, 4 if f32 else 48), (max(1, p * 3 // 4), p), (64, _spread(rng, 64, 128 if f32 else 1024)),
                  (max(1, n // 2), n), (1, _spread(rng, 16, 256 if f32 else 2048)), tree, resident=rng.random() < 0.5, new=rng.choice([0, 0, 0, n // 3]))
        while c["pages"] > 1 and work(c)["bytes"] > 9e8:
            c["pages"] -= 1
    del c["name"]
    return c


# ------------------------------------------------------------------ structure

def _pages(case):
    """The case's pages: dicts of prefix, stream and branch lengths."""
    rng = np.random.default_rng([case["tree"], 1])
    between = lambda lo, hi: int(rng.integers(lo, hi + 1))  # noqa: E731
    decode = case["kind"] == "decode"
    pages = []
    for _ in range(case["pages"]):
        P, S, N = (between(case[k + "_lo"], case[k + "_hi"]) for k in ("prefix", "stream", "branch"))
        new = case.get("new", 0)  # branches opened in this step: 8 tokens, all of them queries
        fork = np.sort(rng.integers(1, S if decode else S + 1, size=N + new))
        if case["len_median"]:
            L = rng.lognormal(math.log(case["len_median"]), 0.5, size=N)
            L = np.clip(np.rint(L), case["len_lo"], case["len_hi"]).astype(np.int64)
        else:
            L = rng.integers(case["len_lo"], case["len_hi"] + 1, size=N)
        L = [int(x) for x in L] + [8] * new
        q = [1] * N + [8] * new if decode else L
        pages.append({"prefix_len": P, "prefix_q": 0 if decode else P, "stream_len": S, "stream_q": 1 if decode else S,
                      "branches": [{"fork": int(f), "length": n, "q_len": m} for f, n, m in zip(fork, L, q)]})
    return pages


def _segments(pages):
    """(length, queries, [(first K/V row of an ancestor, rows seen)], own first row, first query row) of every segment in packed order."""
    out, kv, q = [], 0, 0
    for pg in pages:
        prefix = kv
        out.append((pg["prefix_len"], pg["prefix_q"], [], kv, q))
        kv, q = kv + pg["prefix_len"], q + pg["prefix_q"]
        stream = kv
        out.append((pg["stream_len"], pg["stream_q"], [(prefix, pg["prefix_len"])], kv, q))
        kv, q = kv + pg["stream_len"], q + pg["stream_q"]
        for b in pg["branches"]:
            out.append((b["length"], b["q_len"], [(prefix, pg["prefix_len"]), (stream, b["fork"])], kv, q))
            kv, q = kv + b["length"], q + b["q_len"]
    return out, kv, q


def _esize(case):
    return 2 if case["dtype"] == "bf16" else 4


def work(case):
    """Every K/V row, query and output once; flops of the products over the visible (query, key) pairs."""
    es = _esize(case)
    if case["kind"] == "relayout":
        return {"bytes": 4 * case["blocks"] * case["hkv"] * BLOCK * case["d"] * es, "flops": 0}
    pages = _pages(case)
    segs, T, nq = _segments(pages)
    new_rows = 0
    pairs = 0
    if case["kind"] == "session":  # only the new streams' tokens query; their rows are read and written to the cache
        segs = [s for s in segs if len(s[2]) == 2]
        nq = new_rows = sum(s[0] for s in segs)
    for n, m, anc, _, _ in segs:
        pairs += m * sum(a[1] for a in anc) + m * (n - m) + m * (m + 1) // 2
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    kv = 2 * T * hkv * d * es
    qo = nq * hq * d * es
    if case["kind"] == "backward":  # reads q, k, v, o, dout, lse; writes dq, dk, dv
        return {"bytes": 2 * kv + 4 * qo + nq * hq * 4, "flops": 10 * d * hq * pairs}
    return {"bytes": kv + 2 * qo + nq * hq * 4 + 4 * new_rows * hkv * d * es, "flops": 4 * d * hq * pairs}


def tolerance(case):
    """About four times the largest error against 64 bits: 4.7e-7 in fp32 (the decode step), 2.5e-3 in bf16 (probabilities and outputs rounded to it)."""
    if case["kind"] == "relayout":
        return "exact"
    return {"rel": 2e-6 if case["dtype"] == "f32" else 1e-2}


# ------------------------------------------------------------------ values

def _normal(shape, seed, stream, case):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed * 1000003 + stream)
    x = torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32)
    return x.to(torch.bfloat16) if case["dtype"] == "bf16" else x


def _packed_inputs(case, seed):
    _, T, nq = _segments(_pages(case))
    q = _normal((nq, case["hq"], case["d"]), seed, 1, case)
    k = _normal((T, case["hkv"], case["d"]), seed, 2, case)
    v = _normal((T, case["hkv"], case["d"]), seed, 3, case)
    return q, k, v


def _step_queries(n, case, seed, stream):
    """The first n rows of a step's query buffer, which has room for a few streams more."""
    return _normal((n + 16, case["hq"], case["d"]), seed, stream, case)[:n]


def _paged_inputs(case, seed):
    """Queries, the two caches (blocks in drawn places of a pool a quarter larger) and the block table."""
    segs, _, nq = _segments(_pages(case))
    need = sum(-(-s[0] // BLOCK) for s in segs)
    pool = need + need // 4 + 8
    q = _step_queries(nq, case, seed, 1)
    kc = _normal((pool, case["hkv"], case["d"] // 8, BLOCK, 8), seed, 2, case)
    vc = _normal((pool, case["hkv"], case["d"], BLOCK), seed, 3, case)
    table = np.random.default_rng([seed, 4]).permutation(pool)[:need].astype(np.int32)
    return q, kc, vc, table


def _aligned_bytes(n):
    raw = torch.empty(n + 256, dtype=torch.uint8, device=DEVICE)
    at = (-raw.data_ptr()) % 256
    return raw[at:at + n]


def _session_inputs(case, seed):
    """K/V of the prefixes and streams (packed, pages in turn), and the new streams' queries and K/V."""
    segs, _, _ = _segments(_pages(case))
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    old = sum(s[0] for s in segs if len(s[2]) < 2)
    new = sum(s[0] for s in segs if len(s[2]) == 2)
    return {"k_old": _normal((old, hkv, d), seed, 1, case), "v_old": _normal((old, hkv, d), seed, 2, case),
            "q": _step_queries(new, case, seed, 3), "k_new": _normal((new, hkv, d), seed, 4, case),
            "v_new": _normal((new, hkv, d), seed, 5, case)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "relayout":
        shape = (case["blocks"], case["hkv"], BLOCK, case["d"])
        return {"kind": kind, "k": _normal(shape, seed, 1, case), "v": _normal(shape, seed, 2, case)}
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    pages = _pages(case)
    if kind in ("forward", "backward"):
        q, k, v = _packed_inputs(case, seed)
        plan = pa.TreePlan(pa.segments_from_pages(pages, 0), hq, hkv, d, case["dtype"], 0, num_kv_rows=k.shape[0], num_q_rows=q.shape[0])
        st = {"kind": kind, "plan": plan, "q": q, "k": k, "v": v}
        if kind == "backward":
            st["o"], st["lse"] = pa.tree_attn_fwd(q, k, v, plan)
            st["dout"] = _normal(q.shape, seed, 4, case)
        return st
    if kind == "decode":
        q, kc, vc, table = _paged_inputs(case, seed)
        plan = pa.TreePlan(pa.segments_from_pages(pages, BLOCK), hq, hkv, d, case["dtype"], BLOCK, num_kv_rows=kc.shape[0], num_q_rows=q.shape[0],
                           block_table_host=table)
        st = {"kind": kind, "plan": plan, "q": q, "k": kc, "v": vc, "table": torch.from_numpy(table).to(DEVICE), "resident": case["resident"],
              "o": torch.empty_like(q), "lse": torch.empty(q.shape[:2], dtype=torch.float32, device=DEVICE), "ws": _aligned_bytes(plan.workspace_bytes)}
        if case["resident"]:
            pa.plan_upload(plan, st["ws"])
        return st
    # session: the pages' prefixes and layout streams are cached and the streams open
    x = _session_inputs(case, seed)
    lens = [(pg["prefix_len"], pg["stream_len"]) for pg in pages]
    n_new = [b["length"] for pg in pages for b in pg["branches"]]
    blocks = sum(-(-n // BLOCK) for pair in lens for n in pair) + sum(-(-n // BLOCK) for n in n_new) + 8
    kc = torch.zeros((blocks, hkv, d // 8, BLOCK, 8), dtype=x["q"].dtype, device=DEVICE)
    vc = torch.zeros((blocks, hkv, d, BLOCK), dtype=x["q"].dtype, device=DEVICE)
    table = torch.zeros(4 * blocks + 1024, dtype=torch.int32, device=DEVICE)
    ses = pa.DecodeSession(hq, hkv, d, blocks, case["dtype"], kc, vc, table)
    roots = [ses.open() for _ in pages]
    at = np.cumsum([0] + [n for pair in lens for n in pair])
    rows = lambda which: torch.cat([torch.arange(at[2 * i + which], at[2 * i + which + 1]) for i in range(len(lens))]).to(DEVICE)  # noqa: E731
    pr, sr = rows(0), rows(1)
    ses.step(None, x["k_old"][pr], x["v_old"][pr], [a for a, _ in lens], [0] * len(lens))
    streams = [ses.open(r, a) for r, (a, _) in zip(roots, lens)]
    for r in roots:
        ses.close(r)
    ses.step(None, x["k_old"][sr], x["v_old"][sr], [b for _, b in lens], [0] * len(lens))
    zero = np.zeros(len(lens), np.int32)
    count = np.concatenate([zero, np.asarray(n_new, np.int32)])
    opens = [(s, b["fork"]) for s, pg in zip(streams, pages) for b in pg["branches"]]
    return {"kind": kind, "session": ses, "opens": opens, "count": count, "q": x["q"], "k": x["k_new"], "v": x["v_new"]}


def run(st):
    kind = st["kind"]
    if kind == "forward":
        return pa.tree_attn_fwd(st["q"], st["k"], st["v"], st["plan"])
    if kind == "backward":
        return pa.tree_attn_bwd(st["q"], st["k"], st["v"], st["o"], st["lse"], st["dout"], st["plan"])
    if kind == "decode":
        call = pa.branch_decode_resident if st["resident"] else pa.branch_decode
        return call(st["q"], st["k"], st["v"], st["table"], st["plan"], st["o"], st["lse"], st["ws"])
    if kind == "relayout":
        return pa.cache_from_rows(st["k"], st["v"])
    ses = st["session"]
    ids = [ses.open(s, f) for s, f in st["opens"]]
    out = ses.step(st["q"], st["k"], st["v"], st["count"], st["count"])
    for i in ids:
        ses.close(i)
    return out


# ------------------------------------------------------------------ 64 bits

def _attend(segs, q, k, v, d, grad=None):
    """Attention of every segment's queries in float64; q [nq, Hkv, G, d], k and v [T, Hkv, d].  With grad = (o, dout): dq, dk, dv."""
    scale = 1.0 / math.sqrt(d)
    hkv, G = q.shape[1], q.shape[2]
    if grad is None:
        o = torch.empty_like(q)
        lse = torch.empty(q.shape[:3], dtype=torch.float64, device=q.device)
    else:
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        D = (grad[0] * grad[1]).sum(-1)
    for n, m, anc, own, q0 in segs:
        spans = [(a, a + c) for a, c in anc] + [(own, own + n)]
        kk = torch.cat([k[a:b] for a, b in spans])
        vv = torch.cat([v[a:b] for a, b in spans])
        seen = kk.shape[0] - m  # keys that the first query sees, less its own
        for c0 in range(0, m, 512):
            c1 = min(m, c0 + 512)
            last = seen + torch.arange(c0, c1, device=q.device)
            hidden = (torch.arange(kk.shape[0], device=q.device)[None, :] > last[:, None]).repeat_interleave(G, 0)
            for h in range(hkv):
                qq = q[q0 + c0:q0 + c1, h].reshape(-1, d)
                s = (qq @ kk[:, h].t().contiguous() * scale).masked_fill_(hidden, -math.inf)
                ls = torch.logsumexp(s, 1)
                p = torch.exp_(s.sub_(ls[:, None]))
                if grad is None:
                    o[q0 + c0:q0 + c1, h] = (p @ vv[:, h].contiguous()).reshape(-1, G, d)
                    lse[q0 + c0:q0 + c1, h] = ls.reshape(-1, G)
                    continue
                g = grad[1][q0 + c0:q0 + c1, h].reshape(-1, d)
                pv = p.t().contiguous() @ g
                ds = p * (g @ vv[:, h].t().contiguous() - D[q0 + c0:q0 + c1, h].reshape(-1, 1))
                dq[q0 + c0:q0 + c1, h] = (ds @ kk[:, h].contiguous() * scale).reshape(-1, G, d)
                pk = ds.t().contiguous() @ qq * scale
                at = 0
                for a, b in spans:
                    dv[a:b, h] += pv[at:at + b - a]
                    dk[a:b, h] += pk[at:at + b - a]
                    at += b - a
    return (o, lse) if grad is None else (dq, dk, dv)


def _kslot(t):
    return (t & 3) | ((t & 4) << 1) | ((t & 8) >> 1)


def exact(case, seed):
    kind = case["kind"]
    hkv, d = case["hkv"], case["d"]
    slot = [_kslot(t) for t in range(BLOCK)]
    if kind == "relayout":
        st = prepare(case, seed)
        k = st["k"].reshape(-1, hkv, BLOCK, d // 8, 8).permute(0, 1, 3, 2, 4)[:, :, :, slot]  # kslot is its own inverse
        return k.contiguous(), st["v"].transpose(2, 3).contiguous()
    segs, T, nq = _segments(_pages(case))
    if kind in ("forward", "backward"):
        q, k, v = (x.double() for x in _packed_inputs(case, seed))
    elif kind == "decode":
        q, kc, vc, table = _paged_inputs(case, seed)
        ids = torch.from_numpy(table).to(DEVICE).long()
        k = kc[ids][:, :, :, slot].permute(0, 3, 1, 2, 4).reshape(-1, hkv, d).double()
        v = vc[ids].permute(0, 3, 1, 2).reshape(-1, hkv, d).double()
        q = q.double()
        keep = torch.cat([torch.arange(-(-s[0] // BLOCK) * BLOCK) < s[0] for s in segs]).to(DEVICE)
        k, v = k[keep], v[keep]
    else:
        x = _session_inputs(case, seed)
        k = torch.empty((T, hkv, d), dtype=torch.float64, device=DEVICE)
        v = torch.empty_like(k)
        old = new = 0
        some = []
        for n, m, anc, own, _ in segs:
            src, at = ("old", old) if len(anc) < 2 else ("new", new)
            k[own:own + n] = x["k_" + src][at:at + n].double()
            v[own:own + n] = x["v_" + src][at:at + n].double()
            if src == "old":
                old += n
            else:
                some.append((n, m, anc, own, new))
                new += n
        segs, q = some, x["q"].double()
    q4 = q.reshape(q.shape[0], hkv, -1, d)
    if kind != "backward":
        o, lse = _attend(segs, q4, k, v, d)
        return o.reshape(q.shape), lse.reshape(q.shape[:2])
    dout = _normal(q.shape, seed, 4, case).double().reshape(q4.shape)
    o, _ = _attend(segs, q4, k, v, d)
    o = o.to(torch.bfloat16).double()  # the backward takes the forward's stored output
    dq, dk, dv = _attend(segs, q4, k, v, d, grad=(o, dout))
    return dq.reshape(q.shape), dk, dv
