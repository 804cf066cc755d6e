"""The work whose speed is measured: the framework's public calls over the sizes they serve.

Four families, each through the entry points of ``paper_2606_00487_amd``:

* ``round``   one decoding round of a request batch: selection, tree attention, acceptance
  walk and KV commit;
* ``select``  the selection alone (vocabulary scan, scores, budgeted tree), per scorer;
* ``attn``    the tree-masked verification attention alone (contiguous or paged cache);
* ``layer``   one attention layer of the target over the trees (contiguous or paged cache).

Marginals follow the workload recipe of this repository: Gaussian logits with one planted
spike per row that fades with depth.  Queries, cache rows and hidden states are N(0, 1).
Context lengths of a batch are spread over [ctx_lo, ctx_hi] on a log scale; the seed orders
them.  ``exact`` follows the calls' definitions (include/taps.h) in plain 64-bit torch.
"""
from __future__ import annotations

import heapq
import math
import random

import torch

import paper_2606_00487_amd as taps

SCORERS = {"sibling": taps.SIBLING, "marginal": taps.MARGINAL, "learned": taps.LEARNED}
EMB, HIDDEN = 16, 32          # the learned scorer's embedding and hidden sizes
LAMBDA1, LAMBDA2 = 1.0, 0.125


# ------------------------------------------------------------------------------ the cases
def _round(batch, block, vocab, K, budget, Hq, Hkv, hd, ctx_lo, ctx_hi, dtype, **kw):
    return dict(op="round", batch=batch, block=block, vocab=vocab, K=K, budget=budget, Hq=Hq,
                Hkv=Hkv, hd=hd, ctx_lo=ctx_lo, ctx_hi=ctx_hi, dtype=dtype, scorer="sibling", **kw)


def _select(batch, block, vocab, K, budget, dtype, scorer, **kw):
    return dict(op="select", batch=batch, block=block, vocab=vocab, K=K, budget=budget,
                dtype=dtype, scorer=scorer, **kw)


def _attn(batch, budget, Hq, Hkv, hd, ctx_lo, ctx_hi, dtype, page_rows=0, **kw):
    return dict(op="attn", batch=batch, budget=budget, Hq=Hq, Hkv=Hkv, hd=hd, ctx_lo=ctx_lo,
                ctx_hi=ctx_hi, dtype=dtype, page_rows=page_rows, **kw)


def _layer(batch, budget, Hq, Hkv, hidden, ctx_lo, ctx_hi, page_rows=0, **kw):
    return dict(op="layer", batch=batch, budget=budget, Hq=Hq, Hkv=Hkv, hd=128, hidden=hidden,
                ctx_lo=ctx_lo, ctx_hi=ctx_hi, dtype="bf16", page_rows=page_rows, **kw)


def listed():
    return [
        # the smallest round: a toy vocabulary, fp32 probabilities and an fp32 cache (latency)
        _round(1, 8, 1000, 4, 16, 4, 2, 64, 256, 256, "fp32", name="round_tiny_fp32"),
        # the headline round: one request of the Qwen3-8B shape at 8K context (latency)
        _round(1, 16, 151936, 8, 64, 32, 8, 128, 8192, 8192, "bf16", name="round_qwen3_8b"),
        # batched serving: the selection of 16 requests over the full vocabulary
        _select(16, 16, 151936, 8, 128, "bf16", "sibling", name="select_serve16"),
        # a trained scorer in front of the selection, one request (compute per edge)
        _select(1, 16, 151936, 8, 64, "bf16", "learned", name="select_learned"),
        # the scoring ablation over fp32 logits and a vocabulary of odd length (rows that are
        # not 16-byte aligned)
        _select(4, 8, 50257, 8, 64, "fp32", "marginal", name="select_marginal_odd"),
        # batched serving: 16 requests of very different lengths
        _attn(16, 128, 32, 8, 128, 512, 16384, "bf16", name="attn_serve16"),
        # long contexts and large trees over a paged cache (the largest attention)
        _attn(4, 256, 32, 8, 128, 32768, 32768, "bf16", 128, name="attn_stress_paged"),
        # a model with head_dim 64, a small batch
        _attn(4, 64, 32, 8, 64, 2048, 8192, "bf16", name="attn_hd64"),
        # full precision: an fp32 cache, one request
        _attn(1, 32, 32, 8, 128, 2048, 2048, "fp32", name="attn_fp32"),
        # the layer of the Qwen3-8B shape for one request (bound by reading the weights)
        _layer(1, 64, 32, 8, 4096, 8192, 8192, name="layer_qwen3_8b"),
        # the same layer for 16 requests (bound by the matrix products)
        _layer(16, 128, 32, 8, 4096, 512, 16384, name="layer_serve16"),
        # the Qwen3-4B layer shape, four requests, an odd budget, a paged cache
        _layer(4, 99, 32, 8, 2560, 700, 6000, 64, name="layer_mid_paged"),
    ]


HEADS = [(32, 8), (16, 8), (8, 8), (40, 8), (64, 8), (16, 2), (4, 2)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = {"flops": 5.5e11, "bytes": 5.4e8}   # those of the largest listed case
    while True:
        op = rng.choice(["round", "select", "select", "attn", "attn", "attn", "layer", "layer"])
        batch = _log(rng, 1, 16)
        Hq, Hkv = rng.choice(HEADS)
        hi = _log(rng, 200, 32768)
        lo = _log(rng, min(128, hi), hi)
        budget = _log(rng, 12, 384)
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        if op in ("round", "select"):
            scorer = rng.choice(["sibling", "sibling", "marginal", "learned"])
            K = rng.choice([4, 6, 8, 8, 16])
            block = rng.randrange(6, 25 if K < 16 else 17)
            vocab = rng.choice([151936, _log(rng, 1000, 160000)])
            case = (_select(batch, block, vocab, K, budget, dtype, scorer) if op == "select" else
                    _round(batch, block, vocab, K, min(budget, 128), Hq, Hkv,
                           rng.choice([64, 128]), lo, min(hi, 8192), dtype))
            case["ctx_lo"] = min(lo, 8192) if op == "round" else 0
        elif op == "attn":
            paged = rng.random() < 0.35
            case = _attn(batch, budget, Hq, Hkv, 128 if paged else rng.choice([64, 128, 128]),
                         lo, hi, "bf16" if paged else dtype,
                         rng.choice([32, 64, 128, 256]) if paged else 0)
        else:
            case = _layer(batch, budget, Hq, Hkv, 64 * rng.randrange(8, 81), lo, min(hi, 16384),
                          rng.choice([0, 0, 64, 128]))
            case["ctx_lo"] = min(lo, 16384)
        if op == "select":
            del case["ctx_lo"]
        w = work(case)
        # an fp32 product costs far more than a bf16 one: at most the listed fp32 attention's
        scale = 500 if case["dtype"] == "fp32" and op != "select" else 1
        if w["flops"] * scale <= most["flops"] and w["bytes"] <= most["bytes"]:
            return case


# ------------------------------------------------------------------------------ inputs
def _ctx_lens(case):
    """The batch's context lengths, spread over [ctx_lo, ctx_hi] on a log scale."""
    B, lo, hi = case["batch"], case["ctx_lo"], case["ctx_hi"]
    return [int(round(lo * (hi / lo) ** ((b + 0.5) / B))) for b in range(B)]


def _tdt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _bf(case):
    return taps.BF16 if case["dtype"] == "bf16" else taps.FP32


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(g, *shape, dtype=torch.float32, scale=None):
    x = torch.randn(*shape, generator=g, device="cuda", dtype=dtype)
    return x if scale is None else x.mul_(scale)


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


def _is_probs(case):
    # fp32 rounds take probabilities, everything else logits
    return case["op"] == "round" and case["dtype"] == "fp32"


def _marginals(case, g, r):
    B, D, V = case["batch"], case["block"], case["vocab"]
    x = _randn(g, B, D, V)
    if not _is_probs(case):
        x.mul_(3.0)
    t = torch.arange(D, device="cuda", dtype=torch.float32) / max(1, D - 1)
    spike = torch.full_like(t, 4.0) if _is_probs(case) else 8.0 - 6.0 * t
    at = torch.tensor([[r.randrange(V) for _ in range(D)] for _ in range(B)], device="cuda")
    x.scatter_add_(2, at[..., None], spike.expand(B, D)[..., None].contiguous())
    if _is_probs(case):
        x = torch.softmax(x, dim=-1)
    return x.to(_tdt(case))


def _mlp(case, g, r):
    if case.get("scorer") != "learned":
        return None
    F = 2 * EMB + 3
    return taps.ScorerWeights(
        emb=_randn(g, case["vocab"], EMB, scale=0.5), W1=_randn(g, HIDDEN, F, scale=F ** -0.5),
        b1=_randn(g, HIDDEN, scale=0.1), w2=_randn(g, HIDDEN, scale=HIDDEN ** -0.5), b2=0.05,
        root_token=_i32([r.randrange(case["vocab"]) for _ in range(case["batch"])]))


def _random_tree(n, r):
    """Parents of a draft tree of n nodes in breadth-first order, and the depths."""
    parent, depth = [-1], [0]
    w = max(4, n // 6)
    for i in range(1, n):
        p = i - 1 - r.randrange(min(i, w))
        parent.append(max(p, parent[-1], 0))
        depth.append(depth[parent[-1]] + 1)
    return parent, depth


def _trees(case, r):
    """Full trees of the batch as device arrays (a TreeBuffers whose other fields are empty)."""
    B, N = case["batch"], case["budget"]
    made = [_random_tree(N, r) for _ in range(B)]
    t = taps.TreeBuffers.empty(B, 1, 1, N)
    t.parent.copy_(_i32([m[0] for m in made]))
    t.depth.copy_(_i32([m[1] for m in made]))
    t.n_nodes.fill_(N)
    return t


def _cache(case, g, r, state):
    """K and V with room for every request's context and nodes, contiguous or in pages."""
    ctx = _ctx_lens(case)
    r.shuffle(ctx)
    rows = [c + case["budget"] for c in ctx]
    state.update(ctx=_i32(ctx), ctx_host=ctx)
    dt, hv = _tdt(case), (case["Hkv"], case["hd"])
    pr = case.get("page_rows", 0)
    if not pr:
        offs = [0]
        for x in rows[:-1]:
            offs.append(offs[-1] + x)
        state["off"] = torch.tensor(offs, dtype=torch.int64, device="cuda")
        state["off_host"] = offs
        shape = (sum(rows), *hv)
    else:
        need = [-(-x // pr) for x in rows]
        ids = list(range(sum(need)))
        r.shuffle(ids)
        table = [[0] * -(-(case["ctx_hi"] + case["budget"]) // pr) for _ in rows]
        for b, m in enumerate(need):
            for j in range(m):
                table[b][j] = ids.pop()
        state["table"] = _i32(table)
        shape = (sum(need), pr, *hv)
    state["K"], state["V"] = _randn(g, *shape, dtype=dt), _randn(g, *shape, dtype=dt)


def prepare(case, seed):
    g, r = _gen(seed), random.Random(seed)
    c, op = case, case["op"]
    s = {"case": dict(case), "seed": seed}
    B, N = c["batch"], c["budget"]
    if op in ("round", "select"):
        s["marg"] = _marginals(c, g, r)
        s["mlp"] = _mlp(c, g, r)
        s["sel"] = taps.Selector(B, c["block"], c["vocab"], c["K"], N, dtype=_bf(c),
                                 kind=taps.PROBS if _is_probs(c) else taps.LOGITS,
                                 lambda1=LAMBDA1, lambda2=LAMBDA2, scorer=SCORERS[c["scorer"]],
                                 mlp=s["mlp"])
    if op != "select":
        _cache(c, g, r, s)
    if op in ("round", "attn"):
        s["Q"] = _randn(g, B, N, c["Hq"], c["hd"], dtype=_tdt(c))
        s["O"] = torch.zeros_like(s["Q"])
        if c.get("page_rows"):
            s["att"] = taps.PagedTreeAttention(B, N, c["Hq"], c["Hkv"], c["ctx_hi"], c["page_rows"])
        else:
            s["att"] = taps.TreeAttention(B, N, c["Hq"], c["Hkv"], c["hd"], c["ctx_hi"],
                                          dtype=_bf(c))
    if op in ("attn", "layer"):
        s["tree"] = _trees(c, r)
    if op == "round":
        # the target's greedy token after each node: mostly a drafted child's token
        s["plain"] = _plain_select(c, s)
        s["target"] = _i32([_targets(t, N, c["vocab"], r) for t in s["plain"]])
        s["walk"] = taps.AcceptWalk(B, N, c["block"])
        s["commit"] = taps.KVCommit(B, N, c["block"], c["Hkv"], c["hd"], c["ctx_hi"], dtype=_bf(c))
    if op == "layer":
        H, nq, nk = c["hidden"], c["Hq"] * c["hd"], c["Hkv"] * c["hd"]
        b16 = dict(dtype=torch.bfloat16)
        s["X"] = _randn(g, B, N, H, **b16)
        s["w"] = taps.LayerWeights(
            _randn(g, nq, H, scale=H ** -0.5, **b16), _randn(g, nk, H, scale=H ** -0.5, **b16),
            _randn(g, nk, H, scale=H ** -0.5, **b16), _randn(g, H, nq, scale=nq ** -0.5, **b16),
            _randn(g, c["hd"], scale=0.1, **b16).add_(1.0), _randn(g, c["hd"], scale=0.1, **b16).add_(1.0))
        if c["page_rows"]:
            s["lay"] = taps.PagedVerifyLayer(B, N, c["Hq"], c["Hkv"], c["hd"], H, c["ctx_hi"],
                                             c["page_rows"])
        else:
            s["lay"] = taps.VerifyLayer(B, N, c["Hq"], c["Hkv"], c["hd"], H, c["ctx_hi"])
    return s


# ------------------------------------------------------------------------------ one pass
def _tree_out(t):
    return {"parent": t.parent, "token": t.token, "depth": t.depth, "rank": t.rank,
            "q_reach": t.q_reach, "n_nodes": t.n_nodes, "topk_idx": t.topk_idx,
            "topk_val": t.topk_val}


def run(s):
    c, op = s["case"], s["case"]["op"]
    if op == "select":
        return _tree_out(s["sel"](s["marg"]))
    if op == "round":
        tree = s["sel"](s["marg"])
        O = s["att"](s["Q"], s["K"], s["V"], s["off"], s["ctx"], tree.parent, tree.n_nodes,
                     out=s["O"])
        path, plen, bonus = s["walk"](tree, s["target"])
        new_ctx, tokens, n = s["commit"](s["K"], s["V"], s["off"], s["ctx"], tree, path, plen,
                                         bonus)
        return {**_tree_out(tree), "O": O, "path": path, "path_len": plen, "bonus": bonus,
                "new_ctx": new_ctx, "tokens": tokens, "n": n, "K": s["K"], "V": s["V"]}
    where = (s["table"],) if c["page_rows"] else (s["off"],)
    if op == "attn":
        return {"O": s["att"](s["Q"], s["K"], s["V"], *where, s["ctx"], s["tree"].parent,
                              s["tree"].n_nodes, out=s["O"])}
    Y = s["lay"](s["X"], s["w"], s["K"], s["V"], *where, s["ctx"], s["tree"])
    return {"Y": Y, "K": s["K"], "V": s["V"]}


def work(case):
    c, op = case, case["op"]
    B, N = c["batch"], c["budget"]
    es = 2 if c["dtype"] == "bf16" else 4
    by = fl = 0
    if op in ("round", "select"):
        el = B * c["block"] * c["vocab"]
        by += el * es + B * N * 24
        fl += el
    if op != "select":
        ctx = _ctx_lens(c)
        row = c["Hkv"] * c["hd"] * es
        by += sum(x + N for x in ctx) * row * 2
        fl += sum(4 * N * c["Hq"] * c["hd"] * (x + 1) for x in ctx)
        if op == "layer":   # queries and attention outputs need not leave the chip
            H, nq, nk = c["hidden"], c["Hq"] * c["hd"], c["Hkv"] * c["hd"]
            by += 2 * H * (2 * nq + 2 * nk) + 2 * 2 * B * N * H
            fl += 2 * B * N * H * (2 * nq + 2 * nk)
        else:
            by += 2 * B * N * c["Hq"] * c["hd"] * es
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # the selection is defined bit for bit in 64-bit arithmetic with stated tie breaks
    if case["op"] == "select":
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 4e-6}
    # bf16 outputs (half an ulp: 1.7e-3 rms) of bf16 weights, queries and probabilities
    return {"rel": 1e-2}


# ------------------------------------------------------------------------------ 64 bits
def _edge_tables(c, x, idx, val, mlp, b):
    """q_cond[i][parent rank][child rank] of one request (nested lists; one parent row where
    the parent does not matter)."""
    D = c["block"]
    if c["scorer"] == "marginal":
        return [[row] for row in torch.softmax(x, -1).gather(1, idx).tolist()]
    if c["scorer"] == "sibling":
        e = val if _is_probs(c) else torch.exp(val - val[:, :1])
        return [[row] for row in (e / e.sum(-1, keepdim=True)).tolist()]
    M = x.max(-1, keepdim=True).values
    t = torch.exp(x - M)
    Z = t.sum(-1, keepdim=True)
    logz = torch.log(Z)
    ent = logz - (t * (x - M)).sum(-1, keepdim=True) / Z
    emb = mlp.emb.double()
    tables = []
    for i in range(D):
        child = emb[idx[i]]
        par = emb[mlp.root_token[b].long()][None] if i == 0 else emb[idx[i - 1]]
        P, K = par.shape[0], child.shape[0]
        f = torch.cat([par[:, None].expand(P, K, -1), child[None].expand(P, K, -1),
                       torch.full((P, K, 1), i + 1.0, dtype=torch.float64, device=x.device),
                       (val[i] - M[i] - logz[i])[None, :, None].expand(P, K, 1),
                       ent[i].expand(P, K, 1)], -1)
        a = torch.relu(f @ mlp.W1.double().T.contiguous() + mlp.b1.double())
        tables.append(torch.softmax(a @ mlp.w2.double(), -1).tolist())   # b2 cancels
    return tables


def _plain_select(c, s):
    """The selected tree of every request: dicts of lists in breadth-first order."""
    out = []
    K, D, N = c["K"], c["block"], c["budget"]
    for b in range(c["batch"]):
        x = s["marg"][b].double()
        top = torch.sort(x, dim=-1, descending=True, stable=True)
        idx, val = top.indices[:, :K].contiguous(), top.values[:, :K].contiguous()
        q = _edge_tables(c, x, idx, val, s["mlp"], b)
        tok = idx.tolist()
        chosen = {(): 1.0}
        heap = []

        def push(path, reach):
            i = len(path)
            if i == D:
                return
            row = q[i][path[-1] if path and len(q[i]) > 1 else 0]
            for k in range(K):
                u = reach * row[k] / (LAMBDA1 + LAMBDA2 * (i + 1))
                if u > 0:
                    heapq.heappush(heap, (-u, i + 1, path + (k,), reach * row[k]))

        push((), 1.0)
        while heap and len(chosen) < N:
            _, _, path, reach = heapq.heappop(heap)
            chosen[path] = reach
            push(path, reach)
        order = sorted(chosen, key=lambda p: (len(p), p))
        at = {p: i for i, p in enumerate(order)}
        out.append({"parent": [at[p[:-1]] if p else -1 for p in order],
                    "token": [tok[len(p) - 1][p[-1]] if p else -1 for p in order],
                    "q_reach": [chosen[p] for p in order], "topk_val": val})
    return out


def _targets(t, N, vocab, r):
    kids = {}
    for i, p in enumerate(t["parent"]):
        kids.setdefault(p, []).append(i)
    pick = [t["token"][kids[i][0]] if i in kids and r.random() < 0.7 else r.randrange(vocab)
            for i in range(len(t["parent"]))]
    return pick + [-1] * (N - len(pick))


def _walked(t, target):
    path = [0]
    while True:
        nxt = [i for i, p in enumerate(t["parent"])
               if p == path[-1] and t["token"][i] == target[path[-1]]]
        if not nxt:
            return path
        path.append(nxt[0])


def _logical(case, s, x, b):
    """Request b's cache rows (context, then nodes) as [rows][Hkv][hd]."""
    n = s["ctx_host"][b] + case["budget"]
    if case.get("page_rows"):
        pages = x[s["table"][b].long()]
        return pages.reshape(-1, *pages.shape[2:])[:n]
    return x[s["off_host"][b]:s["off_host"][b] + n]


def _plain_attention(q, k, v, ctx, parent, G):
    """q [n][Hq][hd], k and v [ctx + n ..][Hkv][hd], 64 bits."""
    n, Hq, hd = q.shape
    see = torch.zeros(n, ctx + n, dtype=torch.bool)
    see[:, :ctx] = True
    for i in range(n):
        if parent[i] >= 0:
            see[i, ctx:] = see[parent[i], ctx:]
        see[i, ctx + i] = True
    see = see.repeat_interleave(G, 0).to(q.device)
    out = torch.empty_like(q)
    for g in range(Hq // G):
        qg = q[:, g * G:(g + 1) * G].reshape(n * G, hd).contiguous()
        kt = k[:ctx + n, g].T.contiguous()
        sc = (qg @ kt).mul_(hd ** -0.5).masked_fill_(~see, -math.inf)
        o = torch.softmax(sc, -1) @ v[:ctx + n, g].contiguous()
        out[:, g * G:(g + 1) * G] = o.reshape(n, G, hd)
    return out


def _rope(x, pos, theta):
    hd = x.shape[-1]
    j = torch.arange(hd // 2, dtype=torch.float64, device=x.device)
    ang = pos[:, None, None].double() * theta ** (-2.0 * j / hd)
    a, b = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _norm(x, w, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * w.double()


def _exact_tree(c, plain):
    N, dev = c["budget"], "cuda"
    q = torch.zeros(c["batch"], N, dtype=torch.float64, device=dev)
    for b, t in enumerate(plain):
        q[b, :len(t["q_reach"])] = torch.tensor(t["q_reach"], dtype=torch.float64)
    out = dict.fromkeys(("parent", "token", "depth", "rank", "n_nodes", "topk_idx"))
    return {**out, "q_reach": q, "topk_val": torch.stack([t["topk_val"] for t in plain])}


def exact(case, seed):
    c, op = case, case["op"]
    s = prepare(case, seed)
    if op == "select":
        return _exact_tree(c, _plain_select(c, s))
    G = c["Hq"] // c["Hkv"]
    if op == "layer":
        w, B, N = s["w"], c["batch"], c["budget"]
        K, V = s["K"].double(), s["V"].double()
        Y = torch.empty(B, N, c["hidden"], dtype=torch.float64, device="cuda")
        for b in range(B):
            x, ctx = s["X"][b].double(), s["ctx_host"][b]
            pos = ctx + s["tree"].depth[b]
            q, k, v = ((x @ m.double().T.contiguous()).reshape(N, -1, c["hd"])
                       for m in (w.Wq, w.Wk, w.Wv))
            q = _rope(_norm(q, w.q_norm, w.norm_eps), pos, w.rope_theta)
            k = _rope(_norm(k, w.k_norm, w.norm_eps), pos, w.rope_theta)
            if c["page_rows"]:
                at = ctx + torch.arange(N, device="cuda")
                page, slot = s["table"][b].long()[at // c["page_rows"]], at % c["page_rows"]
                K[page, slot], V[page, slot] = k, v
            else:
                r0 = s["off_host"][b] + ctx
                K[r0:r0 + N], V[r0:r0 + N] = k, v
            o = _plain_attention(q, _logical(c, s, K, b), _logical(c, s, V, b), ctx,
                                 s["tree"].parent[b].tolist(), G)
            Y[b] = o.reshape(N, -1) @ w.Wo.double().T.contiguous()
        return {"Y": Y, "K": K, "V": V}
    plain = s.get("plain")
    O = torch.zeros(s["Q"].shape, dtype=torch.float64, device="cuda")
    for b in range(c["batch"]):
        parent = plain[b]["parent"] if plain else s["tree"].parent[b].tolist()
        n = len(parent)
        O[b, :n] = _plain_attention(s["Q"][b, :n].double(), _logical(c, s, s["K"], b).double(),
                                    _logical(c, s, s["V"], b).double(), s["ctx_host"][b], parent, G)
    if op == "attn":
        return {"O": O}
    K, V = s["K"].double(), s["V"].double()
    for b, t in enumerate(plain):
        r0 = s["off_host"][b] + s["ctx_host"][b]
        path = _walked(t, s["target"][b].tolist())
        for x in (K, V):
            x[r0:r0 + len(path)] = x[[r0 + i for i in path]]
    none = dict.fromkeys(("path", "path_len", "bonus", "new_ctx", "tokens", "n"))
    return {**_exact_tree(c, plain), **none, "O": O, "K": K, "V": V}
