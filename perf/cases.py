"""Performance cases of the trie decoder: what a program that decodes with it asks of it.

Kinds of case (``case["kind"]``):

* ``request``: a whole request batch from its prompt: ``init_prompt``, then ``steps``
  decode steps (attention of every layer, then the fused selection and append), the
  selection applied, as Alg 2's loop does.
* ``attend``: the attention of one decode step over a trie in the middle of a run (a trie
  loaded from a saved state, every leaf's K/V stored).
* ``select``: the log-softmax and top-b alone (the entry without a context, or a
  context's).
* ``tree``: multi-query tree attention: the prefill of a stored trie (every node a query)
  or the verification of the newest nodes as drafts.
* ``batch``: the batch-based beam search baseline, whole requests.

``calls`` says how a program issues the attention: "layer" is one call per layer, as a
model interleaves it with its other work; "all" is one call over every layer.  K, V and Q
are N(0, 1) and logits N(0, 3^2), the distributions of this repository's workloads.
"""
from __future__ import annotations

import math

import numpy as np
import torch

LOGIT_STD = 3.0


# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------
def _case(kind, layers, q_heads, kv_heads, head_dim, beams, prompt, dtype="bf16", **kw):
    c = dict(kind=kind, tries=1, layers=layers, q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim,
             dtype=dtype, beams=beams, prompt=prompt, prompt_min=prompt, window=0, gc=1, calls="all")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest request a program makes: one fp32 layer, a short prompt (latency and launches)
        _case("request", 1, 4, 4, 64, 3, 32, "f32", name="tiny_request", vocab=1000, steps=8, eos=-1),
        # the headline decode: Llama-3.1-8B shape, one call for all layers
        _case("request", 32, 32, 8, 128, 8, 2048, name="llama_request", vocab=128256, steps=6, eos=-1),
        # the same shape as a model issues it, one call per layer, 64 steps into a run
        _case("attend", 32, 32, 8, 128, 8, 2048, name="llama_layers", steps=64, calls="layer"),
        # multi-head attention at head_dim 96, an end-of-sequence token
        _case("request", 32, 32, 32, 96, 4, 1024, name="phi_request", vocab=32064, steps=6, eos=32000),
        # a long prompt under a sliding window
        _case("request", 40, 32, 8, 128, 8, 8192, name="mistral_request", vocab=131072, steps=4, eos=-1, window=4096),
        # a serving batch: 16 requests of ragged length, 16 beams each
        _case("request", 32, 32, 8, 128, 16, 1024, name="batch16_request", tries=16, prompt_min=256,
              vocab=128256, steps=3, eos=-1),
        # many beams (four 32-row blocks per KV head), collections every 15 positions, 600 steps in
        _case("attend", 32, 32, 8, 128, 30, 2048, name="beams30_layers", steps=600, gc=15, calls="layer"),
        # the selection of a serving batch by the entry that needs no context
        dict(kind="select", name="select_batch16", entry="static", tries=16, beams=16, vocab=128256, eos=-1),
        # prefill: every node of a stored trie is a query, one call per layer
        _case("tree", 32, 32, 8, 128, 8, 2048, name="prefill_layers", steps=16, queries=2048 + 48, calls="layer"),
        # verification of draft nodes: the newest 24 nodes are the queries
        _case("tree", 32, 32, 8, 128, 8, 2048, name="drafts_layers", steps=32, queries=24, calls="layer"),
        # fp32 storage (and, drawn, the head sizes beyond the bf16 matrix-core ones)
        _case("attend", 8, 32, 8, 128, 8, 2048, "f32", name="f32_attend", steps=32),
        # the baseline: every beam owns its cache, copied at each step
        _case("batch", 32, 32, 8, 128, 8, 1024, name="batch_baseline", vocab=128256, steps=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng):
    kv = rng.choice([1, 2, 4, 8, 16, 32])
    group = rng.choice([g for g in (1, 2, 3, 4, 7, 8) if g * kv <= 64])
    return kv * group, kv


def draw(rng):
    kind = rng.choice(["request", "request", "attend", "attend", "select", "tree", "batch"])
    if kind == "select":
        beams, vocab = _log_int(rng, 1, 48), _log_int(rng, 1000, 131072)
        most = max(1, 8192 // (beams * ((vocab + 4095) // 4096)))
        return dict(kind=kind, entry=rng.choice(["static", "context"]), tries=_log_int(rng, 1, min(32, most)),
                    beams=beams, vocab=vocab, eos=-1)
    q_heads, kv_heads = _heads(rng)
    mfma_only = kind == "tree"
    dtype = "bf16" if mfma_only or rng.random() < 0.75 else "f32"
    head_dim = rng.choice([64, 96, 128] if mfma_only or rng.random() < 0.8 else [32, 160, 192, 256])
    beams = _log_int(rng, 1, 32)
    prompt = _log_int(rng, 17, 6000)
    tries = _log_int(rng, 1, 12)
    layers = _log_int(rng, 1, 32)
    # the K/V of one pass bounded below the largest listed case
    row = 4 * kv_heads * head_dim * (2 if dtype == "f32" else 1)
    budget = 1.2e9 if kind in ("request", "attend") and dtype == "bf16" and head_dim in (64, 96, 128) else 2.5e8
    if kind == "batch":
        row, budget = row * beams * 3, 4e9
    layers = max(1, min(layers, int(budget / (row * prompt * tries))))
    if row * prompt * tries * layers > budget:
        tries = 1
        prompt = max(17, min(prompt, int(budget / (row * layers))))
    c = _case(kind, layers, q_heads, kv_heads, head_dim, beams, prompt, dtype, tries=tries,
              prompt_min=max(9, int(prompt * rng.choice([1.0, 1.0, 0.3]))), calls=rng.choice(["layer", "all"]),
              window=rng.choice([0, 0, 0, max(8, prompt // 2 + rng.randrange(9))]))
    if kind in ("request", "batch"):
        c["steps"] = rng.randrange(2, 4)
        c["vocab"] = min(_log_int(rng, 1000, 131072), 4096 * (2000 // beams), 60_000_000 // (beams * tries))
    else:
        c["steps"] = _log_int(rng, 4, 300)
    if kind == "request":
        c["eos"] = rng.choice([-1, -1, c["vocab"] // 3])
    if kind in ("request", "attend"):
        c["gc"] = rng.choice([1, 1, 4, 15])
    if kind == "tree":
        full = prompt + rng.randrange(1, 64)
        c["queries"] = rng.choice([full, full, _log_int(rng, 1, 48)])
        flops = 4.0 * head_dim * q_heads * layers * tries * c["queries"] * prompt / 2
        c["layers"] = max(1, min(layers, int(layers * 1.0e12 / max(flops, 1.0))))
    return c


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _lengths(c):
    """Prompt lengths of the tries: spread evenly over [prompt_min, prompt]."""
    return [int(x) for x in np.linspace(c["prompt"], c["prompt_min"], c["tries"])]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(gen, shape, dtype=torch.float32, std=1.0):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def _grown(rng, c, prompt):
    """The trie of one request after ``steps`` decode steps: b children per step, the parent
    of rank r drawn with weight 1/(r+1), dead and evicted nodes collected at the positions
    that are multiples of ``gc``.  Returns it in the layout of td_state."""
    b, steps, window, g = c["beams"], c["steps"], c["window"], c["gc"]
    weight = 1.0 / (np.arange(b) + 1.0)
    parent, depth = list(range(-1, prompt - 1)), list(range(prompt))
    leaves = [prompt - 1]
    collected, from_node, evicted = None, 0, -1
    for s in range(steps):
        w = weight[:len(leaves)]
        ranks = rng.choice(len(leaves), size=b, p=w / w.sum())
        first = len(parent)
        parent += [leaves[r] for r in ranks]
        depth += [prompt + s] * b
        leaves = list(range(first, first + b))
        if (prompt + s + 1) % g == 0:
            collected, from_node, evicted = leaves, first + b, prompt + s - window if window else -1
    keep = np.zeros(len(parent), bool)
    keep[from_node:] = True
    for leaf in collected if collected is not None else []:
        n = leaf
        while n >= 0 and not keep[n]:
            keep[n] = True
            n = parent[n]
    depth = np.array(depth, np.int32)
    keep &= depth > evicted
    old = np.nonzero(keep)[0]
    slot = np.full(len(parent) + 1, -1, np.int32)  # (the last entry: the parent of a root)
    slot[old] = np.arange(len(old))
    bits = [(1 << b) - 1] * prompt + [0] * (len(parent) - prompt)  # (the prompt is on every path)
    for i, leaf in enumerate(leaves):
        n = leaf
        while n >= prompt:
            bits[n] |= 1 << i
            n = parent[n]
    mask = np.array(bits, np.uint64)
    n = len(old)
    return dict(n_nodes=n, n_live=b, next_id=len(parent), kv_pending=0, step=steps, node_id=old.astype(np.int32),
                parent_slot=slot[np.array(parent)[old]], token=rng.integers(0, 1000, n).astype(np.int32),
                depth=depth[old], mask=mask[old], leaf_slot=np.arange(n - b, n, dtype=np.int32),
                leaf_score=-np.sort(rng.random(b) * 8.0 + 20.0).astype(np.float32))


def _attn_inputs(c, gen, rows, steps=None):
    """q / k_new / v_new of the layout of trie_attn_decode, for ``rows`` query owners per trie."""
    lead = () if steps is None else (steps,)
    L, T, dt = c["layers"], c["tries"], _dtype(c)
    q = _normal(gen, lead + (L, T, rows, c["q_heads"], c["head_dim"]), dt)
    if steps is None:
        return q, None, None
    kv = lead + (L, T, rows, c["kv_heads"], c["head_dim"])
    return q, _normal(gen, kv, dt), _normal(gen, kv, dt)


def _inputs(c, seed):
    """Every input of the case, from the seed alone."""
    gen, rng, kind = _gen(seed), np.random.default_rng(seed), c["kind"]
    T, b = c["tries"], c["beams"]
    x = {}
    if kind == "select":
        x["logits"] = _normal(gen, (T, b, c["vocab"]), std=LOGIT_STD)
        x["score"] = torch.from_numpy(-np.sort(rng.random((T, b)) * 8.0 + 20.0).astype(np.float32)).cuda()
        return x
    L, dt = c["layers"], _dtype(c)
    x["lengths"] = _lengths(c)
    if kind in ("request", "batch"):
        slots = max(x["lengths"])
        x["tokens"] = torch.from_numpy(rng.integers(0, c["vocab"], (T, slots)).astype(np.int32)).cuda()
        x["q"], x["k_new"], x["v_new"] = _attn_inputs(c, gen, b, c["steps"])
        x["logits"] = _normal(gen, (c["steps"], T, b, c["vocab"]), std=LOGIT_STD)
        if c.get("eos", -1) >= 0:
            x["logits"][..., c["eos"]] += 10.0  # (an end of sequence that ranks now and then)
    else:
        x["tries"] = [_grown(rng, c, n) for n in x["lengths"]]
        slots = max(t["n_nodes"] for t in x["tries"])
        rows = b
        if kind == "tree":
            rows = c["queries"]
            qs = np.full((T, rows), -1, np.int32)
            for t, s in enumerate(x["tries"]):
                n = min(rows, s["n_nodes"])
                qs[t, :n] = np.arange(s["n_nodes"] - n, s["n_nodes"])
            x["qslots"] = torch.from_numpy(qs).cuda()
        x["q"] = _attn_inputs(c, gen, rows)[0]
    x["k"] = _normal(gen, (T, L, c["kv_heads"], slots, c["head_dim"]), dt)
    x["v"] = _normal(gen, (T, L, c["kv_heads"], slots, c["head_dim"]), dt)
    return x


def _selection(T, b, steps=()):
    i32, f32 = dict(dtype=torch.int32, device="cuda"), dict(dtype=torch.float32, device="cuda")
    s = tuple(steps) + (T, b)
    return dict(sel_parent=torch.zeros(s, **i32), sel_token=torch.zeros(s, **i32), sel_score=torch.zeros(s, **f32),
                sel_logprob=torch.zeros(s, **f32), lse=torch.zeros(s, **f32))


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------
def prepare(case, seed):
    import paper_2502_00085_amd.binding as B
    c, x = case, _inputs(case, seed)
    kind, T, b = c["kind"], c["tries"], c["beams"]
    st = dict(case=c, x=x)
    if kind == "select":
        st["sel"] = _selection(T, b)
        st["n_live"] = torch.full((T,), b, dtype=torch.int32, device="cuda")
        if c["entry"] == "context":
            dec = B.TrieDecoder(T, b, 8 + 2 * b, c["vocab"], 1, 1, 1, 32, eos_token=c["eos"])
            rng = np.random.default_rng(seed)
            for t in range(T):
                s = _grown(rng, dict(beams=b, steps=1, window=0, gc=1), 8)
                s["leaf_score"] = x["score"][t].cpu().numpy()
                dec.load_state(t, s)
            st["dec"] = dec
        return st
    L, Hq, Hkv, D = c["layers"], c["q_heads"], c["kv_heads"], c["head_dim"]
    slots = x["k"].shape[3]
    st["scale"] = 1.0 / math.sqrt(D)
    if kind == "batch":
        dec = B.BatchBeamDecoder(T, b, slots + c["steps"] + 1, c["vocab"], L, Hq, Hkv, D, c["window"], c["dtype"])
        for pool, rows in zip(dec.prompt_cache(), (x.pop("k"), x.pop("v"))):
            pool[:, 0, :, :, :slots].copy_(rows)
    else:
        # (a request's pool never has to be re-packed, which would move its prompt's rows)
        room = (c["steps"] + c["gc"]) * b if kind == "request" else b
        dec = B.TrieDecoder(T, b, slots + room + b, c.get("vocab", 1000), L, Hq, Hkv, D, c["window"], c["dtype"],
                            gc_interval=c["gc"], eos_token=c.get("eos", -1))
        for pool, rows in ((dec.k_pool, x.pop("k")), (dec.v_pool, x.pop("v"))):
            pool[:, :, :, :slots].copy_(rows)
    st["dec"] = dec
    st["out"] = torch.zeros_like(x["q"])
    if kind in ("request", "batch"):
        st["sel"] = _selection(T, b, (c["steps"],))
    else:
        for t, s in enumerate(x["tries"]):
            dec.load_state(t, s)
    return st


def _attention(st, q, k_new, v_new, out):
    c, dec = st["case"], st["dec"]
    if c["calls"] == "all":
        dec.attn_decode(0, c["layers"], q, k_new, v_new, out, st["scale"])
        return
    for l in range(c["layers"]):
        dec.attn_decode(l, 1, q[l], None if k_new is None else k_new[l], None if v_new is None else v_new[l], out[l],
                        st["scale"])


def run(state):
    st, c, x = state, state["case"], state["x"]
    kind, dec, sel = c["kind"], st.get("dec"), st.get("sel")
    if kind == "select":
        if c["entry"] == "static":
            import paper_2502_00085_amd.binding as B
            B.beam_topk_static(c["tries"], c["beams"], c["vocab"], x["logits"], st["n_live"], x["score"],
                               sel["sel_parent"], sel["sel_token"], sel["sel_score"], sel["sel_logprob"], sel["lse"])
        else:
            dec.logsoftmax_topk(x["logits"], sel["sel_parent"], sel["sel_token"], sel["sel_score"],
                                sel["sel_logprob"], sel["lse"])
        return sel
    if kind == "attend":
        _attention(st, x["q"], None, None, st["out"])
        return st["out"]
    if kind == "tree":
        if c["calls"] == "all":
            dec.tree_attn(0, c["layers"], x["qslots"], x["q"], st["out"], st["scale"])
        else:
            for l in range(c["layers"]):
                dec.tree_attn(l, 1, x["qslots"], x["q"][l], st["out"][l], st["scale"])
        return st["out"]
    dec.init_prompt(x["lengths"], x["tokens"])
    for s in range(c["steps"]):
        new = s > 0
        _attention(st, x["q"][s], x["k_new"][s] if new else None, x["v_new"][s] if new else None, st["out"][s])
        pick = [sel[k][s] for k in ("sel_parent", "sel_token", "sel_score", "sel_logprob", "lse")]
        if kind == "batch":
            dec.logsoftmax_topk(x["logits"][s], *pick)
            dec.reorder(*pick[:3])
        else:
            dec.topk_append(x["logits"][s], *pick)
    res = dict(sel, out=st["out"])
    if c.get("eos", -1) >= 0:  # the finished hypotheses, best first, in arrays of one size
        for name, dt in (("norm", np.float32), ("score", np.float32), ("step", np.int32), ("parent", np.int32)):
            res["finished_" + name] = np.zeros((c["tries"], c["beams"]), dt)
        for t in range(c["tries"]):
            f = dec.read_finished(t)
            for name in ("norm", "score", "step", "parent"):
                res["finished_" + name][t, :f["count"]] = f[name]
    return res


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without, and how exact its outputs are
# ---------------------------------------------------------------------------------------------
def work(case):
    c = case
    T, b = c["tries"], c["beams"]
    if c["kind"] == "select":
        return {"bytes": 4.0 * T * b * (c["vocab"] + 6), "flops": 3.0 * T * b * c["vocab"]}
    L, Hq, Hkv, D, W = c["layers"], c["q_heads"], c["kv_heads"], c["head_dim"], c["window"]
    esz = 4 if c["dtype"] == "f32" else 2
    row, qrow = 2.0 * L * Hkv * D * esz, L * Hq * D * esz  # K+V of a node; q of a query, all layers
    seen = lambda n: min(n, W) if W else n  # noqa: E731
    by = fl = 0.0
    for P in _lengths(c):
        if c["kind"] == "tree":
            n = P + c["beams"]
            q = min(c["queries"], n)
            by += row * min(n, q + seen(n)) + 2 * qrow * q
            fl += 4.0 * D * Hq * L * sum(seen(i + 1) for i in range(n - q, n))
        elif c["kind"] == "attend":
            n = P + c["steps"]
            by += row * (seen(n) + b - 1) + 2 * qrow * b
            fl += 4.0 * D * Hq * L * b * seen(n)
        else:
            for s in range(c["steps"]):
                live = b if s else 1
                if c["kind"] == "batch":
                    # every beam reads its own cache; the reorder reads and writes every new beam's
                    by += row * live * seen(P + s) + 2 * row * b * (P + s)
                else:
                    by += row * (seen(P + s) + live - 1)
                by += 2 * qrow * live + (2 * row * live if s else 0) + 4.0 * live * c["vocab"]
                fl += 4.0 * D * Hq * L * live * seen(P + s)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # bf16 outputs and probabilities: 8 bits of mantissa (2e-3 against 64 bits, measured);
    # fp32 ones and the scores: sums in another order (3e-7 and 2e-7).  The selected parents
    # and tokens are exact either way.
    if case["kind"] == "select":
        return {"rel": 1e-6, "max": 4e-6, "differ": 0.0}
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}
    return {"rel": 1e-2, "max": 1e-1, "differ": 0.0}


# ---------------------------------------------------------------------------------------------
# the same in 64 bits, by plain torch
# ---------------------------------------------------------------------------------------------
def _attend64(q, k, v, visible, scale):
    """q [n][Hq][d], k / v [Hkv][N][d], visible [n][N]: softmax attention, zeros for a query
    that sees nothing."""
    n, Hq, D = q.shape
    Hkv = k.shape[0]
    G = Hq // Hkv
    qd = q.double().view(n, Hkv, G, D).permute(1, 0, 2, 3).reshape(Hkv, n * G, D)
    s = torch.bmm(qd, k.double().transpose(1, 2).contiguous()).mul_(scale).view(Hkv, n, G, -1)
    s.masked_fill_(~visible[None, :, None, :], -math.inf)
    p = torch.nan_to_num(torch.softmax(s, -1)).view(Hkv, n * G, -1)
    return torch.bmm(p, v.double()).view(Hkv, n, G, D).permute(1, 0, 2, 3).reshape(n, Hq, D)


def _select64(logits, score32, score64, b, eos):
    """The b best candidates of one trie's live rows [n][V], by the 32-bit scores that define
    the order (ties to the lower index), with 64-bit scores beside them."""
    lse = torch.logsumexp(logits.double(), 1)
    s = score32[:, None] + (logits - lse.float()[:, None])
    if eos >= 0:
        s[:, eos] = -math.inf
    s = s.reshape(-1)
    at = torch.nonzero(s >= torch.topk(s, b).values[-1]).view(-1)
    at = at[torch.sort(s[at], descending=True, stable=True).indices[:b]]
    par, tok = at // logits.shape[1], at % logits.shape[1]
    lp = logits[par, tok].double() - lse[par]
    return lse, par, tok, s[at], score64[par] + lp, lp


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    kind, T, b = c["kind"], c["tries"], c["beams"]
    if kind == "select":
        res = dict(sel_parent=None, sel_token=None)
        got = [_select64(x["logits"][t], x["score"][t], x["score"][t].double(), b, c["eos"]) for t in range(T)]
        for name, i in (("sel_score", 4), ("sel_logprob", 5), ("lse", 0)):
            res[name] = torch.stack([g[i] for g in got])
        return res
    L, W, scale = c["layers"], c["window"], 1.0 / math.sqrt(c["head_dim"])
    out = torch.zeros(x["q"].shape, dtype=torch.float64, device="cuda")
    if kind in ("attend", "tree"):
        for t, s in enumerate(x["tries"]):
            n = s["n_nodes"]
            up = np.zeros((n, n), bool)  # up[i]: i's stored ancestors and itself
            for i in range(n):
                p = s["parent_slot"][i]
                if p >= 0:
                    up[i] = up[p]
                up[i, i] = True
            up[s["mask"] == 0] = False
            qs = x["qslots"][t].cpu().numpy() if kind == "tree" else s["leaf_slot"]
            vis = up[np.maximum(qs, 0)] & (qs >= 0)[:, None]
            if W:
                vis &= s["depth"][np.maximum(qs, 0)][:, None] - s["depth"][None, :] < W
            vis = torch.from_numpy(vis).cuda()
            for l in range(L):
                for q0 in range(0, len(qs), 512):
                    part = slice(q0, min(q0 + 512, len(qs)))
                    out[l, t, part] = _attend64(x["q"][l, t, part], x["k"][t, l, :, :n], x["v"][t, l, :, :n],
                                                vis[part], scale)
        return out
    sel = {k: torch.zeros((c["steps"], T, b), dtype=torch.float64, device="cuda")
           for k in ("sel_score", "sel_logprob", "lse")}
    for t, P in enumerate(x["lengths"]):
        paths = [[]]  # per live beam: its generated nodes, (step, rank) as an index step * b + rank
        s32, s64 = torch.zeros(1, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        for s in range(c["steps"]):
            n = len(paths)
            vis = torch.zeros((n, P + s * b), dtype=torch.bool, device="cuda")
            for i, path in enumerate(paths):
                vis[i, max(0, P + s - W) if W else 0:P] = True
                for d, node in enumerate(path):  # (its position is P + d; the query's is P + s - 1)
                    vis[i, P + node] = not W or s - 1 - d < W
            for l in range(L):
                k, v = x["k"][t, l, :, :P], x["v"][t, l, :, :P]
                if s:  # the nodes of step j hold the rows given at step j + 1
                    kn, vn = (x[m][1:s + 1, l, t].reshape(s * b, c["kv_heads"], -1).transpose(0, 1)
                              for m in ("k_new", "v_new"))
                    k, v = torch.cat([k, kn], 1), torch.cat([v, vn], 1)
                out[s, l, t, :n] = _attend64(x["q"][s, l, t, :n], k, v, vis, scale)
            lse, par, _, s32, sc, lp = _select64(x["logits"][s, t, :n], s32, s64, b, c.get("eos", -1))
            s64 = sc
            sel["lse"][s, t, :n], sel["sel_score"][s, t], sel["sel_logprob"][s, t] = lse, sc, lp
            paths = [paths[p] + [s * b + j] for j, p in enumerate(par.tolist())]
    res = dict(sel, sel_parent=None, sel_token=None, out=out)
    if c.get("eos", -1) >= 0:
        res.update({"finished_" + k: None for k in ("norm", "score", "step", "parent")})
    return res
