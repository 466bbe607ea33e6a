"""Performance cases of the draft-graph verification library, through its public binding.

Shapes are those of the repository's workload configurations (synth.CONFIGS c1 .. c5), of its tests and of bench.py.
Transformer stacks run at the configurations' widths with a few layers instead of 28 or 32: every layer does the same
work, the weights of four layers (1.7 GB) do not stay in any cache, and behind a full stack of random-init layers the
roundings of two correct implementations have drifted apart by more than a comparison could allow.  Weights are
N(0, 0.02) as in synth.  A random-init head is flat (every token at about 1/V, ranks decided by rounding), which no decode
loop meets: a few rows of the vocabulary matrix are therefore fitted, as training would, so that every position of the
block has its own four most likely tokens, most positions above the threshold of 0.9 and some below.
"""
import math

import numpy as np
import torch

from paper_2509_18085_amd import decode, spiffy as sp, synth

DEV = "cuda"

# widths of the models: the five configurations' and two small ones that the matrix-core path does not take
# (head_dim 64, as in the generic-shape tests; the second kind is the fp32 configuration at a usable size)
MODELS = {
    "llada": dict(d=4096, Hq=32, Hkv=32, hd=128, F=12288, V=126464, bias=False),      # c2, c3, c5
    "dream": dict(d=3584, Hq=28, Hkv=4, hd=128, F=18944, V=152064, bias=True),        # c4: grouped heads, biases
    "mid": dict(d=2048, Hq=16, Hkv=8, hd=128, F=5632, V=32000, bias=False),           # generic, matrix-core path
    "small": dict(d=1024, Hq=16, Hkv=4, hd=64, F=2816, V=32000, bias=True),           # generic, head_dim 64
    "tiny": dict(d=256, Hq=4, Hkv=4, hd=64, F=688, V=1024, bias=False),               # c1
}


def _step(name, model, L, G, B, P, dtype="bf16", S=0, seq=0, prev=0, draft=0, hidden=0):
    """One forward pass of the decode loop.  S: cached rows after the block (dual cache); seq: suffix rows recomputed in
    the pass; prev: the finished block before this one is committed in the same pass; draft: the next step's drafts
    follow (top-K with K = draft, drafting, pruning); hidden: the last layer's output is asked for too."""
    return dict(name=name, kind="step", model=model, L=L, G=G, B=B, P=P, dtype=dtype, S=S, seq=seq, prev=prev,
                draft=draft, hidden=hidden)


def listed():
    return [
        # The smallest call: the fp32 configuration c1 (2 layers of width 256, 4 states of 8 tokens).  Launch latency.
        _step("tiny_fp32_step", "tiny", 2, 4, 8, 64, dtype="f32", hidden=1),
        # A vanilla pass: one 32-token state behind 1024 cached rows; what every block of undrafted decoding repeats.
        _step("one_state", "llada", 4, 1, 32, 1024),
        # The paper's operating point: the true block and three drafts, with the next step's drafting, as decode.py runs it.
        _step("four_states_drafting", "llada", 4, 4, 32, 1024, draft=3),
        # The headline configuration c3: a graph of 32 states, 1024 rows.
        _step("draft_graph_32", "llada", 4, 32, 32, 1024),
        # Configuration c4: grouped-query attention, biases, 24 states behind 2048 rows.
        _step("gqa_24_states", "dream", 4, 24, 32, 2048),
        # Configuration c5: 64 states of a 4-token block behind a long cache.
        _step("small_block_long_prefix", "llada", 4, 64, 4, 8192),
        # A full-sequence model (prefix cache only): three drafts and the 224 tokens after the block recomputed.
        _step("full_sequence", "llada", 4, 4, 32, 1024, seq=224, hidden=1),
        # First pass of a block: the finished block is committed with it.  Odd prefix, grouped heads, 5 states.
        _step("block_start_commit", "dream", 4, 5, 32, 1387, prev=1, hidden=1),
        # One layer alone with a dual cache and nothing that divides a tile: 11 states of 24 tokens, 777 + 150 rows.
        dict(name="ragged_layer_dual_cache", kind="layer", model="mid", G=11, B=24, P=777, dtype="bf16", S=150),
        # A model with 64-wide heads (no matrix-core path): two layers, 4 states, head included.
        _step("head_dim_64_bf16", "small", 2, 4, 32, 512, hidden=1),
        # fp32 at a usable size.
        _step("fp32_step", "small", 2, 4, 16, 300, dtype="f32", hidden=1),
        # Offline calibration: best connected 10-node set of a 45-node candidate graph (bench.py's size).
        dict(name="subgraph_45_10", kind="subgraph", levels=15, width=3, D=10),
    ]


def draw(rng):
    """One more case of the same ranges: the matrix-core models with 1 to 64 states and 1 to 1024 rows, 0 to 8192 cached
    rows, all kinds of passes; small models off that path in both types; subgraph searches of up to the listed size."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    u = rng.random()
    if u < 0.12:
        width = rng.choice([2, 3, 4, 5])
        return dict(kind="subgraph", levels=rng.randrange(18, 45) // width, width=width, D=rng.randrange(4, 11))
    if u < 0.37:
        dtype = rng.choice(["bf16", "f32"])
        B = rng.choice([4, 7, 8, 16, 20, 32])
        c = _step("", rng.choice(["tiny", "small"]), rng.randrange(1, 3), min(log_int(1, 16), (128 if dtype == "bf16" else 64) // B),
                  B, log_int(1, 512), dtype=dtype, hidden=rng.randrange(2))
        c.pop("name")
        return c
    model = rng.choice(["llada", "dream", "mid"])
    B = rng.choice([1, 4, 8, 16, 24, 32, 32, 32, 64])
    G = max(1, min(log_int(1, 64), 768 // B))
    P = log_int(1, 8192)
    if u < 0.52:
        return dict(kind="layer", model=model, G=G, B=B, P=P, dtype="bf16", S=rng.choice([0, 0, log_int(1, 600)]))
    kind = rng.choice(["plain", "plain", "draft", "seq", "prev", "dual"])
    if kind in ("seq", "prev"):
        G = min(G, max(1, 256 // B))
    hidden = rng.randrange(2) if kind in ("plain", "dual") else int(kind != "draft")
    c = _step("", model, rng.randrange(1, 4), G, B, P, hidden=hidden, S=log_int(1, 600) if kind == "dual" else 0,
              seq=log_int(16, 400) if kind == "seq" else 0, prev=int(kind == "prev"),
              draft=rng.randrange(1, 5) if kind == "draft" else 0)
    c.pop("name")
    return c


# ---------------------------------------------------------------------------------------------------- inputs

def _cfg(c):
    m = MODELS[c["model"]]
    return synth.Config("case", c.get("L", 1), m["d"], m["Hq"], m["Hkv"], m["hd"], m["F"], m["V"], c["P"], c["B"], c["G"],
                        c["dtype"], 0.9)


def _masked(G, B):
    """Masked positions of each state: the block's state (node 0) has three quarters masked, node i has one to four fewer
    than its parent (i - 1) // 3."""
    n = [max(1, round(0.75 * B))]
    for i in range(1, G):
        n.append(max(0, n[(i - 1) // 3] - 1 - i % 4))
    return n


def _states(G, B, V, seed):
    r = np.random.default_rng(seed)
    mask = V - 1
    n = _masked(G, B)
    st = np.empty((G, B), np.int32)
    st[0] = r.integers(0, V - 1, B)
    st[0, r.permutation(B)[:n[0]]] = mask
    for i in range(1, G):
        st[i] = st[(i - 1) // 3]
        pos = np.nonzero(st[i] == mask)[0]
        k = len(pos) - n[i]
        if k:
            pos = r.choice(pos, k, replace=False)
            st[i, pos] = r.integers(0, V - 1, k)
    edges = []
    for i in range(1, G):
        a = i
        while a:                                   # every ancestor holds a subset of node i's tokens
            a = (a - 1) // 3
            if n[a] > n[i]:
                edges.append((a, i))
    return st, np.asarray(edges, np.int32).reshape(-1, 2)


class _Draw:
    """Seeded normals on the device, one stream per case and seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed * 7919 + 11)

    def normal(self, shape, std, dtype, mean=0.0):
        x = torch.randn(shape, generator=self.g, device=DEV, dtype=torch.float32)
        return x.mul_(std).add_(mean).to(dtype)


def _layer(dr, cfg, bias):
    dt, qd, kvd = cfg.torch_dtype(), cfg.Hq * cfg.hd, cfg.Hkv * cfg.hd
    w = {k: dr.normal(s, 0.02, dt) for k, s in dict(wq=(qd, cfg.d), wk=(kvd, cfg.d), wv=(kvd, cfg.d), wo=(cfg.d, qd),
                                                   w_gate=(cfg.F, cfg.d), w_up=(cfg.F, cfg.d), w_down=(cfg.d, cfg.F)).items()}
    for k in ("norm1", "norm2"):
        w[k] = dr.normal((cfg.d,), 0.02, dt, 1.0)
    if bias:
        for k, n in (("bq", qd), ("bk", kvd), ("bv", kvd)):
            w[k] = dr.normal((n,), 0.02, dt)
    return w


def _cache_rows(c):
    return c["P"] + (c["B"] if c.get("prev") else 0) + c["B"] + max(c.get("S", 0), c.get("seq", 0))


def _formulas(G, K):
    """G - 1 draft formulas: node i unmasks the first ranks of the drafting source, some with a lower-ranked token."""
    out = []
    for i in range(1, G):
        out.append([(r, 1 + (i // 2 if r == 1 + i // 2 else 0) % K) for r in range(1, 2 + i // 2)])
    return out


# Plain torch forward (fp32 attention) that only serves to fit the head's rows; nothing of it is timed or compared.

def _norm(x, g):
    x = x.float()
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5) * g.float()


def _rope(x, pos, base):                              # x [rows, heads, hd]
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * (base ** (-torch.arange(half, device=DEV, dtype=torch.float64) / half))[None, :]
    cs, sn = ang.cos().float()[:, None, :], ang.sin().float()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cs - b * sn, b * cs + a * sn], -1)


def _heads_first(x, rep):                             # [rows, heads, hd] -> [heads * rep, rows, hd]
    return x.permute(1, 0, 2).repeat_interleave(rep, 0).contiguous()


def _attend(q, keys, vals, own_k=None, own_v=None, G=1):
    """q [H, rows, hd] over shared keys [H, n, hd] and, when given, each of the G states over its own rows."""
    H, M, hd = q.shape
    sc = torch.matmul(q, keys.transpose(1, 2).contiguous()) / math.sqrt(hd)
    if own_k is None:
        return torch.matmul(torch.softmax(sc, -1), vals)
    n, qb = keys.shape[1], q.reshape(H * G, M // G, hd)
    own = torch.matmul(qb, own_k.reshape(H * G, M // G, hd).transpose(1, 2).contiguous()) / math.sqrt(hd)
    p = torch.softmax(torch.cat([sc.reshape(H * G, M // G, n), own], -1), -1)
    o = torch.matmul(p[..., :n].reshape(H, M, n).contiguous(), vals).reshape(H * G, M // G, hd)
    return (o + torch.matmul(p[..., n:].contiguous(), own_v.reshape(H * G, M // G, hd))).reshape(H, M, hd)


def _reference_hidden(c, cfg, layers, prefix, w_embed, tokens, extra):
    """Hidden states of the G * B rows of a pass; extra = tokens of the finished block or of the suffix, or None."""
    G, B, P, n_x = c["G"], c["B"], c["P"], 0 if extra is None else len(extra)
    off = B if c["prev"] else 0
    pos = (P + off + torch.arange(B, device=DEV)).repeat(G)
    if n_x:
        pos = torch.cat([pos, (P if c["prev"] else P + B) + torch.arange(n_x, device=DEV)])
    tok = tokens.reshape(-1) if extra is None else torch.cat([tokens.reshape(-1), extra])
    h, M, rep, qd, kvd = w_embed[tok.long()], G * B, cfg.Hq // cfg.Hkv, cfg.Hq * cfg.hd, cfg.Hkv * cfg.hd
    dt = h.dtype
    for w, (pk, pv) in zip(layers, prefix):
        n = _norm(h, w["norm1"]).to(dt)
        q, k, v = (torch.matmul(n, w[a].t()).float() + (w[b].float() if b in w else 0.0) for a, b in (("wq", "bq"), ("wk", "bk"), ("wv", "bv")))
        q = _heads_first(_rope(q.reshape(-1, cfg.Hq, cfg.hd), pos, cfg.rope_base), 1)
        k = _heads_first(_rope(k.reshape(-1, cfg.Hkv, cfg.hd), pos, cfg.rope_base), rep)
        v = _heads_first(v.reshape(-1, cfg.Hkv, cfg.hd), rep)
        ck, cv = (t.float().repeat_interleave(rep, 0) for t in (pk, pv))
        ks, vs = [ck[:, :P]], [cv[:, :P]]
        if n_x:
            ks, vs = ks + [k[:, M:]], vs + [v[:, M:]]
        elif c["S"]:
            ks, vs = ks + [ck[:, P + B:P + B + c["S"]]], vs + [cv[:, P + B:P + B + c["S"]]]
        o = _attend(q[:, :M].contiguous(), torch.cat(ks, 1), torch.cat(vs, 1), k[:, :M].contiguous(), v[:, :M].contiguous(), G)
        if n_x:                                       # the finished block, or the suffix behind the true block
            sees = [ck[:, :P]] + ([k[:, :B]] if c["seq"] else []) + [k[:, M:]]
            sees_v = [cv[:, :P]] + ([v[:, :B]] if c["seq"] else []) + [v[:, M:]]
            o = torch.cat([o, _attend(q[:, M:].contiguous(), torch.cat(sees, 1), torch.cat(sees_v, 1))], 1)
        h = h + torch.matmul(o.permute(1, 0, 2).reshape(-1, qd).to(dt), w["wo"].t())
        n = _norm(h, w["norm2"]).to(dt)
        a = torch.nn.functional.silu(torch.matmul(n, w["w_gate"].t()).float()) * torch.matmul(n, w["w_up"].t()).float()
        h = h + torch.matmul(a.to(dt), w["w_down"].t())
    return h[:M]


def _fit_head(cfg, w_vocab, x, masked, seed):
    """Rewrites four vocabulary rows per block position: ridge regression of their logits at the masked rows x."""
    B, r = cfg.B, np.random.default_rng(seed + 2)
    toks = torch.from_numpy(r.permutation(cfg.V - 1)[:4 * B].copy()).to(DEV)
    floor = math.log(cfg.V) + 0.5 * 0.0004 * cfg.d    # what the other tokens' exponentials add up to
    step = 11.0 / B                                   # lead of the first token: 0.5 .. 12, none near the threshold
    lead = np.array([0.5 + step * i if 0.5 + step * i < 1.6 else 1.6 + step * i for i in range(B)])[r.permutation(B)]
    want = torch.zeros((B, 4 * B), device=DEV)
    for b in range(B):
        want[b, 4 * b:4 * b + 4] = torch.tensor([floor + 2.4 + lead[b], floor + 2.4, floor - 0.6, floor - 3.6], device=DEV)
    rows = torch.nonzero(masked.reshape(-1)).flatten()
    if len(rows):
        x = x[rows]
        gram = torch.matmul(x, x.t().contiguous()).double()
        gram.diagonal().add_(2e-3 * cfg.d)
        coef = torch.linalg.solve(gram, want[rows % B].double())
        w_vocab[toks] = torch.matmul(coef.t().contiguous(), x.double()).to(w_vocab.dtype)


def prepare(case, seed):
    c = case
    if c["kind"] == "subgraph":
        cnt, lvl, edges, _ = synth.candidate_graph(c["levels"], c["width"], seed=seed)
        n = int(sp.lib.spiffy_subgraph_search_workspace_bytes())
        return dict(c=c, count=torch.from_numpy(cnt).to(DEV), level=torch.from_numpy(lvl).to(DEV),
                    edges=torch.from_numpy(np.ascontiguousarray(edges)).to(DEV),
                    ws=torch.empty(n + 256, dtype=torch.uint8, device=DEV))
    cfg, dr = _cfg(c), _Draw(seed)
    m, dt, scfg = MODELS[c["model"]], cfg.torch_dtype(), sp.cfg_from_synth(cfg)
    weights = [_layer(dr, cfg, m["bias"]) for _ in range(cfg.L)]
    rows = _cache_rows(c)
    kv = (cfg.Hkv, rows, cfg.hd)
    cache = [(dr.normal(kv, 1.0, dt), dr.normal(kv, 1.0, dt)) for _ in range(cfg.L)]
    layers = [sp.layer_weights(w) for w in weights]
    prefix = [sp.prefix_kv(k, v, c["P"], c.get("S", 0)) for k, v in cache]
    G, B = c["G"], c["B"]
    if c["kind"] == "layer":
        return dict(c=c, cfg=scfg, w=layers[0], prefix=prefix[0], x=dr.normal((G, B, cfg.d), 1.0, dt),
                    out=torch.empty((G, B, cfg.d), dtype=dt, device=DEV), ws=sp.alloc_workspace(scfg, G, B, c["P"] + c["S"], DEV))
    w_embed, w_vocab = dr.normal((cfg.V, cfg.d), 0.02, dt), dr.normal((cfg.V, cfg.d), 0.02, dt)
    final_norm = dr.normal((cfg.d,), 0.02, dt, 1.0)
    st, edges = _states(G, B, cfg.V, seed)
    tokens, extra = torch.from_numpy(st).to(DEV), None
    if c["seq"]:
        extra = torch.full((c["seq"],), cfg.mask_id, dtype=torch.int32, device=DEV)      # semi-autoregressive order: MASK
    if c["prev"]:
        extra = torch.from_numpy(np.random.default_rng(seed + 1).integers(0, cfg.V - 1, B).astype(np.int32)).to(DEV)
    hid = _reference_hidden(c, cfg, weights, cache, w_embed, tokens, extra)
    _fit_head(cfg, w_vocab, _norm(hid, final_norm), tokens == cfg.mask_id, seed)
    del hid
    s = dict(c=c, cfg=scfg, tokens=tokens, extra=extra, edges=torch.from_numpy(edges).to(DEV) if len(edges) else None)
    kw = dict(logit_scale=1.0, force_one=True, device=DEV)
    if c["seq"]:
        s["plan"] = sp.SeqStepPlan(scfg, layers, prefix, w_embed, final_norm, w_vocab, G, B, c["seq"], c["P"], 0.9, **kw)
    else:
        s["plan"] = sp.StepPlan(scfg, layers, prefix, w_embed, final_norm, w_vocab, G, B, c["P"], 0.9,
                                keep_hidden=bool(c["hidden"]), **kw)
    if c["draft"]:
        s["graph"] = decode.DraftGraph(_formulas(max(G, 2), c["draft"]), device=DEV)
    return s


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "subgraph":
        r = sp.subgraph_search(s["count"], s["level"], s["edges"], c["D"], s["ws"])
        return {k: r[k] for k in ("best_mask", "best_sum", "n_connected", "nodes")}
    if c["kind"] == "layer":
        return sp.verify_layer(s["cfg"], s["w"], s["prefix"], s["x"], c["P"], s["ws"], s["out"])
    plan = s["plan"]
    if c["seq"]:
        o = plan.run(s["tokens"], s["extra"], s["edges"])
    elif c["prev"]:
        o = plan.run_commit(s["extra"], s["tokens"], s["edges"])
        out = dict(o)
        cache = plan._keep[1]                        # the committed rows are results too
        B, P = c["B"], c["P"]
        out["k_rows"] = [p._keep[0][:, P:P + B] for p in cache]
        out["v_rows"] = [p._keep[1][:, P:P + B] for p in cache]
        return out
    else:
        o = plan.run(s["tokens"], s["edges"])
    out = dict(o)
    if not c["hidden"]:
        out.pop("hidden")
    if c["draft"]:
        g = s["graph"]
        tok, prob = sp.head_topk(s["cfg"], plan.w_vocab, s["tokens"], g.K, plan.logit_scale, plan.workspace,
                                 result=o["result"], after_step=True)
        d = sp.draft_prune(o["accepted_state"], s["cfg"].mask_id, tok, prob, g.offsets, g.pairs, g.edges, g.D)
        out.update(topk_tokens=tok, topk_probs=prob, next_states=d["drafts"], buildable=d["buildable"], local=d["local"],
                   score=d["score"])
    return out


def work(case):
    c = case
    if c["kind"] == "subgraph":                      # per set tried: two ANDs, a zero test, an add, a compare on 64 bits
        N = c["levels"] * c["width"]
        return {"bytes": 12 * N, "flops": 10.0 * math.comb(N, c["D"])}
    cfg, m = _cfg(c), MODELS[c["model"]]
    es = 4 if c["dtype"] == "f32" else 2
    qd, kvd = cfg.Hq * cfg.hd, cfg.Hkv * cfg.hd
    attn_out = cfg.d * qd
    per_layer = cfg.d * (qd + 2 * kvd) + attn_out + 3 * cfg.d * cfg.F
    M, extra = c["G"] * c["B"], c.get("seq", 0) + (c["B"] if c.get("prev") else 0)
    keys = c["P"] + c["B"] + c.get("S", 0) + c.get("seq", 0)
    flops = cfg.L * (2.0 * (M + extra) * per_layer + 4.0 * (M + extra) * keys * qd)
    nbytes = cfg.L * es * (per_layer + 2.0 * (c["P"] + c.get("S", 0)) * kvd)
    if c["kind"] == "layer":
        return {"bytes": nbytes + 2 * es * M * cfg.d, "flops": flops}
    masked = sum(_masked(c["G"], c["B"]))
    if not c["hidden"]:                              # nothing but masked rows is read behind the last attention
        flops -= 2.0 * (M - masked) * (attn_out + 3 * cfg.d * cfg.F)
    flops += 2.0 * masked * cfg.V * cfg.d
    nbytes += es * (cfg.V * cfg.d + (M + extra) * cfg.d)
    if c["draft"]:
        flops += 2.0 * masked / c["G"] * c["draft"] * 128 * cfg.d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the present kernels differ by from themselves with the model's width and its FFN width
    permuted (the same function, every sum in another order): hidden states and cached rows 3e-3 (two layers) to 8e-3
    (four), largest 4e-2; confidences, margins and probabilities 1e-3 to 2e-3, largest 1e-2; one layer 1e-3, largest 2e-2;
    fp32 3e-6, largest 1.3e-5, but its confidences 2.5e-5, largest 9e-5, from the same softmax in 64 bits: a sum of 32000
    exponentials in one order loses the ones below half a unit of the sum.  No decision differed."""
    if case["kind"] == "subgraph":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-4, "max": 4e-4, "differ": 0.005}
    if case["kind"] == "layer":
        return {"rel": 5e-3, "max": 0.08}
    if case["hidden"]:
        return {"rel": 3e-2, "max": 0.16, "differ": 0.005}
    return {"rel": 1e-2, "max": 0.05, "differ": 0.005}
