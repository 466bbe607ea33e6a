"""Kernels and branches at the sizes where they can go wrong: edges of tiles, remainders, the smallest and largest of a range."""
import numpy as np
import pytest
import torch

from helpers import cfg_kw, np_weights, to_np
from paper_2509_18085_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def sp():
    from paper_2509_18085_amd import spiffy
    return spiffy


@pytest.mark.parametrize("V,K,B", [(1003, 5, 7), (130, 8, 33), (2049, 1, 1)])
def test_topk_slices_of_the_last_chunk(sp, V, K, B):
    """A chunk of 128 tokens is recomputed by eight workgroups: last chunks of 107, 2 and 1 tokens end inside a slice and inside
    a group of four rows."""
    from test_gpu_parity import check_head_topk
    cfg = synth.CONFIGS["c1"].scaled(dtype="bf16", d=192, V=V, B=B, G=3)
    st = synth.random_states(cfg.G, cfg.B, cfg.V, 0.2, 0.9, 3)
    st[1, :] = cfg.mask_id
    check_head_topk(sp, cfg, st, synth.hidden_states(cfg), synth.head_weights(cfg), 6.0, K, (0, 1))


@pytest.mark.parametrize("V,K,B", [(1003, 7, 10), (2049, 6, 24), (1003, 4, 76), (90, 8, 3)])
def test_topk_shared_by_fewer_workgroups(sp, V, K, B):
    """Four, two and one workgroup a chunk; fewer chunks than K, so that wavefronts of the merge have none."""
    from test_gpu_parity import check_head_topk
    cfg = synth.CONFIGS["c1"].scaled(dtype="bf16", d=192, V=V, B=B, G=2)
    st = synth.random_states(cfg.G, cfg.B, cfg.V, 0.2, 0.9, 4)
    st[1, :] = cfg.mask_id
    check_head_topk(sp, cfg, st, synth.hidden_states(cfg), synth.head_weights(cfg), 6.0, K, (0, 1))


@pytest.mark.parametrize("B,G,P,hq,hkv", [(24, 44, 130, 16, 8), (7, 150, 64, 16, 16), (40, 27, 0, 28, 4), (1, 1030, 65, 16, 2)])
def test_attention_rows_of_any_block_do_not_depend_on_the_query_tile(sp, B, G, P, hq, hkv):
    """Blocks that neither divide 32 nor are multiples of it: the groups of own-block keys start anywhere, and 128-, 64- and
    32-row query tiles (all the states, a third of them, the first ones) visit them the same way.  The rotary embedding and
    the biases come from the projection's epilogue: ragged row tiles, odd table lengths, one token a block."""
    from test_gpu_parity import run_layer, rel_err, tol, oracle_kw, O
    cfg = synth.CONFIGS["c4"].scaled(L=1, F=512, V=1280, d=256, Hq=hq, Hkv=hkv, P=P, B=B, G=G)
    w = synth.layer_weights(cfg, 0, bias=True)
    pk, pv = synth.prefix_kv(cfg, 0)
    x = synth.hidden_states(cfg)
    full = run_layer(sp, cfg, w, pk, pv, x)
    for n in (1, max(1, G // 9), G // 3):
        assert torch.equal(run_layer(sp, cfg, w, pk, pv, x[:n].contiguous()), full[:n]), n
    for g in (0, G - 1):
        ref = O().verify_layer(np_weights(w), to_np(pk), to_np(pv), to_np(x[g:g + 1]), **oracle_kw(cfg))
        e_max, _ = rel_err(to_np(full[g:g + 1]), ref)
        assert e_max < tol(cfg), (g, e_max)


@pytest.mark.parametrize("B,S,P", [(7, 45, 131), (32, 300, 64), (1, 3, 0)])
def test_projection_extends_the_cache(sp, B, S, P):
    """The projection's epilogue stores the true block and the suffix behind it: rows of the full-sequence step equal those that
    committing the same tokens as one block leaves, and rows in front of and behind them stay."""
    cfg = synth.CONFIGS["c4"].scaled(L=1, F=512, V=1280, d=256, P=P, B=B, G=3)
    scfg = sp.cfg_from_synth(cfg)
    w = {k: v.to(DEV) for k, v in synth.layer_weights(cfg, 0, bias=True).items()}
    lw = [sp.layer_weights(w)]
    hw = synth.head_weights(cfg)
    emb = synth.embed_weights(cfg).to(DEV)
    g = torch.Generator().manual_seed(5)
    rows = P + B + S + 4
    k0 = torch.randn((cfg.Hkv, rows, cfg.hd), generator=g).to(torch.bfloat16)
    v0 = torch.randn((cfg.Hkv, rows, cfg.hd), generator=g).to(torch.bfloat16)
    st = torch.from_numpy(synth.random_states(cfg.G, B, cfg.V, 0.2, 0.9, 7)).to(DEV)
    suffix = torch.randint(0, cfg.V - 1, (S,), generator=g, dtype=torch.int32).to(DEV)
    ka, va = k0.to(DEV), v0.to(DEV)
    plan = sp.SeqStepPlan(scfg, lw, [sp.prefix_kv(ka, va, P, 0)], emb, hw["final_norm"].to(DEV), hw["w_vocab"].to(DEV), cfg.G, B,
                          S, P, 0.9, logit_scale=1.0, device=DEV)
    plan.run(st, suffix, None)
    kb, vb = k0.to(DEV), v0.to(DEV)
    for tok, p in ((st[0], P), (suffix, P + B)):         # the layer's keys do not depend on the attention: one layer
        n = tok.numel()
        sp.StepPlan(scfg, lw, [sp.prefix_kv(kb, vb, p, 0)], emb, hw["final_norm"].to(DEV), hw["w_vocab"].to(DEV), 1, n, p, 0.9,
                    logit_scale=1.0, device=DEV).commit_block(tok.contiguous())
    torch.cuda.synchronize()
    assert torch.equal(ka, kb) and torch.equal(va, vb)
    for a, b in ((ka, k0), (va, v0)):
        assert torch.equal(a[:, :P].cpu(), b[:, :P]) and torch.equal(a[:, P + B + S:].cpu(), b[:, P + B + S:])
        assert not torch.equal(a[:, P:P + B + S].cpu(), b[:, P:P + B + S])


@pytest.mark.parametrize("name,d,hq,hkv,F,states", [("c3", 4096, 32, 32, 12288, (6, 9, 11, 19, 24)),
                                                    ("c4", 3584, 28, 4, 18944, (7, 8, 11, 14, 24)),
                                                    ("c4", 2048, 16, 8, 5632, (4, 11, 19, 24, 32))])
def test_layer_rows_are_bit_identical_across_all_tile_heights(sp, name, d, hq, hkv, F, states):
    """The row counts (192 .. 1024) run gate/up in tiles of 192 x 128, 128 x 64, 320 x 128, 192 x 192, 256 x 256, 320 x 192 and
    384 x 128 beside the others, in one and in two column ranges, and the other projections in some of them (every shape of
    every projection: test_layer_rows_in_every_tile_shape); every state equals what it gives alone, where the layer runs in
    tiles of 32 and 64 rows.  Two row counts are not multiples of 32."""
    cfg = synth.CONFIGS[name].scaled(L=1, V=1280, P=64, d=d, Hq=hq, Hkv=hkv, F=F, G=max(states))
    g = torch.Generator(device=DEV).manual_seed(3)
    rn = lambda *s: (torch.randn(s, generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    w = dict(wq=rn(hq * 128, d), wk=rn(hkv * 128, d), wv=rn(hkv * 128, d), wo=rn(d, hq * 128), w_gate=rn(F, d), w_up=rn(F, d),
             w_down=rn(d, F), norm1=1 + rn(d), norm2=1 + rn(d))
    pk, pv = rn(hkv, 64, 128) * 50, rn(hkv, 64, 128) * 50
    scfg, lw, pf = sp.cfg_from_synth(cfg), sp.layer_weights(w), sp.prefix_kv(pk, pv)

    def run(x):
        ws = sp.alloc_workspace(scfg, x.shape[0], x.shape[1], 64, DEV)
        return sp.verify_layer(scfg, lw, pf, x, 64, ws).clone()

    x = rn(max(states), 32, d) * 50
    alone = torch.cat([run(x[i:i + 1].contiguous()) for i in range(max(states))])
    for n in states:
        assert torch.equal(run(x[:n].contiguous()), alone[:n]), n
    x = rn(17, 21, d) * 50                               # 357 rows; 16 states are 336 (a state's place decides how its keys
    full = run(x)                                        # fall into groups of 32, so states keep their places here)
    for n in (1, 3, 16):
        assert torch.equal(run(x[:n].contiguous()), full[:n]), n


@pytest.mark.parametrize("name,d,hq,hkv,F", [("c3", 4096, 32, 32, 12288), ("c4", 3584, 28, 4, 18944), ("c4", 2048, 16, 8, 5632)])
def test_layer_rows_in_every_tile_shape(sp, name, d, hq, hkv, F):
    """Every tile shape that the rule picks for a projection of the model up to 2048 rows, each at the fewest rows it is picked
    for: every state equals what it gives alone."""
    todo = {}
    for rows in range(32, 2049, 32):
        for proj, (epi, N, K) in dict(qkv=(sp.GEMM_STORE, (hq + 2 * hkv) * 128, d), output=(sp.GEMM_RESID, d, hq * 128),
                                      gate_up=(sp.GEMM_SWIGLU, F, d), down=(sp.GEMM_RESID, d, F)).items():
            for launch in sp.layer_gemm_plan(epi, rows, N, K)[0]["launches"]:
                todo.setdefault((proj, launch["tile"]), rows)
    assert len(todo) >= 20
    if d == 4096:
        assert all(k in todo for k in (("qkv", (256, 256)), ("qkv", (320, 128)), ("output", (320, 128)), ("down", (320, 128))))
    cfg = synth.CONFIGS[name].scaled(L=1, V=1280, P=64, d=d, Hq=hq, Hkv=hkv, F=F, G=64)
    g = torch.Generator(device=DEV).manual_seed(4)
    rn = lambda *s: (torch.randn(s, generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    w = dict(wq=rn(hq * 128, d), wk=rn(hkv * 128, d), wv=rn(hkv * 128, d), wo=rn(d, hq * 128), w_gate=rn(F, d), w_up=rn(F, d),
             w_down=rn(d, F), norm1=1 + rn(d), norm2=1 + rn(d))
    if name == "c4":
        w.update(bq=rn(hq * 128), bk=rn(hkv * 128), bv=rn(hkv * 128))
    pk, pv = rn(hkv, 64, 128) * 50, rn(hkv, 64, 128) * 50
    scfg, lw, pf = sp.cfg_from_synth(cfg), sp.layer_weights(w), sp.prefix_kv(pk, pv)
    ws = sp.alloc_workspace(scfg, 64, 32, 64, DEV)
    x = rn(64, 32, d) * 50
    alone = torch.cat([sp.verify_layer(scfg, lw, pf, x[i:i + 1].contiguous(), 64, ws).clone() for i in range(max(todo.values()) // 32)])
    for rows in sorted(set(todo.values())):
        n = rows // 32
        assert torch.equal(sp.verify_layer(scfg, lw, pf, x[:n].contiguous(), 64, ws), alone[:n]), \
            [k for k, v in todo.items() if v == rows]


@pytest.mark.parametrize("epi,M,N,K", [("resid", 1056, 4096, 1024), ("resid", 33, 384, 128), ("resid", 300, 2048, 5632),
                                       ("swiglu", 352, 12288, 256), ("swiglu", 1024, 9440, 192), ("swiglu", 17, 96, 128)])
def test_layer_gemm_equals_gemm(sp, epi, M, N, K):
    g = torch.Generator(device=DEV).manual_seed(M)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
    A, W0, W1, R = rn(M, K), rn(N, K), rn(N, K), rn(M, N)
    ws = torch.empty(4 * M * N * 4 + 256, dtype=torch.uint8, device=DEV)
    args = (sp.GEMM_RESID, A, W0, None, R, None, ws) if epi == "resid" else (sp.GEMM_SWIGLU, A, W0, W1)
    assert torch.equal(sp.layer_gemm(*args), sp.gemm(*args))


def test_projections_of_a_pass_in_two_row_ranges(sp):
    """608 block rows and 1024 suffix rows at 12288 columns: the rule launches the QKV projection once for either range, so the second
    launch's rows have table rows and cache rows of their own.  Hidden rows and cache rows equal those of passes with the
    true block, one other state and the same suffix, which are one launch."""
    G, B, S, P = 19, 32, 1024, 40
    cfg = synth.CONFIGS["c3"].scaled(L=1, F=512, V=1280, P=P, B=B, G=G)
    N = (cfg.Hq + 2 * cfg.Hkv) * cfg.hd
    assert len(sp.layer_gemm_plan(sp.GEMM_STORE, G * B, N, cfg.d, S)) == 2
    assert len(sp.layer_gemm_plan(sp.GEMM_STORE, 2 * B, N, cfg.d, S)) == 1
    scfg = sp.cfg_from_synth(cfg)
    lw = [sp.layer_weights({k: v.to(DEV) for k, v in synth.layer_weights(cfg, 0).items()})]
    hw = {k: v.to(DEV) for k, v in synth.head_weights(cfg).items()}
    emb = synth.embed_weights(cfg).to(DEV)
    g = torch.Generator().manual_seed(6)
    kv0 = [torch.randn((cfg.Hkv, P + B + S + 2, cfg.hd), generator=g).to(torch.bfloat16).to(DEV) for _ in range(2)]
    st = torch.from_numpy(synth.random_states(G, B, cfg.V, 0.2, 0.9, 7)).to(DEV)
    suffix = torch.randint(0, cfg.V - 1, (S,), generator=g, dtype=torch.int32).to(DEV)

    def run(tokens):
        k, v = kv0[0].clone(), kv0[1].clone()
        plan = sp.SeqStepPlan(scfg, lw, [sp.prefix_kv(k, v, P, 0)], emb, hw["final_norm"], hw["w_vocab"], tokens.shape[0], B, S, P,
                              0.9, logit_scale=1.0, device=DEV)
        return plan.run(tokens.contiguous(), suffix, None)["hidden"], k, v

    hid, k, v = run(st)
    for i in (1, 7, G - 1):
        h2, k2, v2 = run(st[[0, i]])
        assert torch.equal(k, k2) and torch.equal(v, v2), i
        assert torch.equal(h2[:B], hid[:B]) and torch.equal(h2[B:2 * B], hid[i * B:(i + 1) * B]), i
        assert torch.equal(h2[2 * B:], hid[G * B:]), i
    assert not torch.equal(k, kv0[0])


@pytest.mark.parametrize("d,G,B,masked", [(4096, 2, 7, "some"), (4096, 20, 32, "some"), (2048, 3, 33, "none"), (2048, 5, 24, "all"),
                                          (384, 6, 5, "one")])
def test_head_rows_from_the_last_reduction(sp, d, G, B, masked):
    """Without hidden states the last layer's reduction leaves the head's normalised rows and their list (1024 or 256 threads a
    row; none, one, some or all rows masked; 384 columns: not sliced, a launch of its own).  Layers with different numbers of
    cached rows share the table and the list that the step's first kernel made.  Every output equals that of the same step
    with hidden states."""
    cfg = synth.CONFIGS["c4"].scaled(L=2, F=512, V=1280, d=d, Hq=d // 128, Hkv=d // 128, P=70, B=B, G=G)
    scfg = sp.cfg_from_synth(cfg)
    lw = [sp.layer_weights({k: v.to(DEV) for k, v in synth.layer_weights(cfg, l).items()}) for l in range(2)]
    kv = [tuple(t.to(DEV) for t in synth.prefix_kv(cfg, l)) for l in range(2)]
    pf = [sp.prefix_kv(kv[0][0], kv[0][1], 70, 0), sp.prefix_kv(kv[1][0], kv[1][1], 3, 0)]
    hw = {k: v.to(DEV) for k, v in synth.head_weights(cfg).items()}
    emb = synth.embed_weights(cfg).to(DEV)
    st = synth.random_states(G, B, cfg.V, 0.2, 0.9, 13)
    if masked in ("none", "one"):
        st[st == cfg.mask_id] = 1
    if masked == "all":
        st[:] = cfg.mask_id
    if masked == "one":
        st[G - 1, B - 1] = cfg.mask_id
    toks = torch.from_numpy(st).to(DEV)
    outs = []
    for keep in (False, True):
        plan = sp.StepPlan(scfg, lw, pf, emb, hw["final_norm"], hw["w_vocab"], G, B, 70, 0.9, logit_scale=8.0, device=DEV,
                           keep_hidden=keep)
        o = plan.run(toks, None)
        outs.append({k: v.clone() for k, v in o.items() if k != "hidden" and torch.is_tensor(v)})
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(40, 2056, 72), (33, 8200, 136), (200, 2056, 1032), (130, 3080, 264), (17, 24, 8), (260, 4104, 520)])
def test_tile_gemm_shapes_by_rounds(sp, M, N, K, dtype):
    """32 x 16, 32 x 32 and 64 x 64 tiles, chosen by rounds of workgroups, last chunks of K cut to 8 .. 56 values and wavefronts
    without a chunk; rows do not depend on the tile (the first 16 rows alone run in 16 x 16 tiles, as do the last).  Bounds as for the edges of
    the tiles: |sum - exact| <= (K + 16) 2^-24 sum |a w|, in bf16 plus one rounding of the result, 2^-8 relative; SwiGLU with both
    sums' errors propagated: |silu'| <= 1.1, |silu(g)| <= |g|, its exponential and division within 2^-20 relative."""
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(M + N + K)
    A, W0, W1 = ((torch.randn(s, generator=g) * f).to(td) for s, f in (((M, K), 1.0), ((N, K), 0.1), ((N, K), 0.1)))
    a, w0, w1 = to_np(A), to_np(W0), to_np(W1)
    eps, out = 2.0 ** -24, 0.0 if dtype == "f32" else 1.02 * 2.0 ** -8
    dev = [t.to(DEV) for t in (A, W0, W1)]
    got = sp.gemm(sp.GEMM_STORE, dev[0], dev[1])
    ref, d0 = a @ w0.T, (K + 16) * eps * (np.abs(a) @ np.abs(w0).T)
    assert (np.abs(to_np(got) - ref) <= d0 + (out + eps) * np.abs(ref) + 1e-30).all()
    assert torch.equal(sp.gemm(sp.GEMM_STORE, dev[0][:16].contiguous(), dev[1]), got[:16])
    sw = sp.gemm(sp.GEMM_SWIGLU, *dev)
    up, d1 = a @ w1.T, (K + 16) * eps * (np.abs(a) @ np.abs(w1).T)
    silu = ref / (1 + np.exp(-ref))
    err = 1.1 * d0 * (np.abs(up) + d1) + np.abs(silu) * d1 + 2.0 ** -19 * np.abs(silu * up)
    assert (np.abs(to_np(sw) - silu * up) <= err + out * (np.abs(silu * up) + err) + 1e-30).all()
    for lo, hi in ((0, 16), (M - 16, M)):
        x = dev[0][lo:hi].contiguous()
        assert torch.equal(sp.gemm(sp.GEMM_SWIGLU, x, dev[1], dev[2]), sw[lo:hi])
        assert torch.equal(sp.gemm(sp.GEMM_STORE, x, dev[1]), got[lo:hi])


@pytest.mark.parametrize("K", [1000, 1560, 2824])
def test_large_fp32_tiles(sp, K):
    """fp32 tiles of 64 x 64 with fragments in registers (16 x 16 of them, the last rows and columns ragged): a last chunk of 8
    or 24 values, wavefronts with one chunk less.  Bounds and row identity as for the other tiles; SwiGLU with both sums' errors
    propagated: |silu'| <= 1.1, |silu(g)| <= |g|, its exponential and division within 2^-20 relative."""
    M, N, F = 1000, 1016, 504
    g = torch.Generator().manual_seed(K)
    A, W0, W1, R = (torch.randn(s, generator=g) * f for s, f in (((M, K), 1.0), ((N, K), 0.1), ((F, K), 0.1), ((M, N), 1.0)))
    a, w0, w1, r = (t.double().numpy() for t in (A, W0, W1, R))
    eps = (K + 16) * 2.0 ** -24
    dev = [t.to(DEV) for t in (A, W0, W1, R)]
    ref, d0 = a @ w0.T, eps * (np.abs(a) @ np.abs(w0).T)
    store, resid = sp.gemm(sp.GEMM_STORE, dev[0], dev[1]), sp.gemm(sp.GEMM_RESID, dev[0], dev[1], R=dev[3])
    assert (np.abs(to_np(store) - ref) <= d0 + 2.0 ** -24 * np.abs(ref)).all()
    assert (np.abs(to_np(resid) - ref - r) <= d0 + 2.0 ** -22 * (np.abs(ref) + np.abs(r))).all()
    gate, up = ref[:, :F], a @ w1.T
    silu = gate / (1 + np.exp(-gate))
    d1 = eps * (np.abs(a) @ np.abs(w1).T)
    wg = dev[1][:F].contiguous()
    sw = sp.gemm(sp.GEMM_SWIGLU, dev[0], wg, dev[2])
    assert (np.abs(to_np(sw) - silu * up) <= 1.1 * d0[:, :F] * (np.abs(up) + d1) + np.abs(silu) * d1 + 2.0 ** -19 * np.abs(silu * up) + 1e-30).all()
    for lo, hi in ((0, 16), (990, 1000)):                # alone: 16 x 16 tiles
        x = dev[0][lo:hi].contiguous()
        assert torch.equal(sp.gemm(sp.GEMM_STORE, x, dev[1]), store[lo:hi])
        assert torch.equal(sp.gemm(sp.GEMM_RESID, x, dev[1], R=dev[3][lo:hi].contiguous()), resid[lo:hi])
        assert torch.equal(sp.gemm(sp.GEMM_SWIGLU, x, wg, dev[2]), sw[lo:hi])


@pytest.mark.parametrize("V,d", [(31900, 192), (31874, 512), (66300, 256)])
def test_head_rows_do_not_depend_on_the_tile_shape(sp, V, d):
    """125 tiles of 256 vocabulary rows: 128 x 128 up to 128 rows, 128 x 256 up to 256, 256 x 192 up to 384, 256 x 256 up to 512,
    256 x 192 again at 571; 259 tiles: 256 x 192 at 160 and 384 rows, 128 x 256 at 256 and 512.  The last tile ends
    in its first or second half, K of three to eight steps.  Every output equals, bit for bit, that of the states alone, and the
    top token that of the float64 logits."""
    G, B = 18, 32
    cfg = synth.CONFIGS["c1"].scaled(d=d, V=V, G=G, B=B, dtype="bf16")
    g = torch.Generator().manual_seed(d)
    x, w = torch.randn((G, B, d), generator=g).bfloat16().to(DEV), (torch.randn((V, d), generator=g) * 0.1).bfloat16().to(DEV)
    gain = torch.ones(d).bfloat16().to(DEV)
    tok = torch.full((G, B), cfg.mask_id, dtype=torch.int32)
    tok[-1, 27:] = 1                                   # 571 rows
    tok = tok.to(DEV)
    scfg = sp.cfg_from_synth(cfg)
    ws = sp.alloc_workspace(scfg, G, B, 0, DEV)
    head = lambda a, b: sp.decode_head(scfg, x[a:b].contiguous(), gain, w, tok[a:b].contiguous(), 0.01, ws)
    alone = [head(s, s + 1) for s in range(G)]
    for n in (3, 5, 6, 8, 12, 16, 18):
        got = head(0, n)
        for s in range(n):
            for k in got:
                assert torch.equal(got[k][s], alone[s][k][0]), (n, s, k)
    xd = x.double()
    nf = (xd / (xd.square().mean(-1, keepdim=True) + cfg.rms_eps).sqrt()).bfloat16().double().view(G * B, d)
    top = torch.topk((nf @ w.double().T), 2, dim=1)
    # bf16 products, float32 sums: at most (d + 16) 2^-24 sum |n w| apart; a norm rounded the other way moves a logit by 2^-8 |n w|
    safe = (top.values[:, 0] - top.values[:, 1]) > 2 * 2.0 ** -8 * (nf.abs() @ w.double().abs().T).amax(1)
    m = (tok.view(-1) == cfg.mask_id) & safe
    assert int(m.sum()) >= 100
    assert torch.equal(torch.cat([a["argmax"].view(-1) for a in alone])[m].long(), top.indices[m, 0])
