"""GEMM, LM head and attention of the shapes off the bf16 matrix-core path, at the edges of their tiles and remainders."""
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (16, 16, 32), (17, 24, 40), (33, 40, 136), (64, 8, 1032), (65, 1032, 72),
                                   (130, 6008, 264), (128, 2816, 1024)])
def test_tile_gemm_edges(sp, M, N, K, dtype):
    """Against the float64 product.  |fp32 sum - exact| <= (K + 16) 2^-24 sum |a w| whatever the order; the residual, the
    activation (a few units of exp and division, |silu'| <= 1.1) and, in bf16, one final rounding of half a unit in the last of 8 significand bits, 2^-8, are added."""
    if dtype == "bf16" and N % 64 == 0 and K % 64 == 0:
        N += 8                                       # keep it off the MFMA kernel
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(M * 1000 + N + K)
    A, W0, W1, R = ((torch.randn(s, generator=g) * f).to(td) for s, f in (((M, K), 1.0), ((N, K), 0.1), ((N, K), 0.1), ((M, N), 1.0)))
    a, w0, w1, r = to_np(A), to_np(W0), to_np(W1), to_np(R)
    eps, out = 2.0 ** -24, 0.0 if dtype == "f32" else 1.02 * 2.0 ** -8
    d0, d1 = (K + 16) * eps * (np.abs(a) @ np.abs(w0).T), (K + 16) * eps * (np.abs(a) @ np.abs(w1).T)
    dev = [t.to(DEV) for t in (A, W0, W1, R)]
    got = to_np(sp.gemm(sp.GEMM_STORE, dev[0], dev[1]))
    ref = a @ w0.T
    assert (np.abs(got - ref) <= d0 + (out + eps) * np.abs(ref) + 1e-30).all()
    got = to_np(sp.gemm(sp.GEMM_RESID, dev[0], dev[1], R=dev[3]))
    assert (np.abs(got - (ref + r)) <= d0 + (out + 2 * eps) * np.abs(ref + r) + d0 * 2 * eps + 1e-30).all()
    got = to_np(sp.gemm(sp.GEMM_SWIGLU, dev[0], dev[1], dev[2]))
    silu, up = ref / (1 + np.exp(-ref)), a @ w1.T
    bound = 1.1 * d0 * np.abs(up) + d1 * np.abs(silu) + 2 * d0 * d1 + (out + (np.abs(ref) + 16) * 8 * eps) * np.abs(silu * up)
    assert (np.abs(got - silu * up) <= bound + 1e-30).all()


def test_tile_gemm_rows_do_not_depend_on_the_batch(sp):
    g = torch.Generator().manual_seed(5)
    A, W = torch.randn((200, 520), generator=g).to(DEV), torch.randn((6008, 520), generator=g).to(DEV)
    full = sp.gemm(sp.GEMM_STORE, A, W)              # 64 x 64 tiles
    for n in (1, 16, 40):
        assert torch.equal(sp.gemm(sp.GEMM_STORE, A[:n].contiguous(), W), full[:n])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hd,Hq,Hkv,B,P,S", [(8, 2, 2, 1, 0, 0), (24, 6, 2, 5, 3, 0), (64, 4, 1, 16, 15, 0), (72, 2, 1, 7, 130, 9),
                                             (136, 1, 1, 17, 16, 0), (200, 3, 3, 3, 1, 40), (256, 2, 1, 9, 70, 1)])
def test_tile_attention_edges(sp, hd, Hq, Hkv, B, P, S, dtype):
    """One layer against the oracle at the head sizes and key counts where fragments and chunks are cut short."""
    from oracle import spiffy_oracle as O
    cfg = synth.CONFIGS["c1"].scaled(dtype=dtype, d=96, Hq=Hq, Hkv=Hkv, hd=hd, F=72, P=P, B=B, G=3)
    w = synth.layer_weights(cfg, 0, bias=True)
    for k in ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down"):
        w[k] = (w[k].float() * 4).to(w[k].dtype)
    g = torch.Generator().manual_seed(hd)
    k, v = (torch.randn((Hkv, P + B + S, hd), generator=g).to(w["wq"].dtype) for _ in range(2))
    x = synth.hidden_states(cfg)
    scfg = sp.cfg_from_synth(cfg)
    ws = sp.alloc_workspace(scfg, cfg.G, B, P + S, DEV)
    out = sp.verify_layer(scfg, sp.layer_weights({n: t.to(DEV) for n, t in w.items()}),
                          sp.prefix_kv(k.to(DEV), v.to(DEV), P, S), x.to(DEV), P, ws)
    kn, vn = to_np(k), to_np(v)
    kw = dict(suffix_k=kn[:, P + B:], suffix_v=vn[:, P + B:]) if S else {}
    ref = O.verify_layer(np_weights(w), kn[:, :P], vn[:, :P], to_np(x), **cfg_kw(cfg), **kw)
    err = np.max(np.abs(to_np(out) - ref) / (np.abs(ref) + np.sqrt(np.mean(ref * ref))))
    assert err < (1e-4 if dtype == "f32" else 2e-2), err      # the bars of test_gpu_parity


@pytest.mark.parametrize("d,V,G,B", [(8, 63, 1, 1), (40, 65, 2, 9), (72, 64, 3, 16), (256, 1000, 5, 13), (264, 33000, 3, 24),
                                     (16000, 3200, 4, 32)])       # the last: barely inside the static scratch
def test_tile_head_edges(sp, d, V, G, B):
    """fp32 head, every position masked, against a float64 softmax: logit error <= (d + 8) 2^-24 sum |x w|."""
    cfg = synth.CONFIGS["c1"].scaled(d=d, V=V, G=G, B=B)
    g = torch.Generator().manual_seed(V)
    x, gain, w = torch.randn((G, B, d), generator=g), torch.ones(d), torch.randn((V, d), generator=g) * 0.3
    tok = torch.full((G, B), cfg.mask_id, dtype=torch.int32)
    scfg = sp.cfg_from_synth(cfg)
    ws = sp.alloc_workspace(scfg, G, B, 0, DEV)
    got = sp.decode_head(scfg, x.to(DEV), gain.to(DEV), w.to(DEV), tok.to(DEV), 0.5, ws, force_one=False)
    if G * B <= sp.STATIC_MAX_ROWS:
        out = {k: torch.empty_like(t) for k, t in got.items()}
        sp.decode_head_static(scfg, x.to(DEV), gain.to(DEV), w.to(DEV), tok.to(DEV), 0.5, out, force_one=False)
        assert torch.equal(out["argmax"], got["argmax"]) and torch.allclose(out["conf"], got["conf"], rtol=1e-5)
    xn = to_np(x).reshape(-1, d)
    n = xn / np.sqrt((xn ** 2).mean(-1, keepdims=True) + 1e-5)
    logit = n @ to_np(w).T
    tie = 2 * (d + 16) * 2.0 ** -24 * (np.abs(n) @ np.abs(to_np(w)).T).max()
    top = np.sort(logit, -1)[:, ::-1]
    clear = top[:, 0] - top[:, 1] > tie             # the bound is a worst case: over 16000 terms it exceeds some margins
    am = got["argmax"].cpu().numpy().reshape(-1)
    assert clear.mean() > 0.5 and (am[clear] == logit.argmax(-1)[clear]).all()
    conf = 1.0 / np.exp(logit - top[:, :1]).sum(-1)
    np.testing.assert_allclose(to_np(got["conf"]).reshape(-1), conf, rtol=tie + V * 2.0 ** -24)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("last_masked", [False, True])
@pytest.mark.parametrize("G", [1, 2, 64, 65])
def test_head_rows_do_not_depend_on_how_the_masked_rows_are_listed(sp, G, last_masked, dtype):
    """Up to 8192 rows the norm's workgroups find their places in the row list themselves, above a list kernel runs first: every
    output of a state equals, bit for bit, that of the state alone; masked and unmasked last rows, a state without MASK."""
    B, d, V = 32, 256, 3000                            # fp32: the merge in slices; bf16: one merge, and the matrix-core head
    cfg = synth.CONFIGS["c1"].scaled(d=d, V=V, G=G, B=B, dtype=dtype)
    g = torch.Generator().manual_seed(G)
    td = cfg.torch_dtype()
    x, w = torch.randn((G, B, d), generator=g).to(td).to(DEV), (torch.randn((V, d), generator=g) * 0.1).to(td).to(DEV)
    gain = torch.ones(d).to(td).to(DEV)
    tok = torch.randint(0, V - 1, (G, B), generator=g, dtype=torch.int32)
    tok[torch.rand((G, B), generator=g) < 0.5] = cfg.mask_id
    if G > 1:
        tok[G // 2] = 1
    tok[G - 1, B - 1] = cfg.mask_id if last_masked else 1
    tok = tok.to(DEV)
    scfg = sp.cfg_from_synth(cfg)
    got = sp.decode_head(scfg, x, gain, w, tok, 0.01, sp.alloc_workspace(scfg, G, B, 0, DEV))
    one = sp.alloc_workspace(scfg, 1, B, 0, DEV)
    for s in sorted({0, G // 2, G - 1}):
        ref = sp.decode_head(scfg, x[s:s + 1].contiguous(), gain, w, tok[s:s + 1].contiguous(), 0.01, one)
        for k in ref:
            assert torch.equal(got[k][s], ref[k][0]), (s, k)


def test_head_rows_do_not_depend_on_the_batch_at_large_widths(sp):
    """128 rows of 16000 leave less of the static scratch than 100 summaries a row take: the vocabulary is cut alike there and
    for 160 rows."""
    d, V, G, B = 16000, 6400, 5, 32
    cfg = synth.CONFIGS["c1"].scaled(d=d, V=V, G=G, B=B)
    g = torch.Generator().manual_seed(3)
    x, w = torch.randn((G, B, d), generator=g).to(DEV), (torch.randn((V, d), generator=g) * 0.01).to(DEV)
    gain, tok = torch.ones(d).to(DEV), torch.full((G, B), cfg.mask_id, dtype=torch.int32).to(DEV)
    scfg = sp.cfg_from_synth(cfg)
    got = sp.decode_head(scfg, x, gain, w, tok, 0.01, sp.alloc_workspace(scfg, G, B, 0, DEV))
    few = sp.decode_head(scfg, x[:4].contiguous(), gain, w, tok[:4].contiguous(), 0.01, sp.alloc_workspace(scfg, 4, B, 0, DEV))
    for k in few:
        assert torch.equal(got[k][:4], few[k]), k
    out = {k: torch.empty_like(t) for k, t in few.items()}
    sp.decode_head_static(scfg, x[:4].contiguous(), gain, w, tok[:4].contiguous(), 0.01, out)
    for k in few:
        assert torch.equal(out[k], few[k]), k


@pytest.mark.parametrize("epi", ["store", "resid", "swiglu"])
def test_tile_gemm_rows_do_not_depend_on_the_batch_bf16(sp, epi):
    g = torch.Generator().manual_seed(6)
    A, W, W1, R = (torch.randn(s, generator=g).to(torch.bfloat16).to(DEV) for s in ((200, 520), (6008, 520), (6008, 520), (200, 6008)))

    def run(n):                                      # 200 rows: 64 x 64 tiles; 40: 32 x 16; 16 and fewer: 16 x 16
        a, r = A[:n].contiguous(), R[:n].contiguous()
        if epi == "swiglu":
            return sp.gemm(sp.GEMM_SWIGLU, a, W, W1)
        return sp.gemm(sp.GEMM_RESID, a, W, R=r) if epi == "resid" else sp.gemm(sp.GEMM_STORE, a, W)

    full = run(200)
    for n in (1, 16, 40):
        assert torch.equal(run(n), full[:n]), n


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hd,Hq,Hkv,P,S", [(64, 4, 4, 300, 0), (96, 8, 4, 130, 140), (64, 4, 4, 2000, 0), (136, 4, 4, 260, 0)])
def test_tile_attention_states_do_not_depend_on_the_batch(sp, hd, Hq, Hkv, P, S, dtype):
    """65 states of 16 tokens are more than 256 workgroups of attention, one or 64 states are not: a state's rows are the same bits;
    the first also against the oracle."""
    from oracle import spiffy_oracle as O
    B, G = 16, 65
    cfg = synth.CONFIGS["c1"].scaled(dtype=dtype, d=96, Hq=Hq, Hkv=Hkv, hd=hd, F=72, P=P, B=B, G=G)
    w = synth.layer_weights(cfg, 0, bias=True)
    for k in ("wq", "wk", "wv", "wo"):
        w[k] = (w[k].float() * 4).to(w[k].dtype)
    g = torch.Generator().manual_seed(hd + P)
    k, v = (torch.randn((Hkv, P + B + S, hd), generator=g).to(w["wq"].dtype) for _ in range(2))
    x = synth.hidden_states(cfg, G=G)
    scfg, lw, pk = sp.cfg_from_synth(cfg), sp.layer_weights({n: t.to(DEV) for n, t in w.items()}), sp.prefix_kv(k.to(DEV), v.to(DEV), P, S)

    def run(a, b):
        return sp.verify_layer(scfg, lw, pk, x[a:b].contiguous().to(DEV), P, sp.alloc_workspace(scfg, b - a, B, P + S, DEV)).clone()

    full = run(0, G)
    for a, b in ((0, 1), (G - 1, G), (1, G)):
        assert torch.equal(run(a, b), full[a:b]), (a, b)
    kn, vn = to_np(k), to_np(v)
    kw = dict(suffix_k=kn[:, P + B:], suffix_v=vn[:, P + B:]) if S else {}
    ref = O.verify_layer(np_weights(w), kn[:, :P], vn[:, :P], to_np(x[:2]), **cfg_kw(cfg), **kw)
    err = np.max(np.abs(to_np(full[:2]) - ref) / (np.abs(ref) + np.sqrt(np.mean(ref * ref))))
    assert err < (1e-4 if dtype == "f32" else 2e-2), err      # the bars of test_gpu_parity


@pytest.mark.parametrize("G", [1, 2, 65])
def test_head_merged_in_slices_does_not_depend_on_the_batch(sp, G):
    """bf16, 34 chunk summaries a row (more than the 32 that one launch merges): every output of a state, and the drafting source's
    tokens and probabilities, which start from the merged row, equal those of the state alone."""
    B, d, V = 32, 256, 4352 - 56
    cfg = synth.CONFIGS["c1"].scaled(d=d, V=V, G=G, B=B, dtype="bf16")
    g = torch.Generator().manual_seed(100 + G)
    x, w = torch.randn((G, B, d), generator=g).bfloat16().to(DEV), (torch.randn((V, d), generator=g) * 0.1).bfloat16().to(DEV)
    gain = torch.ones(d).bfloat16().to(DEV)
    tok = torch.randint(0, V - 1, (G, B), generator=g, dtype=torch.int32)
    tok[torch.rand((G, B), generator=g) < 0.5] = cfg.mask_id
    tok[0, 0] = tok[G - 1, B - 1] = cfg.mask_id
    tok = tok.to(DEV)
    scfg = sp.cfg_from_synth(cfg)
    ws, one = sp.alloc_workspace(scfg, G, B, 0, DEV), sp.alloc_workspace(scfg, 1, B, 0, DEV)
    got = sp.decode_head(scfg, x, gain, w, tok, 0.01, ws)
    for s in sorted({0, G - 1}):
        top = sp.head_topk(scfg, w, tok, 3, 1.0, ws, node=s)
        ts = tok[s:s + 1].contiguous()
        ref = sp.decode_head(scfg, x[s:s + 1].contiguous(), gain, w, ts, 0.01, one)
        for k in ref:
            assert torch.equal(got[k][s], ref[k][0]), (s, k)
        for a, b in zip(top, sp.head_topk(scfg, w, ts, 3, 1.0, one, node=0)):
            assert torch.equal(a, b), s


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("K", [8, 24, 32, 40, 64, 72, 104, 128, 136, 168, 192, 200, 256, 264, 328, 376, 384, 392])
def test_tile_gemm_short_k_rows_do_not_depend_on_the_batch(sp, K, dtype):
    """Up to six chunks of K (128 bytes of a row each) many rows take a wavefront a tile, few rows share one: same bits, at edges
    of the 32 x 32 tiles; and against the float64 product, |fp32 sum - exact| <= (K + 16) 2^-24 sum |a w|."""
    M, N = 513, 2024 if dtype == "f32" else 2088      # 32 x 128 columns of workgroups cut short; bf16 off the MFMA kernel
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(K)
    A, W, W1, R = ((torch.randn(s, generator=g) * f).to(td) for s, f in (((M, K), 1.0), ((N, K), 0.3), ((N, K), 0.3), ((M, N), 1.0)))
    a, w, w1, r = [t.to(DEV) for t in (A, W, W1, R)]
    full = [sp.gemm(sp.GEMM_STORE, a, w), sp.gemm(sp.GEMM_RESID, a, w, R=r), sp.gemm(sp.GEMM_SWIGLU, a, w, w1)]
    for n in (1, 16, 33):
        part = a[-n:].contiguous()
        few = [sp.gemm(sp.GEMM_STORE, part, w), sp.gemm(sp.GEMM_RESID, part, w, R=r[-n:].contiguous()), sp.gemm(sp.GEMM_SWIGLU, part, w, w1)]
        for x, y in zip(full, few):
            assert torch.equal(x[-n:], y), n
    ref, out = to_np(A) @ to_np(W).T, 2.0 ** -24 if dtype == "f32" else 1.02 * 2.0 ** -8
    assert (np.abs(to_np(full[0]) - ref) <= (K + 16) * 2.0 ** -24 * (np.abs(to_np(A)) @ np.abs(to_np(W)).T) + out * np.abs(ref) + 1e-30).all()


def test_layer_of_short_rows_with_masked_rows_only(sp):
    """A layer 64 wide with projections of many columns (one wavefront a tile), biases, and the last layer's device row count:
    the masked rows of the full layer, bit for bit."""
    G, B, P = 17, 32, 20
    cfg = synth.CONFIGS["c1"].scaled(dtype="f32", d=64, Hq=8, Hkv=8, hd=128, F=4104, P=P, B=B, G=G)
    scfg, w = sp.cfg_from_synth(cfg), {n: t.to(DEV) for n, t in synth.layer_weights(cfg, 0, bias=True).items()}
    g = torch.Generator().manual_seed(1)
    k, v = (torch.randn((8, P + B, 128), generator=g).to(DEV) for _ in range(2))
    x = synth.hidden_states(cfg, G=G).to(DEV)
    tok = torch.where(torch.rand((G, B), generator=g) < 0.9, cfg.mask_id, 1).to(torch.int32).to(DEV)
    lw, pk, ws = sp.layer_weights(w), sp.prefix_kv(k, v, P, 0), sp.alloc_workspace(scfg, G, B, P, DEV)
    full = sp.verify_layer(scfg, lw, pk, x, P, ws).clone()
    last = sp.verify_layer_last(scfg, lw, pk, x, tok, P, ws, torch.zeros_like(x))
    masked = tok == cfg.mask_id
    assert torch.equal(last[masked], full[masked])
    one = sp.verify_layer(scfg, lw, pk, x[3:4].contiguous(), P, sp.alloc_workspace(scfg, 1, B, P, DEV))
    assert torch.equal(one[0], full[3])


@pytest.mark.parametrize("G,last_masked", [(256, True), (256, False), (257, True), (257, False)])
def test_head_rows_at_the_line_between_the_two_row_lists(sp, G, last_masked):
    """8192 and 8224 rows: each state's outputs are those of the state alone, bit for bit."""
    B, d, V = 32, 64, 600
    cfg = synth.CONFIGS["c1"].scaled(d=d, V=V, G=G, B=B)
    g = torch.Generator().manual_seed(G)
    x, w = torch.randn((G, B, d), generator=g).to(DEV), (torch.randn((V, d), generator=g) * 0.1).to(DEV)
    gain, tok = torch.ones(d).to(DEV), torch.randint(0, V - 1, (G, B), generator=g, dtype=torch.int32)
    tok[torch.rand((G, B), generator=g) < 0.5] = cfg.mask_id
    tok[G // 2], tok[G - 1, B - 1] = 1, cfg.mask_id if last_masked else 1
    tok = tok.to(DEV)
    scfg = sp.cfg_from_synth(cfg)
    got = sp.decode_head(scfg, x, gain, w, tok, 0.01, sp.alloc_workspace(scfg, G, B, 0, DEV))
    one = sp.alloc_workspace(scfg, 1, B, 0, DEV)
    for s in (0, 1, G // 2, G - 2, G - 1):
        ref = sp.decode_head(scfg, x[s:s + 1].contiguous(), gain, w, tok[s:s + 1].contiguous(), 0.01, one)
        for k in ref:
            assert torch.equal(got[k][s], ref[k][0]), (s, k)
