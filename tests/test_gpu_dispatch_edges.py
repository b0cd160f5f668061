"""Sizes at the edges of kernel tiles and of the rules that choose between kernels, against
the float64 oracle under the gates of tests/gpu_util.py."""
import pytest
import torch

import oracle
from bpt_inputs import make_inputs, small_workload
from gpu_util import run_gpu, run_oracle, say
from paper_2305_19370_amd import bpt
from test_gpu_parity import compare_all

pytestmark = pytest.mark.gpu


# fp32: attention blocks of 16 rows shared by 4 waves (S around 16 and 64, one token), GEMM
# tiles of 32, 64 and 128 (the largest from 256 tiles of 128 x 128 on: the FFN of the last case)
@pytest.mark.parametrize("B,S,D,H,F,causal", [
    (1, 1, 128, 2, 64, True), (3, 15, 128, 1, 192, True), (2, 17, 192, 3, 256, False), (1, 65, 256, 2, 320, True),
    (2, 129, 128, 2, 512, False), (1, 1100, 512, 4, 1024, True), (1, 2048, 256, 2, 2048, True)])
def test_f32_tile_edges(B, S, D, H, F, causal):
    w = small_workload("f32", B=B, S=S, D=D, H=H, F=F, causal=causal, Bq=min(S, 64), Bkv=min(S, 64))
    inp = make_inputs(w, seed=3, affine=True, biases=True)
    say(f"case {w.name}")
    gpu = run_gpu(w, inp, qkv_grads=True)
    Yr, _, g = run_oracle(w, inp)
    compare_all(w, inp, gpu, Yr, g, "fp32", w.name)


# token embedding gradient: rows owned by workgroups, tokens in chunks of 16384 and lists of 2048, rows named
# by many tokens of a list spanning the waves, columns in slices of 512
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,D,V", [(1, 8, 1), (33, 504, 3), (8192, 520, 2), (8193, 64, 257), (16385, 1032, 50),
                                   (3000, 512, 70001), (40000, 512, 3)])
def test_embedding_gradient(dtype, T, D, V):
    say(f"case embed {dtype} T={T} D={D} V={V}")
    g = torch.Generator().manual_seed(5)
    tok = torch.pow(float(V + 1), torch.rand(T, generator=g)).long().sub_(1).clamp_(0, V - 1)   # low ids frequent
    tok[::7] = V                                      # outside the vocabulary: adds nothing
    tok[3::11] = -1
    dX = torch.randn(T, D, generator=g).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    cfg = bpt.make_embed_config(1, T, D, V, dtype=dtype)
    outs = []
    for _ in range(2):
        dWte = torch.full((V, D), float("nan"), device="cuda")
        bpt.embed_bwd(cfg, tok.int().cuda(), dX.cuda(), dWte, None)
        outs.append(dWte.cpu())
    assert torch.equal(outs[0], outs[1])              # fixed order of the sums
    ok = (tok >= 0) & (tok < V)
    ref = torch.zeros(V, D, dtype=torch.float64).index_add_(0, tok[ok], dX[ok].double())
    # n additions in float32: error <= n 2^-24 sum |terms|
    mag = torch.zeros(V, D, dtype=torch.float64).index_add_(0, tok[ok], dX[ok].double().abs())
    n = torch.bincount(tok[ok], minlength=V).double()[:, None]
    assert ((outs[0].double() - ref).abs() <= n * 2.0 ** -24 * mag).all()


# final LayerNorm: rows in one wave (up to 512, 1024, 1536 / 2048 columns), in four waves (up
# to 4096, 6144, 8192), or walked (beyond); a partial last group of 512 columns; few rows and
# more rows than workgroups
@pytest.mark.parametrize("in_dtype,out_dtype", [("bf16", "bf16"), ("f32", "f32"), ("bf16", "f32"), ("f32", "bf16")])
@pytest.mark.parametrize("rows,D,affine", [(1, 8, True), (4100, 512, True), (9, 520, True), (700, 1544, False),
                                           (33, 2048, True), (4099, 2056, True), (5, 4104, True), (17, 6152, True),
                                           (40, 8192, False), (40, 8200, True)])
def test_final_layernorm(in_dtype, out_dtype, rows, D, affine):
    say(f"case ln {in_dtype}->{out_dtype} rows={rows} D={D} affine={affine}")
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}
    g = torch.Generator().manual_seed(7)
    X = (torch.randn(rows, D, generator=g) + 0.5).to(dt[in_dtype])
    dY = torch.randn(rows, D, generator=g).to(dt[out_dtype])
    gam = torch.randn(D, generator=g) * 0.1 + 1 if affine else None
    bet = torch.randn(D, generator=g) * 0.1 if affine else None
    dev = lambda t: None if t is None else t.cuda()
    cfg = bpt.make_ln_config(rows, D, in_dtype=in_dtype, out_dtype=out_dtype)
    Xg, dYg, gg, bg = dev(X), dev(dY), dev(gam), dev(bet)
    Y, dX = torch.empty_like(dYg), torch.empty_like(Xg)
    mean, rstd, dg, db = (torch.empty(n, device="cuda") for n in (rows, rows, D, D))
    ws = torch.empty(bpt.ln_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    bpt.ln_fwd(cfg, Xg, gg, bg, Y, mean, rstd)
    bpt.ln_bwd(cfg, Xg, gg, mean, rstd, dYg, dX, dg, db, ws)
    x = X.double().requires_grad_()
    gr = (gam.double() if affine else torch.ones(D, dtype=torch.float64)).requires_grad_()
    br = (bet.double() if affine else torch.zeros(D, dtype=torch.float64)).requires_grad_()
    y = torch.nn.functional.layer_norm(x, (D,), gr, br, 1e-5)
    y.backward(dY.double())
    for name, got, ref, od in (("Y", Y, y.detach(), out_dtype), ("dX", dX, x.grad, in_dtype), ("dg", dg, gr.grad, "f32"),
                               ("db", db, br.grad, "f32")):
        # float32 sums (1e-4 of the RMS, the fp32 gate) and, for a bf16 result, half an ulp
        lim = 1e-4 * ref.square().mean().sqrt() + (2.0 ** -8 * ref.abs() if od == "bf16" else 1e-5 * ref.abs())
        assert ((got.cpu().double() - ref).abs() <= lim).all(), name


# LayerNorm backward with an fp32 dY: partial sums of as many workgroups as fill the chip, and of
# the 128 that the least workspace holds; rows in one wave and in four
@pytest.mark.parametrize("in_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,D", [(4100, 512), (2300, 2056), (5, 4096), (1025, 8)])
def test_layernorm_backward_workspaces(in_dtype, rows, D):
    say(f"case ln bwd {in_dtype} rows={rows} D={D}")
    g = torch.Generator().manual_seed(8)
    X = (torch.randn(rows, D, generator=g) + 0.5).to(torch.bfloat16 if in_dtype == "bf16" else torch.float32).cuda()
    dY, gam = torch.randn(rows, D, generator=g).cuda(), (torch.randn(D, generator=g) * 0.1 + 1).cuda()
    cfg = bpt.make_ln_config(rows, D, in_dtype=in_dtype, out_dtype="f32")
    Y, mean, rstd = torch.empty_like(dY), torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    bpt.ln_fwd(cfg, X, gam, None, Y, mean, rstd)
    xh = (X.double() - mean.double()[:, None]) * rstd.double()[:, None]
    ref = {"dg": (dY.double() * xh).sum(0), "db": dY.double().sum(0)}
    mag = {"dg": (dY.double() * xh).abs().sum(0), "db": dY.double().abs().sum(0)}
    outs = []
    for n in (bpt.ln_workspace_bytes(cfg), 1024 * D):
        ws = torch.empty(n + 256, dtype=torch.uint8, device="cuda")
        ws[n:] = 77
        dX = torch.empty_like(X)
        out = {n_: torch.full((D,), float("nan"), device="cuda") for n_ in ("dg", "db")}
        bpt.ln_bwd(cfg, X, gam, mean, rstd, dY, dX, out["dg"], out["db"], ws[:n])
        assert (ws[n:] == 77).all()
        for name in out:              # a sum of `rows` terms in float32, each of an xhat of three roundings
            assert ((out[name].double() - ref[name]).abs() <= (rows + 3) * 2.0 ** -24 * mag[name]).all(), name
        outs.append(dX)
    assert torch.equal(*outs)


# bf16 weight gradients over the whole batch: sequences padded to 64 columns in one operand and
# not in the other, K of any length (T not a multiple of 32), K cut into slices, dWq, dWk, dWv
# as one product (D % 128 == 0) or three, sequences shorter than a stage
@pytest.mark.parametrize("B,S,D,H,F,causal", [
    (7, 1, 256, 2, 256, True), (5, 33, 256, 2, 512, True), (3, 100, 320, 5, 448, False), (9, 95, 128, 1, 192, True),
    (2, 1000, 768, 6, 1536, True), (4, 320, 512, 8, 1024, False)])
def test_bf16_weight_gradients_ragged(B, S, D, H, F, causal):
    w = small_workload("bf16", B=B, S=S, D=D, H=H, F=F, causal=causal, Bq=min(S, 128), Bkv=min(S, 128))
    inp = make_inputs(w, seed=11, affine=True, biases=True)
    say(f"case {w.name}")
    gpu = run_gpu(w, inp, qkv_grads=True)
    Yr, _, g = run_oracle(w, inp)
    compare_all(w, inp, gpu, Yr, g, "bf16", w.name)


# weight gradients cut along K, whose slices wait in buffers of the backward that are idle then: one
# FFN group and several, dWq, dWk, dWv as one product and (D = 192 in bf16) one at a time, and slices
# that do not fit the idle buffers (the last case); `slices`: products that are cut, which the
# profiler counts by their additions. Only these products are compared: the gate on the mean error
# holds for matrices (a vector of 128 column sums, as dln1_b here, is above it with any order of sums)
@pytest.mark.parametrize("dtype,B,S,D,H,F,groups,slices", [
    ("bf16", 2, 2000, 256, 4, 1024, 0, 4), ("bf16", 3, 1300, 128, 1, 256, 1, 8), ("bf16", 1, 4100, 192, 3, 256, 0, 6),
    ("f32", 2, 2000, 256, 2, 512, 1, 6), ("f32", 3, 1300, 128, 2, 256, 0, 4), ("f32", 6, 500, 704, 11, 128, 1, 2)])
def test_weight_gradient_slices(dtype, B, S, D, H, F, groups, slices):
    w = small_workload(dtype, B=B, S=S, D=D, H=H, F=F, Bq=S, Bkv=S)
    inp = make_inputs(w, seed=19, affine=True, biases=True)
    say(f"case {w.name} groups={groups}")
    bpt.profile_enable(True)
    gpu = run_gpu(w, inp, group_blocks=groups, qkv_grads=True)
    bpt.profile_enable(False)
    assert bpt.profile_report()["reduce.ksplit"]["count"] == slices
    gpu = {n: t for n, t in gpu.items() if t.dim() > 1}
    Yr, _, g = run_oracle(w, inp)
    compare_all(w, inp, gpu, Yr, g, "fp32" if dtype == "f32" else "bf16", w.name)


# few rows: FFN2, dv, dU and, with the fewest, Wo and dO cut along K, whose slices one kernel adds with
# residual and bias; more slices than the room holds (500 x 3072, 700 x 2048: as many as fit)
@pytest.mark.parametrize("dtype,S,D,H,F,slices", [
    ("bf16", 64, 1536, 12, 1536, 5), ("bf16", 250, 1024, 8, 4096, 3), ("bf16", 130, 640, 5, 2560, 3),
    ("bf16", 500, 3072, 24, 6144, 3), ("f32", 700, 2048, 16, 2048, 5)])
def test_few_row_slices(dtype, S, D, H, F, slices):
    w = small_workload(dtype, B=1, S=S, D=D, H=H, F=F, Bq=S, Bkv=S, init="unit")
    inp = make_inputs(w, seed=23, affine=True, biases=True)
    say(f"case {w.name}")
    bpt.profile_enable(True)
    gpu = run_gpu(w, inp)
    bpt.profile_enable(False)
    assert bpt.profile_report()["reduce.ksplit"]["count"] == slices
    low = run_gpu(w, inp, out_dtype="bf16")           # the same sums, rounded once
    assert all(torch.equal(low[n], gpu[n].bfloat16().float()) for n in ("Y", "dX"))
    cfg = bpt.make_config(1, S, D, H, F, S, S, w.causal, dtype, "f32")
    dev = {n: v.cuda() for n, v in inp.items()}
    Y = torch.empty(dev["X"].shape, device="cuda")
    saved = torch.empty(bpt.saved_bytes(cfg), dtype=torch.uint8, device="cuda")
    bpt.layer_fwd_noalloc(cfg, dev["X"], dev, Y, saved)            # the same slices in the static scratch
    assert torch.equal(Y.cpu(), gpu["Y"])
    Yr, _, g = run_oracle(w, inp)
    compare_all(w, inp, gpu, Yr, g, "fp32" if dtype == "f32" else "bf16", w.name)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_some_gradients_only(dtype):
    """A gradient asked for alone equals the one of a full backward up to the order of its sums."""
    w = small_workload(dtype, B=3, S=150, D=256, H=2, F=512)
    inp = make_inputs(w, seed=2, affine=True, biases=True)
    dev = {k: v.cuda() for k, v in inp.items()}
    layer = bpt.Layer(bpt.make_config(w.B, w.S, w.D, w.H, w.F, w.Bq, w.Bkv, w.causal, dtype, "f32"))
    _, saved = layer.forward(dev["X"], dev)
    dX, full = layer.backward(dev["X"], dev, saved, dev["dY"])
    for want in (("dWk",), ("dWq", "dWv", "dln1_g"), ("dln2_b", "db1", "dW2")):
        dX1, some = layer.backward(dev["X"], dev, saved, dev["dY"], want=want)
        assert torch.equal(dX, dX1) and set(some) == set(want)
        for n in want:                # float32 sums of the same terms in another order
            assert (some[n] - full[n]).abs().max() <= 1e-5 * full[n].abs().max(), n


# head: summaries of 64 columns in tiles of 256 and 128 (few and many rows), a last group with one
# column of the vocabulary, dh cut along the vocabulary (narrow D) with and without the room for it
@pytest.mark.parametrize("T,D,V", [(1, 64, 1), (70, 128, 449), (300, 192, 12801), (2100, 128, 8000)])
def test_head_edges(T, D, V):
    from bpt_inputs import make_xent_inputs
    say(f"case head T={T} D={D} V={V}")
    cfg = bpt.make_xent_config(T, D, V)
    inp = {k: v.cuda() for k, v in make_xent_inputs(T, D, V, cfg.ldw, seed=4).items()}
    h, W, y = inp["h"], inp["W"], inp["targets"]
    head = bpt.LMHeadLoss(cfg)
    loss, lse = head.forward(h, W, y)
    dh, dW = head.backward(h, W, y, lse, dloss=0.5)
    z = h.double() @ W.double()[:, :V].contiguous()
    ref = torch.logsumexp(z, 1)
    assert (lse.double() - ref).abs().max() <= 1e-4 * ref.abs().max().clamp_min(1.0)
    tok = ref - z.gather(1, y.long()[:, None])[:, 0]
    assert (loss.double() - tok.mean()).abs().max() <= 1e-4 * ref.abs().max().clamp_min(1.0)
    G = torch.softmax(z, 1)
    G[torch.arange(T, device="cuda"), y.long()] -= 1.0
    G = (G * (0.5 / T)).to(torch.bfloat16).double()        # the operand of both products
    # exp in float32 may round an element of G to the neighbouring bf16 value: 2^-8 of it
    for got, want, mag in ((dh, G @ W.double()[:, :V].t(), G.abs() @ W.double()[:, :V].abs().t()),
                           (dW[:, :V], h.double().t().contiguous() @ G, h.double().abs().t().contiguous() @ G.abs())):
        assert ((got.double() - want).abs() <= 2.0 ** -8 * mag + 2.0 ** -8 * want.abs() + 1e-12).all()
    small = torch.empty(cfg.ldw * ((min(T, 8192) + 63) // 64 * 64) * 2, dtype=torch.uint8, device="cuda")
    dh1 = torch.empty_like(dh)
    bpt.xent_bwd(cfg, h, W, y, lse, 0.5, dh1, None, small)
    assert ((dh1.double() - dh.double()).abs() <= 2.0 ** -7 * dh.double().abs() + 1e-4 * dh.double().abs().max()).all()


# bf16 products whose 64 x 64 tiles share K among four groups of waves (by the rule's arithmetic): Wo with
# residual, FFN1, its recomputation, dZ and dO; dWo, both operands K-major; Q, K and V one by one; with dropout,
# Wo and FFN2 stored in fp32
@pytest.mark.parametrize("B,S,D,H,F,dropout", [(1, 121, 2816, 22, 512, 0.0), (2, 500, 320, 5, 320, 0.0),
                                               (1, 60, 2112, 33, 128, 0.0), (1, 64, 2560, 20, 2560, 0.1)])
def test_products_that_share_k(B, S, D, H, F, dropout):
    w = small_workload("bf16", B=B, S=S, D=D, H=H, F=F, Bq=S, Bkv=S, init="unit")
    inp = make_inputs(w, seed=29, affine=True, biases=True)
    say(f"case {w.name} dropout {dropout}")
    gpu = run_gpu(w, inp, qkv_grads=True, dropout=dropout, dropout_seed=5)
    p = oracle.params_from_inputs(inp)
    p.dropout, p.dropout_seed = dropout, 5
    Yr, cache = oracle.layer_fwd(inp["X"].double().numpy(), p, w.H, w.causal)
    g = oracle.layer_bwd(cache, p, inp["dY"].double().numpy())
    compare_all(w, inp, gpu, Yr, g, "bf16", w.name, dropout=dropout, dropout_seed=5)


# bf16 attention blocks of 128 rows (few blocks) and of 256 (many): edges of both, ragged last
# block and tile, heads of 64 and 128
@pytest.mark.parametrize("B,S,D,H,causal", [(1, 127, 256, 2, True), (1, 129, 128, 2, True), (2, 385, 256, 2, False),
                                            (1, 64, 128, 1, False), (20, 193, 896, 14, True), (11, 320, 768, 6, False)])
def test_bf16_attention_blocks(B, S, D, H, causal):
    w = small_workload("bf16", B=B, S=S, D=D, H=H, F=128, causal=causal, Bq=64, Bkv=64)
    inp = make_inputs(w, seed=13)
    say(f"case {w.name}")
    gpu = run_gpu(w, inp, qkv_grads=True)
    Yr, _, g = run_oracle(w, inp)
    compare_all(w, inp, gpu, Yr, g, "bf16", w.name)


# the two block sizes give the same bits: one sequence alone runs blocks of 128 rows, as one of many
# it runs blocks of 256 (LN, residual and products of a row do not depend on the others; the products here
# take no form that shares K)
@pytest.mark.parametrize("D,H,causal", [(256, 4, True), (256, 2, True), (256, 2, False)])
def test_attention_block_sizes_agree(D, H, causal):
    S, B = 300, 90 if H == 4 else 150
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(31)
    rn = lambda *s: torch.randn(*s, generator=g, device=dev)
    X = rn(B, S, D).bfloat16()
    p = {n: (rn(D, D) * D ** -0.5).bfloat16() for n in ("Wq", "Wk", "Wv", "Wo")}
    p["W1"], p["W2"] = (rn(D, 64) * D ** -0.5).bfloat16(), (rn(64, D) * 0.125).bfloat16()
    dY = rn(B, S, D).bfloat16()
    outs = []
    for b in (1, B):
        cfg = bpt.make_config(b, S, D, H, 64, S, S, causal, "bf16", "f32")
        rows = bpt.describe(cfg)
        assert ("attention: q-tile=128" if b == 1 else "attention: q-tile=256") in rows, rows
        layer = bpt.Layer(cfg)
        Xb = X[:b].contiguous()
        Y, saved = layer.forward(Xb, p)
        _, grads = layer.backward(Xb, p, saved, dY[:b].contiguous(), qkv_grads=True)
        v = layer.saved_views(saved)
        outs.append([v["qkv"][:S], v["o"][:S], v["lse"][:1], *(grads[n][:1] for n in ("dQ", "dK", "dV"))])
    for name, a, c in zip(("qkv", "o", "lse", "dQ", "dK", "dV"), *outs):
        assert torch.equal(a[..., :S] if name == "lse" else a, c[..., :S] if name == "lse" else c), name


# residual dropout: the mask of dh applied inside the LN2 backward (rows in one wave and in four)
@pytest.mark.parametrize("dtype,D,H", [("f32", 192, 3), ("bf16", 192, 3), ("bf16", 2176, 17)])
def test_dropout_gradient_rows(dtype, D, H):
    w = small_workload(dtype, B=2, S=70, D=D, H=H, F=128, Bq=64, Bkv=64, init="unit")
    inp = make_inputs(w, seed=17, affine=True, biases=True)
    say(f"case {w.name} dropout")
    gpu = run_gpu(w, inp, qkv_grads=True, dropout=0.1, dropout_seed=99)
    p = oracle.params_from_inputs(inp)
    p.dropout, p.dropout_seed = 0.1, 99
    Yr, cache = oracle.layer_fwd(inp["X"].double().numpy(), p, w.H, w.causal)
    g = oracle.layer_bwd(cache, p, inp["dY"].double().numpy())
    compare_all(w, inp, gpu, Yr, g, "fp32" if dtype == "f32" else "bf16", w.name, dropout=0.1, dropout_seed=99)
