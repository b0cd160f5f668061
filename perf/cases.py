"""The work that programs have libbpt do, as cases that can be timed and compared.

Kinds of case, each run through the package's public entry points:

  layer   one BPT layer: a training step (forward, then dX and every parameter gradient), a
          forward alone, or the forward that allocates nothing
  head    the LM head's cross-entropy, forward and backward
  gpt     forward and backward of a whole GPT
  adamw   one optimiser step
  ln      the final LayerNorm, forward and backward
  embed   token and position embedding, forward and backward

Shapes are those of bpt_inputs.WORKLOADS and of the GPT benchmark where they exist, else
generic widths. Weights are drawn at unit gain, activations and upstream gradients ~ N(0, 1),
tokens by a Zipf-like law (rank r with probability ~ 1/r), as text has them.
"""
from __future__ import annotations

import math

import torch

from paper_2305_19370_amd import bpt, gpt

DT = {"bf16": torch.bfloat16, "f32": torch.float32}

LAYER = dict(kind="layer", mode="train", dtype="bf16", out_dtype="bf16", causal=True, activation="gelu", affine=False,
             biases=False, dropout=0.0)


def _layer(name, B, S, D, H, F, Bq, **kw):
    return {"name": name, **LAYER, "B": B, "S": S, "D": D, "H": H, "F": F, "Bq": Bq, "Bkv": Bq, **kw}


def listed():
    return [
        # the float32 parity workload (bpt_inputs: fp32_s512_d256): what a float32 user trains and
        # checks a port with
        _layer("layer_f32_s512_d256", 1, 512, 256, 4, 1024, 128, dtype="f32", out_dtype="f32"),
        # latency: one short sequence through a serving loop that may not allocate
        _layer("layer_noalloc_s250_d1024", 1, 250, 1024, 8, 4096, 125, mode="noalloc"),
        # a small model's training layer on a few odd-length sequences, with every parameter
        # and heads of 64
        _layer("layer_b4_s1000_d768", 4, 1000, 768, 12, 3072, 500, affine=True, biases=True),
        # the GPT 1B-shaped training layer (bpt_inputs: bf16_1b_s4096)
        _layer("layer_1b_s4096", 2, 4096, 2048, 16, 8192, 512),
        # the GPT 7B-shaped training layer at 32K tokens, the default benchmark
        # (bpt_inputs: bf16_7b_s32768)
        _layer("layer_7b_s32768", 1, 32768, 4096, 32, 16384, 1024),
        # RL trajectories: 1000 steps of (return, state, action), residual dropout 0.1, ReLU
        # (eq. (2) as printed), all parameters; the layer shape of bpt_inputs' bf16_rl_s96000
        _layer("layer_rl_b8_s3000_dropout", 8, 3000, 1024, 8, 4096, 1000, activation="relu", affine=True, biases=True,
               dropout=0.1),
        # a forward alone (evaluation, encoding) without the causal mask, heads of 64; the layer of
        # bpt_inputs' bf16_dh64_nc_s32768 at a shorter length
        _layer("layer_fwd_dh64_nc_s8192", 1, 8192, 2048, 32, 8192, 1024, mode="fwd", causal=False),
        # the LM head of a 1B-shaped GPT on one batch of tokens, loss and both gradients
        {"name": "head_t8192_d2048_v50257", "kind": "head", "dtype": "bf16", "T": 8192, "D": 2048, "V": 50257},
        # forward and backward of a small GPT with every parameter, as its training loop calls them
        {"name": "gpt_l4_s1024_d768", "kind": "gpt", "dtype": "bf16", "L": 4, "B": 4, "S": 1024, "D": 768, "H": 12,
         "F": 3072, "V": 50257, "activation": "gelu", "biases": True, "pos_table": True},
        # optimiser step over the matrices of one 1B-shaped layer (float32 masters, bf16 copy)
        {"name": "adamw_n50331648", "kind": "adamw", "n": 12 * 2048 * 2048, "lowp": True},
        # final LayerNorm of the GPT-XL benchmark step: 16384 tokens
        {"name": "ln_t16384_d2048", "kind": "ln", "rows": 16384, "D": 2048, "dtype": "bf16", "out_dtype": "bf16",
         "affine": True},
        # embedding of the GPT-XL benchmark step: 16384 tokens, 50257 rows
        {"name": "embed_t16384_d2048_v50257", "kind": "embed", "dtype": "bf16", "B": 1, "S": 16384, "D": 2048, "V": 50257,
         "pos_table": True},
    ]


# ---------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _to(x, m, lo, hi):
    return max(lo, min(hi, (x + m // 2) // m * m))


def _draw_layer(rng):
    f32 = rng.random() < 0.25
    while True:
        dh = rng.choice((64, 128))
        D = _to(_log(rng, 128, 1024) if f32 else _log(rng, 256, 5120), dh, dh, 1024 if f32 else 5120)
        F = _to(int(D * rng.choice((2, 3, 4, 4))), 64, 64, 4 * D)
        S = _log(rng, 16, 1500 if f32 else 24000)
        if rng.random() < 0.4:
            S = _to(S, 64, 64, 24000)
        B = 1 if rng.random() < 0.4 else _log(rng, 1, max(1, min(16, (2000 if f32 else 32768) // S)))
        Bq, Bkv = min(S, _log(rng, 64, 1024)), min(S, _log(rng, 64, 1024))
        dtype = "f32" if f32 else "bf16"
        c = dict(LAYER, dtype=dtype, out_dtype=dtype if rng.random() < 0.7 else "f32", B=B, S=S, D=D, H=D // dh, F=F,
                 Bq=Bq, Bkv=Bkv, mode=rng.choice(("train", "train", "train", "fwd")), causal=rng.random() < 0.8,
                 activation="gelu" if rng.random() < 0.7 else "relu", affine=rng.random() < 0.5,
                 biases=rng.random() < 0.5, dropout=0.1 if rng.random() < 0.25 else 0.0)
        if work(c)["flops"] < (6e10 if f32 else 2e13):
            return c


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "layer", "head", "gpt", "adamw", "ln", "embed"))
    if kind == "layer":
        return _draw_layer(rng)
    if kind == "head":
        f32 = rng.random() < 0.2
        return {"kind": "head", "dtype": "f32" if f32 else "bf16", "T": _log(rng, 64, 1024 if f32 else 16384),
                "D": _to(_log(rng, 256, 512 if f32 else 4096), 64, 64, 4096), "V": _log(rng, 1000, 8000 if f32 else 50257)}
    if kind == "gpt":
        dh = rng.choice((64, 128))
        D = _to(_log(rng, 256, 1536), dh, dh, 1536)
        S = _log(rng, 100, 2048)
        return {"kind": "gpt", "dtype": "bf16", "L": rng.choice((1, 2, 3, 4)), "B": _log(rng, 1, max(1, min(8, 4096 // S))),
                "S": S, "D": D, "H": D // dh, "F": rng.choice((2, 4)) * D, "V": _log(rng, 1000, 50257),
                   "activation": "gelu", "biases": rng.random() < 0.7, "pos_table": rng.random() < 0.7}
    if kind == "adamw":
        return {"kind": "adamw", "n": _log(rng, 10_000, 100_000_000), "lowp": rng.random() < 0.8}
    if kind == "ln":
        dtype = "bf16" if rng.random() < 0.75 else "f32"
        return {"kind": "ln", "rows": _log(rng, 100, 60_000), "D": _to(_log(rng, 128, 8192), 8, 8, 8192), "dtype": dtype,
                "out_dtype": dtype, "affine": rng.random() < 0.8}
    S = _log(rng, 100, 16384)
    return {"kind": "embed", "dtype": "bf16" if rng.random() < 0.75 else "f32", "B": _log(rng, 1, max(1, 16384 // S)), "S": S,
            "D": _to(_log(rng, 128, 4096), 8, 8, 4096), "V": _log(rng, 1000, 50257), "pos_table": rng.random() < 0.7}


# ---------------------------------------------------------------- what a pass cannot do without
def _pairs(c):
    return c["B"] * c["H"] * (c["S"] * (c["S"] + 1) // 2 if c["causal"] else c["S"] * c["S"])


def _layer_flops(c):
    T, D, F = c["B"] * c["S"], c["D"], c["F"]
    return 8.0 * T * D * D + 4.0 * T * D * F + 4.0 * (D // c["H"]) * _pairs(c)


def work(case):
    c = case
    e = 2 if c.get("dtype") == "bf16" else 4
    if c["kind"] == "layer":
        T, D, F = c["B"] * c["S"], c["D"], c["F"]
        mats = 4 * D * D + 2 * D * F
        vecs = (4 * D if c["affine"] else 0) + (F + D if c["biases"] else 0)
        eo = 2 if c["out_dtype"] == "bf16" else 4
        fwd = T * D * (e + eo) + mats * e + vecs * 4
        if c["mode"] != "train":
            return {"bytes": fwd, "flops": _layer_flops(c)}
        return {"bytes": fwd + T * D * (e + eo) + 4 * (mats + vecs), "flops": 3.0 * _layer_flops(c)}
    if c["kind"] == "head":
        T, D, V = c["T"], c["D"], c["V"]
        return {"bytes": 2 * T * D * e + D * V * (e + 4) + 8 * T, "flops": 6.0 * T * D * V}
    if c["kind"] == "gpt":
        T, D, F, V, L = c["B"] * c["S"], c["D"], c["F"], c["V"], c["L"]
        n = L * (4 * D * D + 2 * D * F) + 2 * D * V
        return {"bytes": (e + 4) * n, "flops": 3.0 * (L * _layer_flops(dict(c, causal=True)) + 2.0 * T * D * V)}
    if c["kind"] == "adamw":
        return {"bytes": c["n"] * (28 + (2 if c["lowp"] else 0)), "flops": 14.0 * c["n"]}
    if c["kind"] == "ln":
        n = c["rows"] * c["D"]
        return {"bytes": 5 * n * e, "flops": 20.0 * n}     # X and dY read, Y and dX written; X read by both directions
    T, D, V = c["B"] * c["S"], c["D"], c["V"]
    pos = c["S"] * D if c["pos_table"] else 0
    return {"bytes": T * D * 3 * e + pos * (e + 4) + V * D * 4, "flops": 2.0 * T * D}


def tolerance(case):
    """What another order of the sums gives between two implementations at the same precision."""
    if case["kind"] == "adamw":          # elementwise; a last-bit change may flip the rounding of a bf16 copy
        return {"rel": 1e-4, "max": 1e-2} if case["lowp"] else {"rel": 1e-5, "max": 1e-4}
    if case["kind"] == "embed":          # dWte sums in any order; X is one rounding of an exact sum
        return {"rel": 1e-5, "max": 1e-3}
    if case.get("activation") == "relu" and case["mode"] == "train":
        # a z near 0 that changes sign takes its whole token out of a gradient column
        return {"rel": 1e-3, "max": 0.3} if case["dtype"] == "f32" else {"rel": 3e-2, "max": 0.9}
    if case["dtype"] == "f32":
        return {"rel": 2e-5, "max": 1e-3}
    if case["kind"] == "ln":             # a last-bit change of a statistic flips bf16 roundings
        return {"rel": 2e-3, "max": 1e-2}
    if case["kind"] == "gpt":
        return {"rel": 3e-2, "max": 0.5}
    return {"rel": 1e-2, "max": 0.1}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return lambda *s, std=1.0, dt=torch.float32: torch.randn(s, generator=g, device="cuda").mul_(std).to(dt)


def _zipf(T, V, seed):
    """T int32 indices in [0, V), index r with probability ~ 1 / (r + 1)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    u = torch.rand(T, generator=g, device="cuda", dtype=torch.float64)
    return (torch.pow(float(V + 1), u) - 1.0).long().clamp_(0, V - 1).to(torch.int32)


def _layer_inputs(c, seed):
    rn, dt = _gen(seed), DT[c["dtype"]]
    B, S, D, F = c["B"], c["S"], c["D"], c["F"]
    p = {n: rn(D, D, std=D ** -0.5, dt=dt) for n in ("Wq", "Wk", "Wv", "Wo")}
    p["W1"], p["W2"] = rn(D, F, std=D ** -0.5, dt=dt), rn(F, D, std=F ** -0.5, dt=dt)
    for n in ("ln1_g", "ln1_b", "ln2_g", "ln2_b"):
        p[n] = rn(D, std=0.1) + (1.0 if n.endswith("_g") else 0.0) if c["affine"] else None
    p["b1"], p["b2"] = (rn(F, std=0.1), rn(D, std=0.1)) if c["biases"] else (None, None)
    return rn(B, S, D, dt=dt), p, rn(B, S, D, dt=dt)


def _gpt_std(c, name):
    return 0.02 / math.sqrt(2 * c["L"]) if name.endswith((".Wo", ".W2")) else 0.02


def _gpt_shapes(c):
    D, F, V, ldw = c["D"], c["F"], c["V"], (c["V"] + 63) // 64 * 64
    out = {"Wte": (V, D), **({"Wpe": (c["S"], D)} if c["pos_table"] else {}), "Wout": (D, ldw), "lnf_g": (D,), "lnf_b": (D,)}
    for l in range(c["L"]):
        out.update({f"{l}.{n}": (D, D) for n in ("Wq", "Wk", "Wv", "Wo")})
        out.update({f"{l}.W1": (D, F), f"{l}.W2": (F, D)})
        out.update({f"{l}.{n}": (D,) for n in ("ln1_g", "ln1_b", "ln2_g", "ln2_b")})
        if c["biases"]:
            out.update({f"{l}.b1": (F,), f"{l}.b2": (D,)})
    return out


def _gpt_inputs(c, seed):
    """Float32 parameters by name, tokens and targets."""
    rn, p = _gen(seed), {}
    for name, shape in _gpt_shapes(c).items():
        if len(shape) == 2:
            p[name] = rn(*shape, std=_gpt_std(c, name))
        else:
            p[name] = rn(*shape, std=0.1) + (1.0 if name.endswith("_g") else 0.0)
    p["Wout"][:, c["V"]:] = 0.0
    T = c["B"] * c["S"]
    return p, _zipf(T, c["V"], seed + 1), _zipf(T, c["V"], seed + 2)


def _head_inputs(c, seed):
    rn, dt, ldw = _gen(seed), DT[c["dtype"]], (c["V"] + 63) // 64 * 64
    W = rn(c["D"], ldw, std=2.0 * c["D"] ** -0.5)
    W[:, c["V"]:] = 0.0
    return rn(c["T"], c["D"], dt=dt), W.to(dt), _zipf(c["T"], c["V"], seed + 1)


def _adamw_inputs(c, seed):
    rn = _gen(seed)
    n = c["n"]
    return rn(n, std=0.02), rn(n, std=1e-3), rn(n, std=3e-4), rn(n, std=1e-3).square_()


def _ln_inputs(c, seed):
    rn, D = _gen(seed), c["D"]
    g, b = (rn(D, std=0.1) + 1.0, rn(D, std=0.1)) if c["affine"] else (None, None)
    return rn(c["rows"], D, dt=DT[c["dtype"]]), g, b, rn(c["rows"], D, dt=DT[c["out_dtype"]])


def _embed_inputs(c, seed):
    rn, dt = _gen(seed), DT[c["dtype"]]
    T, D = c["B"] * c["S"], c["D"]
    return (_zipf(T, c["V"], seed + 1), rn(c["V"], D, std=0.02, dt=dt),
            rn(c["S"], D, std=0.02, dt=dt) if c["pos_table"] else None, rn(T, D, std=1e-3, dt=dt))


def _bytes(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    c = case
    if c["kind"] == "layer":
        X, p, dY = _layer_inputs(c, seed)
        cfg = bpt.make_config(c["B"], c["S"], c["D"], c["H"], c["F"], c["Bq"], c["Bkv"], causal=c["causal"],
                              dtype=c["dtype"], out_dtype=c["out_dtype"], activation=c["activation"],
                              dropout=c["dropout"], dropout_seed=1234)
        st = {"case": c, "cfg": cfg, "layer": bpt.Layer(cfg), "X": X, "p": p}
        if c["mode"] == "noalloc":
            st["Y"] = torch.empty(X.shape, dtype=DT[c["out_dtype"]], device="cuda")
            st["saved"] = _bytes(bpt.saved_bytes(cfg))
        else:
            st["ws"] = _bytes(max(bpt.workspace_bytes(cfg, False),
                                  bpt.workspace_bytes(cfg, True) if c["mode"] == "train" else 0))
        if c["mode"] == "train":
            st["dY"] = dY
        return st
    if c["kind"] == "head":
        h, W, tgt = _head_inputs(c, seed)
        return {"case": c, "head": bpt.LMHeadLoss(bpt.make_xent_config(c["T"], c["D"], c["V"], dtype=c["dtype"])), "h": h,
                "W": W, "tgt": tgt}
    if c["kind"] == "gpt":
        p, tok, tgt = _gpt_inputs(c, seed)
        bq = min(1024, c["S"])
        m = gpt.GPT(gpt.GPTShape(c["L"], c["B"], c["S"], c["D"], c["H"], c["F"], c["V"], Bq=bq, Bkv=bq, dtype=c["dtype"],
                                 activation=c["activation"], biases=c["biases"], pos_table=c["pos_table"]), init=False)
        for name, v in p.items():
            m.master(name).copy_(v)
        m.sync_lowp()
        return {"case": c, "m": m, "tok": tok, "tgt": tgt}
    if c["kind"] == "adamw":
        p, g, m, v = _adamw_inputs(c, seed)
        return {"case": c, "p": p, "g": g, "m": m, "v": v, "low": p.to(torch.bfloat16) if c["lowp"] else None}
    if c["kind"] == "ln":
        X, g, b, dY = _ln_inputs(c, seed)
        cfg = bpt.make_ln_config(c["rows"], c["D"], in_dtype=c["dtype"], out_dtype=c["out_dtype"])
        return {"case": c, "cfg": cfg, "X": X, "g": g, "b": b, "dY": dY, "Y": torch.empty_like(dY),
                "dX": torch.empty_like(X), "mean": torch.empty(c["rows"], device="cuda"),
                "rstd": torch.empty(c["rows"], device="cuda"), "dg": torch.empty(c["D"], device="cuda"),
                "db": torch.empty(c["D"], device="cuda"), "ws": _bytes(bpt.ln_workspace_bytes(cfg))}
    tok, Wte, Wpe, dX = _embed_inputs(c, seed)
    cfg = bpt.make_embed_config(c["B"], c["S"], c["D"], c["V"], dtype=c["dtype"])
    return {"case": c, "cfg": cfg, "tok": tok, "Wte": Wte, "Wpe": Wpe, "dX": dX, "X": torch.empty_like(dX),
            "dWte": torch.empty(Wte.shape, device="cuda"),
            "dWpe": torch.empty(Wpe.shape, device="cuda") if Wpe is not None else None}


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "layer":
        if c["mode"] == "noalloc":
            bpt.layer_fwd_noalloc(s["cfg"], s["X"], s["p"], s["Y"], s["saved"])
            return {"Y": s["Y"]}
        Y, saved = s["layer"].forward(s["X"], s["p"], workspace=s["ws"])
        if c["mode"] == "fwd":
            return {"Y": Y}
        dX, grads = s["layer"].backward(s["X"], s["p"], saved, s["dY"], workspace=s["ws"])
        return {"Y": Y, "dX": dX, **grads}
    if c["kind"] == "head":
        loss, lse = s["head"].forward(s["h"], s["W"], s["tgt"])
        dh, dW = s["head"].backward(s["h"], s["W"], s["tgt"], lse)
        return {"loss": loss, "lse": lse, "dh": dh, "dW": dW}
    if c["kind"] == "gpt":
        m = s["m"]
        loss = m.forward(s["tok"], s["tgt"])
        m.backward(s["tok"], s["tgt"])
        return {"loss": loss, "lse": m.lse, **{n: m.grad(n) for n in m.names()}}
    if c["kind"] == "adamw":
        bpt.adamw_step(s["p"], s["g"], s["m"], s["v"], step=10, lr=2e-4, p_lowp=s["low"])
        return {"p": s["p"], "m": s["m"], "v": s["v"], **({"low": s["low"]} if c["lowp"] else {})}
    if c["kind"] == "ln":
        bpt.ln_fwd(s["cfg"], s["X"], s["g"], s["b"], s["Y"], s["mean"], s["rstd"])
        bpt.ln_bwd(s["cfg"], s["X"], s["g"], s["mean"], s["rstd"], s["dY"], s["dX"], s["dg"], s["db"], s["ws"])
        return {n: s[n] for n in ("Y", "mean", "rstd", "dX", "dg", "db")}
    bpt.embed_fwd(s["cfg"], s["tok"], s["Wte"], s["Wpe"], s["X"])
    bpt.embed_bwd(s["cfg"], s["tok"], s["dX"], s["dWte"], s["dWpe"])
    return {"X": s["X"], "dWte": s["dWte"], **({"dWpe": s["dWpe"]} if s["Wpe"] is not None else {})}


# ---------------------------------------------------------------- the same in 64 bits, plain torch
_M32 = 0xFFFFFFFF


def _keep(T, D, site, rate, seed):
    """Dropout factors [T, D] of a branch: Philox4x32-10 at counter (n / 4, t, site, 0)."""
    n, t = torch.arange(D // 4, device="cuda").expand(T, -1), torch.arange(T, device="cuda")[:, None].expand(-1, D // 4)
    c0, c1, c2, c3 = n, t, torch.full_like(n, site), torch.zeros_like(n)
    k0, k1 = seed & _M32, seed >> 32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57      # 64-bit products, as bits
        c0, c1, c2, c3 = ((b >> 32) & _M32) ^ c1 ^ k0, b & _M32, ((a >> 32) & _M32) ^ c3 ^ k1, a & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    rate = float(torch.tensor(rate, dtype=torch.float32))
    kept = torch.stack((c0, c1, c2, c3), -1).reshape(T, D) >= int(rate * 4294967296.0)
    return kept.double() / (1.0 - rate)


def _ln64(x, g, b, eps=1e-5):
    mu = x.mean(1, keepdim=True)
    rs = (x.var(1, unbiased=False, keepdim=True) + eps).rsqrt()
    xh = (x - mu) * rs
    y = xh if g is None else xh * g + b
    return y, xh, mu, rs


def _ln64_bwd(dy, xh, rs, g):
    gd = dy if g is None else dy * g
    return rs * (gd - gd.mean(1, keepdim=True) - xh * (gd * xh).mean(1, keepdim=True))


def _attn64(q, k, v, causal, do=None):
    """One head [S, dh]: the output, or (dq, dk, dv) for an upstream do."""
    S, dh = q.shape
    out = torch.empty_like(q)
    if do is not None:
        dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    for a in range(0, S, 8192):
        e = min(S, a + 8192)
        n = e if causal else S
        s = q[a:e] @ k[:n].t().contiguous()
        s /= math.sqrt(dh)
        if causal:
            s.masked_fill_(torch.arange(n, device="cuda")[None] > torch.arange(a, e, device="cuda")[:, None], -math.inf)
        p = torch.softmax(s, 1)
        if do is None:
            out[a:e] = p @ v[:n]
            continue
        dp = do[a:e] @ v[:n].t().contiguous()
        dv[:n] += p.t() @ do[a:e]
        dp -= (p * dp).sum(1, keepdim=True)
        dp *= p
        dp /= math.sqrt(dh)
        out[a:e] = dp @ k[:n]
        dk[:n] += dp.t() @ q[a:e]
    return out if do is None else (out, dk, dv)


def _layer64_fwd(c, X, p):
    """X [T, D]; every tensor in 64 bits. Y and what the backward needs."""
    T, D = X.shape
    B, H, S, dh = c["B"], c["H"], T // c["B"], D // c["H"]
    u, xh1, _, rs1 = _ln64(X, p["ln1_g"], p["ln1_b"])
    q, k, v = u @ p["Wq"], u @ p["Wk"], u @ p["Wv"]
    o = torch.empty_like(q)
    for b in range(B):
        for h in range(H):
            r, f = slice(b * S, (b + 1) * S), slice(h * dh, (h + 1) * dh)
            o[r, f] = _attn64(q[r, f].contiguous(), k[r, f].contiguous(), v[r, f].contiguous(), c["causal"])
    m0 = _keep(T, D, 0, c["dropout"], 1234) if c["dropout"] else 1.0
    m1 = _keep(T, D, 1, c["dropout"], 1234) if c["dropout"] else 1.0
    hd = X + (o @ p["Wo"]) * m0
    w, xh2, _, rs2 = _ln64(hd, p["ln2_g"], p["ln2_b"])
    z = w @ p["W1"]
    if p["b1"] is not None:
        z += p["b1"]
    if c["activation"] == "relu":
        cdf, G = (z > 0).double(), z.clamp_min(0)
    else:
        cdf = 0.5 + 0.5 * torch.erf(z / math.sqrt(2.0))
        G = z * cdf
    f = G @ p["W2"]
    if p["b2"] is not None:
        f += p["b2"]
    return hd + f * m1, (u, xh1, rs1, q, k, v, o, m0, m1, w, xh2, rs2, z, cdf, G)


def _layer64_bwd(c, p, keep, dY):
    u, xh1, rs1, q, k, v, o, m0, m1, w, xh2, rs2, z, cdf, G = keep
    T, D = dY.shape
    B, H, S, dh = c["B"], c["H"], T // c["B"], D // c["H"]
    g = {}
    dF = dY * m1
    g["db2"] = dF.sum(0)
    g["dW2"] = G.t() @ dF
    dz = dF @ p["W2"].t()
    if c["activation"] != "relu":
        cdf = cdf + z * torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)
    dz *= cdf
    g["db1"], g["dW1"] = dz.sum(0), w.t() @ dz
    dw = dz @ p["W1"].t()
    g["dln2_g"], g["dln2_b"] = (dw * xh2).sum(0), dw.sum(0)
    dh_ = dY + _ln64_bwd(dw, xh2, rs2, p["ln2_g"])
    da = dh_ * m0
    g["dWo"] = o.t() @ da
    do = da @ p["Wo"].t()
    dq, dk, dv = (torch.empty_like(q) for _ in range(3))
    for b in range(B):
        for h in range(H):
            r, f = slice(b * S, (b + 1) * S), slice(h * dh, (h + 1) * dh)
            dq[r, f], dk[r, f], dv[r, f] = _attn64(*(t[r, f].contiguous() for t in (q, k, v)), c["causal"],
                                                   do[r, f].contiguous())
    g["dWq"], g["dWk"], g["dWv"] = u.t() @ dq, u.t() @ dk, u.t() @ dv
    du = dq @ p["Wq"].t() + dk @ p["Wk"].t() + dv @ p["Wv"].t()
    g["dln1_g"], g["dln1_b"] = (du * xh1).sum(0), du.sum(0)
    for n in ("ln1_g", "ln1_b", "ln2_g", "ln2_b", "b1", "b2"):
        if p[n] is None:
            del g["d" + n]
    return dh_ + _ln64_bwd(du, xh1, rs1, p["ln1_g"]), g


def _head64(h, W, V, tgt):
    """loss, lse, dh, dW of 64-bit h [T, D] and W [D, ldw], a block of tokens at a time."""
    T = h.shape[0]
    Wv = W[:, :V].contiguous()
    lse, loss = torch.empty(T, dtype=torch.float64, device="cuda"), 0.0
    dh, dW = torch.empty_like(h), torch.zeros_like(W)
    for a in range(0, T, 4096):
        e = min(T, a + 4096)
        z = h[a:e] @ Wv
        lse[a:e] = torch.logsumexp(z, 1)
        y = tgt[a:e].long()[:, None]
        loss = loss + (lse[a:e] - z.gather(1, y)[:, 0]).sum()
        z -= lse[a:e, None]
        z.exp_()
        z.scatter_add_(1, y, torch.full(y.shape, -1.0, dtype=torch.float64, device="cuda"))
        z /= T
        dh[a:e] = z @ Wv.t()
        dW[:, :V] += h[a:e].t() @ z
    return (loss / T).reshape(1), lse, dh, dW


def _d(p):
    return {n: (v.double() if v is not None else None) for n, v in p.items()}


def exact(case, seed):
    c = case
    if c["kind"] == "layer":
        X, p, dY = _layer_inputs(c, seed)
        p, T, D = _d(p), c["B"] * c["S"], c["D"]
        Y, keep = _layer64_fwd(c, X.double().view(T, D), p)
        if c["mode"] != "train":
            return {"Y": Y.view(X.shape)}
        dX, g = _layer64_bwd(c, p, keep, dY.double().view(T, D))
        return {"Y": Y.view(X.shape), "dX": dX.view(X.shape), **g}
    if c["kind"] == "head":
        h, W, tgt = _head_inputs(c, seed)
        loss, lse, dh, dW = _head64(h.double(), W.double(), c["V"], tgt)
        return {"loss": loss, "lse": lse, "dh": dh, "dW": dW}
    if c["kind"] == "gpt":
        p, tok, tgt = _gpt_inputs(c, seed)
        dt = DT[c["dtype"]]
        p = {n: (v.to(dt) if v.dim() == 2 else v).double() for n, v in p.items()}
        lc, T, D = dict(c, causal=True, dropout=0.0), c["B"] * c["S"], c["D"]
        x = p["Wte"][tok.long()]
        if c["pos_table"]:
            x = x + p["Wpe"].repeat(c["B"], 1)
        keeps, lps = [], []
        for l in range(c["L"]):
            lps.append({n: p.get(f"{l}.{n}") for n in ("ln1_g", "ln1_b", "Wq", "Wk", "Wv", "Wo", "ln2_g", "ln2_b", "W1", "b1",
                                                       "W2", "b2")})
            x, keep = _layer64_fwd(lc, x, lps[l])
            keeps.append(keep)
        hf, xh, _, rs = _ln64(x, p["lnf_g"], p["lnf_b"])
        loss, lse, dh, dW = _head64(hf, p["Wout"], c["V"], tgt)
        out = {"loss": loss, "lse": lse, "Wout": dW, "lnf_g": (dh * xh).sum(0), "lnf_b": dh.sum(0)}
        d = _ln64_bwd(dh, xh, rs, p["lnf_g"])
        for l in range(c["L"] - 1, -1, -1):
            d, g = _layer64_bwd(lc, lps[l], keeps[l], d)
            out.update({f"{l}.{n[1:]}": v for n, v in g.items()})
        out["Wte"] = torch.zeros_like(p["Wte"]).index_add_(0, tok.long(), d)
        if c["pos_table"]:
            out["Wpe"] = d.view(c["B"], c["S"], D).sum(0)
        return out
    if c["kind"] == "adamw":
        p, g, m, v = (t.double() for t in _adamw_inputs(c, seed))
        lr, b1, b2, eps, wd = (float(torch.tensor(x, dtype=torch.float32)) for x in (2e-4, 0.9, 0.95, 1e-8, 0.1))
        m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
        p = p * (1 - lr * wd) - lr * (m / (1 - b1 ** 10)) / ((v / (1 - b2 ** 10)).sqrt() + eps)
        return {"p": p, "m": m, "v": v, **({"low": p} if c["lowp"] else {})}
    if c["kind"] == "ln":
        X, g, b, dY = _ln_inputs(c, seed)
        g, b = (t.double() if t is not None else None for t in (g, b))
        Y, xh, mu, rs = _ln64(X.double(), g, b)
        dY = dY.double()
        return {"Y": Y, "mean": mu[:, 0], "rstd": rs[:, 0], "dX": _ln64_bwd(dY, xh, rs, g), "dg": (dY * xh).sum(0),
                "db": dY.sum(0)}
    tok, Wte, Wpe, dX = _embed_inputs(c, seed)
    X = Wte.double()[tok.long()]
    out = {"dWte": torch.zeros(Wte.shape, dtype=torch.float64, device="cuda").index_add_(0, tok.long(), dX.double())}
    if Wpe is not None:
        X = X + Wpe.double().repeat(c["B"], 1)
        out["dWpe"] = dX.double().view(c["B"], c["S"], c["D"]).sum(0)
    return {"X": X, **out}
