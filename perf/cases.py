"""The work that the performance of this framework is judged by.

Every case is one call sequence that a training program makes through the
binding of the C ABI: whole stage steps (forward, recompute, backward) and the
layers they are made of (attention, the linear layers' GEMMs in their three
directions with their fused epilogues, LayerNorm and bias gradients), at the
shapes of the workloads in ``paper_2206_04959_amd/synth.py``.

A case is a dict of plain values; ``kind`` names the call and the other keys
are its sizes.  Inputs are drawn on the GPU from the seed alone, with the value
recipe of ``synth.py`` (weights and biases N(0, 0.02), LayerNorm gamma around
1, hidden states and upstream gradients N(0, 1)).
"""
from __future__ import annotations

import math

import torch

from paper_2206_04959_amd import binding as B
from paper_2206_04959_amd import flops, synth

DEV = "cuda"


def listed():
    return [
        # The benchmark workload: one step of the 8.3B-shaped shard at
        # tensor-parallel degree 4 (8 x 1024 tokens, half of its blocks
        # recomputed, four sub-micro-batches on two streams).
        _stage_case("stage-8.3b-tp4", synth.GPT_8_3B),
        # A whole step without recomputation on a ragged width (hidden 1600,
        # 25 heads of 64): most GEMM grids end in partial tiles.
        _stage_case("stage-1.5b", synth.GPT_1_5B),
        # The smallest whole call, in the fp32 mode a user checks a model with:
        # launches and latency, not bandwidth.
        _stage_case("stage-tiny-fp32", synth.TINY),
        # Attention forward of one stream's share of the 8.3B-shaped shard.
        {"name": "attn-fwd-4x1024x8x96", "kind": "attn_fwd", "batch": 4, "seq": 1024, "heads": 8, "d": 96,
         "dtype": "bf16"},
        # Attention backward of one stream's share of the 20B-shaped shard
        # (2048-token sequences, 6 local heads of 128).
        {"name": "attn-bwd-2x2048x6x128", "kind": "attn_bwd", "batch": 2, "seq": 2048, "heads": 6, "d": 128,
         "dtype": "bf16"},
        # A short odd sequence (five 64-row blocks, 5 heads of 64): the
        # smallest calls, where a launch's latency is most of the time.
        {"name": "attn-fwd-1x320x5x64", "kind": "attn_fwd", "batch": 1, "seq": 320, "heads": 5, "d": 64,
         "dtype": "bf16"},
        # FC1 forward of the 8.3B-shaped shard: bias + GeLU, both outputs kept.
        {"name": "fc1-fwd-4096x3072x3072", "kind": "gemm_gelu", "m": 4096, "n": 3072, "k": 3072},
        # Projection forward of the 1.5B-shaped stage: ragged in every
        # dimension, bias + residual, partial sum handed off.
        {"name": "proj-fwd-2048x1600x1600", "kind": "gemm_resid", "m": 2048, "n": 1600, "k": 1600},
        # Projection input gradient of the 8.3B-shaped shard: narrow output,
        # long reduction.
        {"name": "proj-dx-4096x768x3072", "kind": "gemm_dx", "m": 4096, "n": 768, "k": 3072},
        # FC2 weight gradient of the 2.5B-shaped shard, added to the gradients
        # of the micro-batches before it.
        {"name": "fc2-dw-1920x3840x4096", "kind": "gemm_dw", "m": 1920, "n": 3840, "k": 4096},
        # LayerNorm forward of one sub-micro-batch of the 1.5B-shaped stage.
        {"name": "ln-fwd-2048x1600", "kind": "ln_fwd", "rows": 2048, "h": 1600},
        # LayerNorm backward with its parameter gradients, one stream's share
        # of the 8.3B-shaped shard.
        {"name": "ln-bwd-4096x3072", "kind": "ln_bwd", "rows": 4096, "h": 3072},
    ]


def _stage_case(name, s):
    return {"name": name, "kind": "stage", "blocks": s.n_blocks, "hidden": s.hidden, "heads": s.n_heads,
            "ffn": s.ffn, "seq": s.seq_len, "batch": s.micro_batch, "tp": s.tp_degree, "n_sub": s.n_sub,
            "mask": s.recompute_mask, "dtype": s.dtype, "x_std": s.x_std}


def _log64(rng, lo, hi):
    """A multiple of 64 in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, 64 * round(v / 64)))


def draw(rng):
    kind = rng.choice(["stage", "stage_fp32", "attn_fwd", "attn_bwd", "attn_bwd", "gemm_bias", "gemm_gelu",
                       "gemm_resid", "gemm_dx", "gemm_gelu_dx", "gemm_dw", "ln_fwd", "ln_bwd", "column_sum"])
    if kind in ("stage", "stage_fp32"):
        # a stage of GPT blocks: widths and splits a tensor-parallel shard can have
        fp32 = kind == "stage_fp32"
        d = rng.choice([64, 96, 128])
        tp = rng.choice([1, 2]) if fp32 else rng.choice([1, 2, 4])
        step = tp * (64 // math.gcd(64, d))       # heads per rank make hidden/tp a multiple of 64
        heads = step * rng.randint(1, 2 if fp32 else max(1, 3072 // (d * step)))
        hidden = heads * d
        n_sub = rng.choice([1, 2] if fp32 else [1, 2, 4])
        blocks = 1 if fp32 else rng.randint(1, 4)
        return {"kind": "stage", "blocks": blocks, "hidden": hidden, "heads": heads, "ffn": 4 * hidden,
                "seq": 64 * rng.randint(1, 3) if fp32 else 64 * rng.randint(2, 16),
                "batch": n_sub * rng.randint(1, 2), "tp": tp, "n_sub": n_sub,
                "mask": 0 if fp32 else (1 << rng.randint(0, blocks)) - 1,
                "dtype": "fp32" if fp32 else "bf16", "x_std": 0.02 if fp32 else 1.0}
    if kind in ("attn_fwd", "attn_bwd"):
        return {"kind": kind, "batch": rng.randint(1, 4), "seq": _log64(rng, 64, 2048), "heads": rng.randint(1, 25),
                "d": rng.choice([64, 96, 128]), "dtype": "bf16"}
    if kind.startswith("gemm"):
        m, n, k = _log64(rng, 512, 8192), _log64(rng, 256, 6400), _log64(rng, 256, 6400)
        if kind == "gemm_dw":  # output features x input features, summed over the tokens
            m, n, k = n, k, m
        return {"kind": kind, "m": m, "n": n, "k": k}
    rows = round(math.exp(rng.uniform(math.log(100), math.log(8192))))
    return {"kind": kind, "rows": rows, "h": _log64(rng, 256, 6144)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
        v = torch.randn(*shape, generator=self.g, device=DEV, dtype=torch.float32)
        return v.mul_(std).add_(mean).to(dtype)


_side = []


def _streams():
    """The program's two streams, made once."""
    if not _side:
        _side.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    return _side


def _shape(c):
    return synth.StageShape("case", n_blocks=c["blocks"], hidden=c["hidden"], n_heads=c["heads"], ffn=c["ffn"],
                            seq_len=c["seq"], micro_batch=c["batch"], tp_degree=c["tp"], n_sub=c["n_sub"],
                            recompute_mask=c["mask"], dtype=c["dtype"], x_std=c["x_std"])


def _dtype(c):
    return torch.float32 if c.get("dtype", "bf16") == "fp32" else torch.bfloat16


def _stage_inputs(c, seed):
    s = _shape(c)
    dt = _dtype(c)
    r = _Draws(seed)
    cfg = B.make_config(s)
    total, offs = B.param_layout(cfg)
    params = torch.zeros(total, dtype=dt, device=DEV)
    for l in range(s.n_blocks):
        for i, (name, shp) in enumerate(s.local_param_shapes().items()):
            n = math.prod(shp)
            o = int(offs[l, i])
            params[o:o + n] = r.normal(n, std=s.w_std, mean=1.0 if name in ("ln1_g", "ln2_g") else 0.0, dtype=dt)
    x = r.normal(s.micro_batch, s.seq_len, s.hidden, std=s.x_std, dtype=dt)
    dy = r.normal(s.micro_batch, s.seq_len, s.hidden, dtype=dt)
    return s, cfg, total, offs, params, x, dy


def _attn_inputs(c, seed):
    """qkv, and for the backward the forward's o (rounded) and lse and the gradient dO."""
    r = _Draws(seed)
    b, s, h, d = c["batch"], c["seq"], c["heads"], c["d"]
    # LayerNorm output times N(0, 0.02) weights over a hidden size of 3072: std near 1.1
    qkv = r.normal(b, s, 3, h, d, std=1.1)
    if c["kind"] == "attn_fwd":
        return qkv, None, None, None
    o, lse = _attention(qkv.float())
    return qkv, o.to(torch.bfloat16), lse, r.normal(b, s, h, d)


def _attention(qkv):
    """Plain causal attention in the precision of qkv: o [b, s, h, d], lse [b, h, s]."""
    b, s, _, h, d = qkv.shape
    q, k, v = (qkv[:, :, i].permute(0, 2, 1, 3).contiguous() for i in range(3))
    kt = k.transpose(2, 3).contiguous()
    sc = torch.matmul(q, kt) / math.sqrt(d)
    sc.masked_fill_(torch.ones(s, s, dtype=torch.bool, device=qkv.device).triu_(1), -math.inf)
    lse = torch.logsumexp(sc, dim=-1)
    o = torch.matmul(torch.exp(sc - lse.unsqueeze(-1)), v)
    return o.permute(0, 2, 1, 3).contiguous(), lse.contiguous()


_GEMM = {"gemm_bias": (B.EPI_BIAS, False, False), "gemm_gelu": (B.EPI_BIAS_GELU, False, False),
         "gemm_resid": (B.EPI_BIAS_RESID, False, False), "gemm_dx": (B.EPI_STORE, False, True),
         "gemm_gelu_dx": (B.EPI_GELU_BWD, False, True), "gemm_dw": (B.EPI_F32, True, True)}


def _gemm_inputs(c, seed):
    r = _Draws(seed)
    m, n, k = c["m"], c["n"], c["k"]
    epi, a_t, b_t = _GEMM[c["kind"]]
    g = {"a": r.normal(k, m) if a_t else r.normal(m, k), "bias": None, "resid": None, "aux": None}
    if c["kind"] == "gemm_dw":   # dY^T X added to the gradients so far
        g["b"] = r.normal(k, n)
        g["c"] = r.normal(m, n, dtype=torch.float32)
        return g
    g["b"] = r.normal(k, n, std=0.02) if b_t else r.normal(n, k, std=0.02)
    g["c"] = torch.empty(m, n, dtype=torch.bfloat16, device=DEV)
    if epi in (B.EPI_BIAS, B.EPI_BIAS_GELU, B.EPI_BIAS_RESID):
        g["bias"] = r.normal(n, std=0.02)
    if epi == B.EPI_BIAS_RESID:
        g["resid"] = r.normal(m, n)
    if epi in (B.EPI_BIAS_GELU, B.EPI_BIAS_RESID):
        g["aux"] = torch.empty(m, n, dtype=torch.bfloat16, device=DEV)
    if epi == B.EPI_GELU_BWD:
        g["aux"] = r.normal(m, n)
    return g


def _ln_inputs(c, seed):
    r = _Draws(seed)
    rows, h = c["rows"], c["h"]
    x = r.normal(rows, h, std=1.4, mean=0.05)
    t = {"x": x, "gamma": r.normal(h, std=0.02, mean=1.0), "beta": r.normal(h, std=0.02)}
    if c["kind"] == "ln_bwd":
        xd = x.double()
        mu = xd.mean(1)
        t["mean"] = mu.float()
        t["rstd"] = torch.rsqrt((xd - mu[:, None]).square().mean(1) + 1e-5).float()
        t["dout"], t["dres"] = r.normal(rows, h), r.normal(rows, h)
    return t


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def prepare(c, seed):
    kind = c["kind"]
    empty = lambda *s, dtype=torch.bfloat16: torch.empty(*s, dtype=dtype, device=DEV)  # noqa: E731
    if kind == "stage":
        s, cfg, total, _, params, x, dy = _stage_inputs(c, seed)
        part = (s.n_blocks, 2, s.tokens, s.hidden)
        return {"kind": kind, "stage": B.Stage(s), "params": params, "x": x, "dy": dy, "y": torch.empty_like(x),
                "dx": torch.empty_like(x), "grads": empty(total, dtype=torch.float32).zero_(),
                "fwd_partials": empty(*part, dtype=x.dtype), "bwd_partials": empty(*part, dtype=x.dtype),
                "streams": _streams()}
    if kind in ("attn_fwd", "attn_bwd"):
        qkv, o, lse, dout = _attn_inputs(c, seed)
        b, s, h, d = c["batch"], c["seq"], c["heads"], c["d"]
        st = {"kind": kind, "dims": (b, s, h, d), "qkv": qkv, "o": o, "lse": lse, "dout": dout}
        if kind == "attn_fwd":
            st["o"], st["lse"] = empty(b, s, h, d), empty(b, h, s, dtype=torch.float32)
        else:
            st["dqkv"], st["delta"] = torch.empty_like(qkv), empty(b, h, s, dtype=torch.float32)
        return st
    if kind in _GEMM:
        return {"kind": kind, "mnk": (c["m"], c["n"], c["k"]), **_gemm_inputs(c, seed)}
    rows, h = c["rows"], c["h"]
    st = {"kind": kind, **_ln_inputs(c, seed)}
    if kind == "ln_fwd":
        st.update(y=empty(rows, h), mean=empty(rows, dtype=torch.float32), rstd=empty(rows, dtype=torch.float32))
    elif kind == "ln_bwd":
        st.update(dx=empty(rows, h), dgamma=empty(h, dtype=torch.float32), dbeta=empty(h, dtype=torch.float32),
                  scratch=empty(2 * B.reduce_scratch_elems(rows, h), dtype=torch.float32))
    else:
        st.update(out=empty(h, dtype=torch.float32),
                  scratch=empty(B.reduce_scratch_elems(rows, h), dtype=torch.float32))
    return st


def run(st):
    kind = st["kind"]
    if kind == "stage":
        s0, s1 = st["streams"]
        cur = torch.cuda.current_stream()
        s0.wait_stream(cur)
        st["stage"].fwd(st["params"], st["x"], st["y"], st["fwd_partials"], streams=(s0, s1))
        st["stage"].recompute(st["params"], streams=(s0, s1))
        st["stage"].bwd(st["params"], st["dy"], st["dx"], st["grads"], False, st["bwd_partials"], streams=(s0, s1))
        cur.wait_stream(s0)
        return {k: st[k] for k in ("y", "dx", "grads", "fwd_partials", "bwd_partials")}
    if kind == "attn_fwd":
        B.attention_fwd(st["qkv"], st["o"], st["lse"], *st["dims"])
        return {"o": st["o"], "lse": st["lse"]}
    if kind == "attn_bwd":
        B.attention_bwd(st["qkv"], st["o"], st["lse"], st["dout"], st["dqkv"], st["delta"], *st["dims"])
        return {"dqkv": st["dqkv"]}
    if kind in _GEMM:
        epi, a_t, b_t = _GEMM[kind]
        B.gemm(st["a"], st["b"], st["c"], *st["mnk"], a_trans=a_t, b_trans=b_t, epilogue=epi, bias=st["bias"],
               resid=st["resid"], aux=st["aux"], accumulate=epi == B.EPI_F32)
        return {"c": st["c"], "aux": st["aux"] if epi in (B.EPI_BIAS_GELU, B.EPI_BIAS_RESID) else None}
    if kind == "ln_fwd":
        B.layernorm_fwd(st["x"], st["gamma"], st["beta"], st["y"], st["mean"], st["rstd"])
        return {k: st[k] for k in ("y", "mean", "rstd")}
    if kind == "ln_bwd":
        B.layernorm_bwd(st["dout"], st["x"], st["mean"], st["rstd"], st["gamma"], st["dres"], st["dx"], st["dgamma"],
                        st["dbeta"], st["scratch"])
        return {k: st[k] for k in ("dx", "dgamma", "dbeta")}
    B.column_sum(st["x"], st["out"], st["scratch"])
    return {"out": st["out"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def work(c):
    kind = c["kind"]
    if kind == "stage":
        s = _shape(c)
        e = 4 if s.dtype == "fp32" else 2
        params = s.n_blocks * sum(math.prod(v) for v in s.local_param_shapes().values())
        act = s.tokens * s.hidden
        # parameters, x and dy in; y, dx, the partial sums and the fp32 gradients out
        return {"bytes": params * (e + 4) + e * act * (4 + 4 * s.n_blocks), "flops": flops.executed_flops(s)}
    if kind in ("attn_fwd", "attn_bwd"):
        b, s, h, d = c["batch"], c["seq"], c["heads"], c["d"]
        f, row = 2.0 * b * h * d * s * (s + 1), b * s * h * d * 2
        if kind == "attn_fwd":
            return {"bytes": 4 * row + 4 * b * h * s, "flops": f}
        return {"bytes": 8 * row + 4 * b * h * s, "flops": 2 * f}
    if kind in _GEMM:
        m, n, k = c["m"], c["n"], c["k"]
        out = {"gemm_gelu": 4, "gemm_resid": 6, "gemm_gelu_dx": 4, "gemm_dw": 8}.get(kind, 2)
        return {"bytes": 2 * (m * k + k * n) + out * m * n, "flops": 2.0 * m * n * k}
    rows, h = c["rows"], c["h"]
    passes, per_elem = {"ln_fwd": (2, 8), "ln_bwd": (4, 12), "column_sum": (1, 1)}[kind]
    return {"bytes": passes * rows * h * 2 + 8 * rows, "flops": float(per_elem * rows * h)}


# ---------------------------------------------------------------------------
# Tolerance and the same results in 64 bits
# ---------------------------------------------------------------------------

def tolerance(c):
    kind = c["kind"]
    if kind == "stage":
        # Measured against 64 bits: 1.2e-6 in fp32; 1e-2 in bf16, whose rounding
        # travels through every block.
        return {"rel": 1e-5} if c["dtype"] == "fp32" else {"rel": 3e-2, "max": 0.5}
    if kind in ("gemm_dw", "column_sum"):
        return {"rel": 1e-5}  # fp32 results of fp32 sums
    return {"rel": 1e-2}      # bf16 results: 1.7e-3 to 2.3e-3 against 64 bits


def exact(c, seed):
    kind = c["kind"]
    if kind == "stage":
        return _exact_stage(c, seed)
    if kind in ("attn_fwd", "attn_bwd"):
        return _exact_attention(c, seed)
    if kind in _GEMM:
        return _exact_gemm(c, seed)
    t = {k: v.double() for k, v in _ln_inputs(c, seed).items()}
    x = t["x"]
    if kind == "column_sum":
        return {"out": x.sum(0)}
    if kind == "ln_fwd":
        mu = x.mean(1)
        rs = torch.rsqrt((x - mu[:, None]).square().mean(1) + 1e-5)
        return {"y": (x - mu[:, None]) * rs[:, None] * t["gamma"] + t["beta"], "mean": mu, "rstd": rs}
    xh = (x - t["mean"][:, None]) * t["rstd"][:, None]
    dxh = t["dout"] * t["gamma"]
    dx = t["dres"] + t["rstd"][:, None] * (dxh - dxh.mean(1, keepdim=True) - xh * (dxh * xh).mean(1, keepdim=True))
    return {"dx": dx, "dgamma": (t["dout"] * xh).sum(0), "dbeta": t["dout"].sum(0)}


def _gelu(u):
    return 0.5 * u * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (u + 0.044715 * u ** 3)))


def _exact_gemm(c, seed):
    kind = c["kind"]
    g = {k: None if v is None else v.double() for k, v in _gemm_inputs(c, seed).items()}
    _, a_t, b_t = _GEMM[kind]
    a = g["a"].t().contiguous() if a_t else g["a"]
    b = g["b"] if b_t else g["b"].t().contiguous()
    acc = torch.matmul(a, b)
    if kind == "gemm_dw":
        return {"c": g["c"] + acc, "aux": None}
    if kind == "gemm_bias":
        return {"c": acc + g["bias"], "aux": None}
    if kind == "gemm_gelu":
        return {"c": _gelu(acc + g["bias"]), "aux": acc + g["bias"]}
    if kind == "gemm_resid":
        return {"c": g["resid"] + acc + g["bias"], "aux": acc}
    if kind == "gemm_gelu_dx":
        u = g["aux"].requires_grad_()
        return {"c": acc * torch.autograd.grad(_gelu(u).sum(), u)[0], "aux": None}
    return {"c": acc, "aux": None}


def _exact_attention(c, seed):
    qkv, o, lse, dout = _attn_inputs(c, seed)
    qkv = qkv.double()
    if c["kind"] == "attn_fwd":
        o, lse = _attention(qkv)
        return {"o": o, "lse": lse}
    heads = lambda t: t.double().permute(0, 2, 1, 3).contiguous()  # noqa: E731
    q, k, v = (heads(qkv[:, :, i]) for i in range(3))
    do, scale = heads(dout), 1.0 / math.sqrt(c["d"])
    tr = lambda t: t.transpose(2, 3).contiguous()  # noqa: E731
    s = c["seq"]
    p = torch.matmul(q, tr(k)).mul_(scale).sub_(lse.double().unsqueeze(-1)).exp_()
    p.masked_fill_(torch.ones(s, s, dtype=torch.bool, device=DEV).triu_(1), 0.0)
    dv = torch.matmul(tr(p), do)
    ds = p * (torch.matmul(do, tr(v)) - (do * heads(o)).sum(-1, keepdim=True))
    dq, dk = torch.matmul(ds, k) * scale, torch.matmul(tr(ds), q) * scale
    back = lambda t: t.permute(0, 2, 1, 3)  # noqa: E731
    return {"dqkv": torch.stack([back(dq), back(dk), back(dv)], dim=2).contiguous()}


def _exact_stage(c, seed):
    s, _, total, offs, params, x, dy = _stage_inputs(c, seed)
    L, T, h, hl = s.n_blocks, s.tokens, s.hidden, s.local_hidden
    w = params.double()
    shapes = s.local_param_shapes()
    par = [{n: w[int(offs[l, i]):int(offs[l, i]) + math.prod(shp)].reshape(shp).clone().requires_grad_()
            for i, (n, shp) in enumerate(shapes.items())} for l in range(L)]
    norm = lambda t, g, b: torch.nn.functional.layer_norm(t, (h,), g, b, s.ln_eps)  # noqa: E731
    x0 = x.double().reshape(T, h).requires_grad_()
    cur, keep = x0, []
    for p in par:
        ln1 = norm(cur, p["ln1_g"], p["ln1_b"])
        qkv = (torch.matmul(ln1, p["w_qkv"].t()) + p["b_qkv"]).reshape(s.micro_batch, s.seq_len, 3, s.local_heads, -1)
        p_o = torch.matmul(_attention(qkv)[0].reshape(T, hl), p["w_o"].t())
        x1 = cur + p_o + p["b_o"]
        ln2 = norm(x1, p["ln2_g"], p["ln2_b"])
        p_f = torch.matmul(_gelu(torch.matmul(ln2, p["w1"].t()) + p["b1"]), p["w2"].t())
        cur = x1 + p_f + p["b2"]
        keep.append((p_o, p_f, ln1, ln2))
    want = [x0] + [v for p in par for v in p.values()] + [v for k in keep for v in k[2:]]
    got = torch.autograd.grad(cur, want, dy.double().reshape(T, h))
    grads = torch.zeros(total, dtype=torch.float64, device=DEV)
    n = len(shapes)
    for l in range(L):
        for i in range(n):
            v = got[1 + l * n + i].reshape(-1)
            grads[int(offs[l, i]):int(offs[l, i]) + v.numel()] = v
    d_ln = torch.stack(got[1 + L * n:]).reshape(L, 2, T, h)
    out = (s.micro_batch, s.seq_len, h)
    return {"y": cur.detach().reshape(out), "dx": got[0].reshape(out), "grads": grads,
            "fwd_partials": torch.stack([torch.stack([k[0], k[1]]) for k in keep]).detach(), "bwd_partials": d_ln}
