"""Calls that a program using this library makes, for timing and comparison.

A case is a plain dict.  ``kind`` names the entry point:

  softmax  fem_softmax_fwd       the causal read, bf16 (matrix cores) or fp32
  variant  fem_softmax_fwd_ex    encoder read, value width d_qk / 2, bf16 output
  gated    fem_softmax_gated_fwd the two-level gated read
  train    fem_softmax_fwd_train + fem_softmax_bwd: a training step's layer
  decode   fem_softmax_decode(_noalloc): one new token against a KV cache
  linear   fem_linear_fwd        the linear-prior scan
  gla      fem_gla_fwd           the decay-gated scan

Distributions are those of ``paper_2602_07160_amd/inputs.py`` (q, k, v ~
N(0, 1), beta log-uniform, gates and decays as described there), drawn on the
GPU.  Output buffers and workspaces are kept between calls, as a serving or
training loop keeps them.
"""

import math

import torch

from paper_2602_07160_amd import binding

DEV = "cuda"


def listed():
    return [
        # The smallest call: one short head in fp32 (a unit-test or debugging
        # size; the repository's first workload).
        dict(name="f32_tiny", kind="softmax", dtype="f32", B=1, H=1, T=128, d=32,
             beta_lo=0.25, beta_hi=4.0),
        # fp32 layer of the paper's GPT-2 timing table (12 heads of 64,
        # context 1024; batch 4).
        dict(name="f32_gpt2", kind="softmax", dtype="f32", B=4, H=12, T=1024, d=64,
             beta_lo=0.25, beta_hi=4.0),
        # An ordinary bf16 layer (the repository's second workload): fewer
        # query blocks than compute units.
        dict(name="read_mid", kind="softmax", dtype="bf16", B=4, H=8, T=1024, d=64,
             beta_lo=0.1, beta_hi=8.0),
        # The headline workload: language-model prefill at context 4096.
        dict(name="read_large", kind="softmax", dtype="bf16", B=8, H=16, T=4096, d=128,
             beta_lo=0.1, beta_hi=8.0),
        # Encoder use (no mask) on a ragged length, half-width values, bf16
        # output for a bf16 model.
        dict(name="encoder_ragged", kind="variant", B=3, H=6, T=1571, d=128, dv=64,
             causal=False, out_bf16=True, beta_lo=0.1, beta_hi=8.0),
        # The full two-level read of the paper's models, language-model layer
        # (16 heads of 128, context 2048).
        dict(name="gated_lm", kind="gated", B=2, H=16, T=2048, d=128, gate=True,
             beta_lo=0.1, beta_hi=8.0),
        # Training layer of the paper's speed table: hidden 512 in 4 heads,
        # context 2048, batch 4.
        dict(name="train_paper", kind="train", B=4, H=4, T=2048, d=128,
             beta_lo=0.1, beta_hi=8.0),
        # The largest call: a training layer at the headline shape.
        dict(name="train_large", kind="train", B=8, H=16, T=4096, d=128,
             beta_lo=0.1, beta_hi=8.0),
        # A single stream's decoding step: short odd cache, few heads, the
        # entry point of loops that cannot allocate.
        dict(name="decode_one", kind="decode", B=1, H=8, L=701, d=64, dv=64, lens=False,
             noalloc=True, beta_lo=0.1, beta_hi=8.0),
        # A serving batch's decoding step: sequences of different lengths.
        dict(name="decode_batch", kind="decode", B=8, H=16, L=4096, d=128, dv=128, lens=True,
             noalloc=False, beta_lo=0.1, beta_hi=8.0),
        # The linear-prior scan at the repository's fifth workload.
        dict(name="linear_long", kind="linear", B=4, H=16, T=8192, chunk=64,
             beta_lo=0.1, beta_hi=4.0),
        # The decay-gated scan, fewer heads and a ragged length.
        dict(name="gla_ragged", kind="gla", B=2, H=12, T=5003, beta_lo=0.1, beta_hi=4.0),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more call of the ranges above, odd sizes among them."""
    kind = rng.choice(["f32", "read", "read", "variant", "gated", "train", "decode", "decode",
                       "linear", "gla"])
    B, H = rng.randint(1, 8), rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
    d = rng.choice([32, 64, 128])
    wide = dict(beta_lo=0.1, beta_hi=8.0)

    def length(lo, hi, per_pair, cap):
        """T (odd ones among them) whose causal pairs keep B H pairs per_pair under cap."""
        top = max(lo, min(hi, int(math.sqrt(2.0 * cap / (B * H * per_pair)))))
        return _logint(rng, lo, top)

    if kind == "f32":
        d = rng.choice([32, 64, 128, rng.randint(1, 256)])
        return dict(kind="softmax", dtype="f32", B=B, H=H, T=length(16, 2048, d, 1.6e9), d=d,
                    beta_lo=0.25, beta_hi=4.0)
    if kind == "read":
        return dict(kind="softmax", dtype="bf16", B=B, H=H, T=length(64, 16384, d, 1.37e11), d=d,
                    **wide)
    if kind == "variant":
        causal = rng.random() < 0.4
        dv = d // 2 if d > 32 and rng.random() < 0.5 else d
        return dict(kind="variant", B=B, H=H, T=length(64, 4096, 2 * d, 1.37e11), d=d, dv=dv,
                    causal=causal, out_bf16=rng.random() < 0.5, **wide)
    if kind == "gated":
        return dict(kind="gated", B=B, H=H, T=length(64, 4096, d, 6.9e10), d=d,
                    gate=rng.random() < 0.7, **wide)
    if kind == "train":
        return dict(kind="train", B=B, H=H, T=length(64, 4096, d, 6.9e10), d=d, **wide)
    if kind == "decode":
        dv = d // 2 if d > 32 and rng.random() < 0.3 else d
        return dict(kind="decode", B=_logint(rng, 1, 64), H=H, L=_logint(rng, 32, 8192), d=d, dv=dv,
                    lens=rng.random() < 0.7, noalloc=rng.random() < 0.3, **wide)
    if kind == "linear":
        return dict(kind="linear", B=B, H=H, T=_logint(rng, 64, 8192),
                    chunk=rng.choice([16, 32, 64, 64, 64, 128]), beta_lo=0.1, beta_hi=4.0)
    return dict(kind="gla", B=B, H=H, T=_logint(rng, 64, 8192), beta_lo=0.1, beta_hi=4.0)


# ---- inputs ------------------------------------------------------------------

def _inputs(case, seed):
    """The call's tensors, from the seed alone."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))

    def normal(*shape, std=1.0):
        return torch.randn(shape, device=DEV, dtype=torch.float32, generator=g) * std

    B, H = case["B"], case["H"]
    kind = case["kind"]
    d = case.get("d", 64)
    dv = case.get("dv", d)
    n = case["L"] if kind == "decode" else case["T"]
    dt = torch.float32 if case.get("dtype") == "f32" else torch.bfloat16
    x = {}
    x["q"] = (normal(B, H, d) if kind == "decode" else normal(B, H, n, d)).to(dt)
    x["k"] = normal(B, H, n, d).to(dt)
    x["v"] = normal(B, H, n, dv).to(dt)
    u = torch.rand((H, dv), device=DEV, dtype=torch.float64, generator=g)
    lo, hi = math.log(case["beta_lo"]), math.log(case["beta_hi"])
    x["beta"] = torch.exp(lo + (hi - lo) * u).float()
    if kind == "gated":
        x["lam"] = torch.sigmoid(normal(B, H, n, d, std=2.0))
        gate = torch.nn.functional.softplus(normal(B, H, n, d))
        x["gate"] = gate / gate.square().mean(-1, keepdim=True).sqrt() if case["gate"] else None
    elif kind == "train":
        x["dout"] = normal(B, H, n, d)
    elif kind == "decode":
        # sequences between a quarter full and full
        x["lens"] = (torch.randint((n + 3) // 4, n + 1, (B,), device=DEV, dtype=torch.int32,
                                   generator=g) if case["lens"] else None)
    elif kind == "gla":
        x["g"] = torch.nn.functional.logsigmoid(normal(B, H, n, d)) / 16.0
    return x


def _f32(*shape):
    return torch.empty(shape, device=DEV, dtype=torch.float32)


def _bytes(entry, *sizes):
    n = binding.workspace_bytes(entry, *sizes)
    return torch.empty(n, device=DEV, dtype=torch.uint8) if n else None


def prepare(case, seed):
    x = _inputs(case, seed)
    kind, B, H = case["kind"], case["B"], case["H"]
    st = dict(case=case, **x)
    if kind == "decode":
        L, d, dv = case["L"], case["d"], case["dv"]
        st["out"] = _f32(B, H, dv)
        st["ws"] = None if case["noalloc"] else _bytes("decode", B, H, L, d, dv)
        return st
    T = case["T"]
    if kind in ("linear", "gla"):
        st["out"] = _f32(B, H, T, 64)
        st["ws"] = _bytes(kind, B, H, T, 64, 64, case.get("chunk", 64))
        return st
    d, dv = case["d"], case.get("dv", case["d"])
    st["out"] = torch.empty((B, H, T, dv), device=DEV,
                            dtype=torch.bfloat16 if case.get("out_bf16") else torch.float32)
    if kind == "train":
        st["lse"] = _f32(B, H, T)
        st["ws"] = _bytes("bwd", B, H, T, d)
    return st


def run(state):
    s, case = state, state["case"]
    kind = case["kind"]
    if kind == "softmax":
        return binding.fem_softmax_fwd(s["q"], s["k"], s["v"], s["beta"], out=s["out"])
    if kind == "variant":
        return binding.fem_softmax_fwd_ex(s["q"], s["k"], s["v"], s["beta"], out=s["out"],
                                          causal=case["causal"], out_dtype=s["out"].dtype)
    if kind == "gated":
        return binding.fem_softmax_gated_fwd(s["q"], s["k"], s["v"], s["beta"], s["lam"],
                                             s["gate"], out=s["out"])
    if kind == "train":
        out, lse = binding.fem_softmax_fwd_train(s["q"], s["k"], s["v"], s["beta"], out=s["out"],
                                                 lse=s["lse"])
        return (out, lse) + tuple(binding.fem_softmax_bwd(s["q"], s["k"], s["v"], s["beta"], out,
                                                          lse, s["dout"], ws=s["ws"]))
    if kind == "decode":
        if case["noalloc"]:
            return binding.fem_softmax_decode_noalloc(s["q"], s["k"], s["v"], s["beta"],
                                                      lens=s["lens"], out=s["out"])
        return binding.fem_softmax_decode(s["q"], s["k"], s["v"], s["beta"], lens=s["lens"],
                                          out=s["out"], ws=s["ws"])
    if kind == "linear":
        return binding.fem_linear_fwd(s["q"], s["k"], s["v"], s["beta"], out=s["out"],
                                      chunk=case["chunk"], ws=s["ws"])
    return binding.fem_gla_fwd(s["q"], s["k"], s["v"], s["g"], s["beta"], out=s["out"], ws=s["ws"])


def work(case):
    """Bytes and operations of the call: inputs read once, outputs written
    once; multiply-adds counted as two, exponentials not at all."""
    kind, B, H = case["kind"], case["B"], case["H"]
    if kind == "decode":
        # (lengths between a quarter and all of the cache: 5/8 on average)
        keys = B * H * case["L"] * (0.625 if case["lens"] else 1.0)
        w = case["d"] + case["dv"]
        return {"bytes": keys * w * 2 + B * H * (2 * case["d"] + 4 * case["dv"]),
                "flops": keys * w * 2}
    T = case["T"]
    tok = B * H * T
    if kind in ("linear", "gla"):
        # the state form: phi(q) S and the update phi(k) E per token
        return {"bytes": tok * (640 + (256 if kind == "gla" else 0)), "flops": tok * 4 * 64 * 64}
    d, dv = case["d"], case.get("dv", case["d"])
    pairs = B * H * (T * (T + 1) // 2 if case.get("causal", True) else T * T)
    es = 4 if case.get("dtype") == "f32" else 2
    io = tok * ((2 * d + dv) * es + dv * (2 if case.get("out_bf16") else 4))
    fl = pairs * 2 * (d + dv)
    if kind == "gated":  # the second value product; lam and gate
        return {"bytes": io + tok * 4 * d * (2 if case["gate"] else 1), "flops": fl + pairs * 2 * d}
    if kind == "train":  # Q K^T again, the posterior weights, dQ, dK and dV; dout, lse, gradients
        return {"bytes": io + tok * (4 + 16 * d), "flops": fl + pairs * 10 * d}
    return {"bytes": io, "flops": fl}


def tolerance(case):
    """About four times the differences from ``exact`` that these ranges show
    (relative 2-norm; largest over the result's root mean square)."""
    kind = case["kind"]
    if kind == "softmax" and case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 6e-5}  # seen 1.2e-6, 1.5e-5
    if kind == "decode":
        return {"rel": 3e-6, "max": 2e-5}  # seen 7e-7, 5e-6: fp32 arithmetic on bf16 inputs
    if kind == "train":
        # seen 2.1e-3, 1e-1 (dQ and dK, whose dS enters a product in bf16; the
        # largest difference sits in the first rows, far above the others)
        return {"rel": 8e-3, "max": 4e-1}
    if kind == "gated":
        return {"rel": 2e-3, "max": 7e-2}  # seen 5.2e-4, 1.7e-2
    if kind == "gla":
        return {"rel": 2.6e-3, "max": 3.6e-2}  # seen 6.6e-4, 8.8e-3
    if case.get("out_bf16"):
        return {"rel": 7e-3, "max": 3.5e-2}  # seen 1.7e-3, 8.5e-3: the output's rounding
    return {"rel": 2e-3, "max": 3e-2}  # seen 4.8e-4 (short contexts), 7.4e-3


# ---- the same read in 64 bits --------------------------------------------------

def _heads(case):
    """Heads per step, so that a [T, T] float64 matrix of them stays near 1 GB."""
    T = case["T"]
    return max(1, min(case["B"] * case["H"], int(1.2e8 / (T * T))))


def _prior(q, k, causal):
    """p [n, T, T] and the log-normaliser [n, T] of float64 q, k [n, T, d]."""
    s = torch.matmul(q, k.transpose(1, 2)) / math.sqrt(q.shape[-1])
    if causal:
        T = s.shape[-1]
        s.masked_fill_(torch.ones((T, T), dtype=torch.bool, device=s.device).triu_(1), -math.inf)
    lse = torch.logsumexp(s, -1)
    return s.sub_(lse.unsqueeze(-1)).exp_(), lse


def _tilt(v, beta):
    """E = exp(beta v - c), c of float64 v [n, T, dv], beta [n, dv]."""
    x = v * beta.unsqueeze(1)
    c = x.amax(1, keepdim=True)
    return torch.exp(x - c), c


def _exact_softmax(case, x):
    B, H, T = case["B"], case["H"], case["T"]
    kind = case["kind"]
    d, dv = case["d"], case.get("dv", case["d"])
    N = B * H
    q, k, v = (x[n].reshape(N, T, -1) for n in ("q", "k", "v"))
    beta = x["beta"].double().repeat(B, 1)
    f64 = dict(device=q.device, dtype=torch.float64)
    out = torch.empty((N, T, dv), **f64)
    train = kind == "train"
    if train:
        lse_o, dbeta = torch.empty((N, T), **f64), torch.empty((N, d), **f64)
        dq, dk, dvv = (torch.empty((N, T, d), **f64) for _ in range(3))
    step = _heads(case)
    for i in range(0, N, step):
        sl = slice(i, min(N, i + step))
        qd, kd, vd, b = q[sl].double(), k[sl].double(), v[sl].double(), beta[sl]
        p, lse = _prior(qd, kd, case.get("causal", True))
        e, c = _tilt(vd, b)
        b = b.unsqueeze(1)
        F = (torch.log(torch.matmul(p, e)) + c) / b
        if kind == "gated":
            mu = torch.matmul(p, vd)
            lam = x["lam"].reshape(N, T, d)[sl].double()
            F = mu + lam * (F - mu)
            if x["gate"] is not None:
                F = F * x["gate"].reshape(N, T, d)[sl].double()
        out[sl] = F
        if train:
            G = x["dout"].reshape(N, T, d)[sl].double()
            W, U = G / b, torch.exp(c - b * F)
            ds = torch.matmul(W * U, e.transpose(1, 2)).sub_(W.sum(-1, keepdim=True)).mul_(p)
            ds /= math.sqrt(d)
            lse_o[sl] = lse
            dq[sl] = torch.matmul(ds, kd)
            dk[sl] = torch.matmul(ds.transpose(1, 2), qd)
            dvv[sl] = e * torch.matmul(p.transpose(1, 2), G * U)
            dbeta[sl] = (G * (U * torch.matmul(p, e * vd) - F) / b).sum(1)
    out = out.reshape(B, H, T, dv)
    if not train:
        return out
    return (out, lse_o.reshape(B, H, T), dq.reshape(B, H, T, d), dk.reshape(B, H, T, d),
            dvv.reshape(B, H, T, d), dbeta.reshape(B, H, d).sum(0))


def _exact_decode(case, x):
    B, H, L, d, dv = case["B"], case["H"], case["L"], case["d"], case["dv"]
    out = torch.empty((B, H, dv), device=DEV, dtype=torch.float64)
    lens = [L] * B if x["lens"] is None else x["lens"].tolist()
    b = x["beta"].double()
    for i in range(B):
        n = lens[i]
        q, k, v = x["q"][i].double(), x["k"][i, :, :n].double(), x["v"][i, :, :n].double()
        p = torch.softmax((k * q.unsqueeze(1)).sum(-1) / math.sqrt(d), -1)
        e, c = _tilt(v, b)
        out[i] = (torch.log((p.unsqueeze(-1) * e).sum(1)) + c.squeeze(1)) / b
    return out


def _rope(x):
    """Rotate the pairs (2m, 2m+1) of float64 x [.., T, d] by t 10000^(-2m/d)."""
    T, d = x.shape[-2:]
    t = torch.arange(T, device=x.device, dtype=torch.float64)
    f = 10000.0 ** (-torch.arange(0, d, 2, device=x.device, dtype=torch.float64) / d)
    a = t[:, None] * f
    x0, x1 = x[..., 0::2], x[..., 1::2]
    return torch.stack((x0 * a.cos() - x1 * a.sin(), x0 * a.sin() + x1 * a.cos()), -1).flatten(-2)


def _exact_scan(case, x):
    """Both scans with the decay kept per key channel, 64 tokens at a time."""
    B, H, T = case["B"], case["H"], case["T"]
    q, k, v = x["q"].double(), x["k"].double(), x["v"].double()
    if case["kind"] == "gla":
        q, k = torch.relu(_rope(q)) + 1e-6, torch.relu(_rope(k)) + 1e-6
        g = x["g"].double()
    else:
        q, k = torch.nn.functional.elu(q) + 1.0, torch.nn.functional.elu(k) + 1.0
        g = torch.zeros_like(q)
    beta = x["beta"].double()[None, :, None, :]
    xv = v * beta
    c = xv.amax(2, keepdim=True)
    # the values' last column is the constant that sums the normaliser
    e = torch.cat((torch.exp(xv - c), torch.ones((B, H, T, 1), device=v.device,
                                                 dtype=torch.float64)), -1)
    S = torch.zeros((B, H, 64, e.shape[-1]), device=v.device, dtype=torch.float64)
    out = torch.empty_like(v)
    for t0 in range(0, T, 64):
        sl = slice(t0, min(T, t0 + 64))
        run_g = torch.cumsum(g[:, :, sl], 2)
        mid, last = run_g[:, :, run_g.shape[2] // 2, None], run_g[:, :, -1, None]
        a = torch.matmul(q[:, :, sl] * torch.exp(run_g - mid),
                         (k[:, :, sl] * torch.exp(mid - run_g)).transpose(2, 3)).tril_()
        y = torch.matmul(a, e[:, :, sl]) + torch.matmul(q[:, :, sl] * torch.exp(run_g), S)
        out[:, :, sl] = torch.log(y[..., :-1] / y[..., -1:])
        S = S * torch.exp(last).transpose(2, 3) + torch.matmul(
            (k[:, :, sl] * torch.exp(last - run_g)).transpose(2, 3), e[:, :, sl])
    return (out + c) / beta


def exact(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "decode":
        return _exact_decode(case, x)
    if case["kind"] in ("linear", "gla"):
        return _exact_scan(case, x)
    return _exact_softmax(case, x)
