"""The workloads that performance work on the fused attention is judged on.

A case is one pass of a user's program through the package's entry points: a training step of one
attention layer (forward, then backward; ``pass`` = "step") or a forward alone (``pass`` = "fwd").
The listed cases are the benchmark configurations, points of the grid of hidden size 2048 that
``bench.py --sweep`` runs, and the decoder-sized, ragged, strided and single-query problems that the
tests cover; ``draw`` spreads the same kinds over their ranges.

Inputs are normal random numbers (for some cases with logits of standard deviation 3), as everywhere
in this repository.  Outputs and workspace are allocated by the calls, as in a plain training loop.
"""
import math

import torch

from paper_2502_12784_amd import (spark_mha_bwd, spark_mha_cross_bwd, spark_mha_cross_fwd,
                                  spark_mha_dropout_bwd, spark_mha_dropout_fwd, spark_mha_fwd,
                                  spark_mha_strided_bwd, spark_mha_strided_fwd)

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


def _case(name, what, B, H, Nq, d, dtype, causal, Nk=None, p=0.0, sigma=1.0, layout="bhnd"):
    c = {"pass": what, "B": B, "H": H, "Nq": Nq, "Nk": Nq if Nk is None else Nk, "d": d, "dtype": dtype,
         "causal": causal, "p": p, "sigma": sigma, "layout": layout}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call in use: one short sequence, two heads.  Host path and launches count.
        _case("tiny-step", "step", 1, 2, 128, 64, "f16", False),
        # One new token of a decoder attending to a long memory: one query row per head.
        _case("one-query-fwd", "fwd", 8, 16, 1, 128, "bf16", False, Nk=2048),
        # An encoder layer of base size on short sequences (12 heads of 64, N = 512).
        _case("encoder-512-step", "step", 8, 12, 512, 64, "f16", False),
        # A causal decoder layer of base size (16 heads of 64, N = 1024).
        _case("causal-1024-step", "step", 8, 16, 1024, 64, "f16", True),
        # The benchmark's headline: wide heads, causal, N = 4096, bf16.
        _case("causal-4096-wide-step", "step", 4, 16, 4096, 128, "bf16", True),
        # A long sequence with peaked attention (logits of standard deviation 3).
        _case("long-8192-step", "step", 2, 16, 8192, 64, "f16", False, sigma=math.sqrt(3.0)),
        # Short end of the hidden-2048 grid with the dropout rate of its measurements: many short heads.
        _case("causal-512-dropout-step", "step", 32, 16, 512, 128, "f16", True, p=0.1),
        # Middle of that grid: narrow heads, no mask, dropout.
        _case("dropout-2048-step", "step", 8, 32, 2048, 64, "f16", False, p=0.1),
        # Long end of that grid, the largest case: one sequence of 16384 tokens.
        _case("causal-16384-step", "step", 1, 16, 16384, 128, "f16", True),
        # Inference over a prompt: forward alone.
        _case("prefill-2048-fwd", "fwd", 4, 16, 2048, 128, "bf16", True),
        # A decoder's second attention layer: 1024 target positions over 4096 source positions.
        _case("cross-1024x4096-step", "step", 4, 16, 1024, 128, "bf16", False, Nk=4096),
        # Slices of a packed [B, N, 3, H, d] projection, ragged length, a head size between the tiles.
        _case("packed-ragged-step", "step", 3, 12, 1333, 80, "bf16", True, layout="packed"),
    ]


def _cost(c):
    """Executed multiply-adds, roughly: rows are padded to 64 or 128 columns, dropout adds a half."""
    tiles = 64 if c["d"] <= 64 else 128
    f = 4.0 * c["B"] * c["H"] * c["Nq"] * c["Nk"] * tiles * (3.5 if c["pass"] == "step" else 1.0)
    return f * (0.5 if c["causal"] else 1.0) * (1.5 if c["p"] else 1.0)


def draw(rng):
    def size(lo, hi):  # spread over the logarithm, odd values among them
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return n if rng.random() < 0.5 else max(lo, min(hi, (n + 63) // 64 * 64))

    while True:
        kind = rng.choice(["self", "self", "self", "fwd", "cross", "few", "packed"])
        d = rng.choice([64, 128, 64, 128, 8 * rng.randint(4, 16)])
        dtype = rng.choice(["f16", "bf16"])
        causal = rng.random() < 0.5
        p = 0.1 if rng.random() < 0.3 else 0.0
        sigma = math.sqrt(3.0) if rng.random() < 0.2 else 1.0
        N = size(128, 16384)
        # heads: from two up to about 16384 tokens of hidden size 2048 in all
        heads = max(2, int(math.exp(rng.uniform(math.log(2), math.log(max(2.0, 2.0 * 16384 * 2048 / (N * d)))))))
        H = rng.choice([h for h in (1, 2, 3, 4, 8, 12, 16, 32) if h <= heads])
        B = max(1, heads // H)
        if kind == "cross":
            c = _case(None, "step", B, H, size(64, 4096), d, dtype, False, Nk=N, p=p, sigma=sigma)
        elif kind == "few":
            c = _case(None, "fwd", B, H, rng.choice([1, 1, 2, 4, 7, 16, 40]), d, dtype, False, Nk=N, sigma=sigma)
        elif kind == "packed":
            c = _case(None, "step", B, H, N, d, dtype, causal, p=p, sigma=sigma, layout="packed")
        else:
            c = _case(None, "fwd" if kind == "fwd" else "step", B, H, N, d, dtype, causal, p=p, sigma=sigma)
        if _cost(c) <= 3.0e12:  # the largest listed case costs 3.8e12
            return c


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt = DTYPES[case["dtype"]]
    B, H, Nq, Nk, d = (case[k] for k in ("B", "H", "Nq", "Nk", "d"))

    def normal(*shape, sigma=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * sigma).to(dt)

    s = {"case": case, "scale": 1.0 / math.sqrt(d), "dropout": (case["p"], int(seed) * 1000003 + 17, 0)}
    if case["layout"] == "packed":
        qkv = normal(B, Nq, 3, H, d)
        qkv[:, :, :2] *= case["sigma"]
        s["Q"], s["K"], s["V"] = (qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3))
        s["dO"] = normal(B, Nq, H, d).permute(0, 2, 1, 3)
    else:
        s["Q"] = normal(B, H, Nq, d, sigma=case["sigma"])
        s["K"] = normal(B, H, Nk, d, sigma=case["sigma"])
        s["V"] = normal(B, H, Nk, d)
        s["dO"] = normal(B, H, Nq, d)
    return s


def run(s):
    c, Q, K, V, dO, scale, causal = s["case"], s["Q"], s["K"], s["V"], s["dO"], s["scale"], s["case"]["causal"]
    step = c["pass"] == "step"
    if c["layout"] == "packed":
        O, LSE = spark_mha_strided_fwd(Q, K, V, scale, causal, *s["dropout"])
        grads = spark_mha_strided_bwd(Q, K, V, O, LSE, dO, scale, causal, *s["dropout"]) if step else ()
    elif c["p"]:
        O, LSE = spark_mha_dropout_fwd(Q, K, V, scale, causal, *s["dropout"])
        grads = spark_mha_dropout_bwd(Q, K, V, O, LSE, dO, scale, causal, *s["dropout"]) if step else ()
    elif c["Nq"] != c["Nk"]:
        O, LSE = spark_mha_cross_fwd(Q, K, V, scale)
        grads = spark_mha_cross_bwd(Q, K, V, O, LSE, dO, scale) if step else ()
    else:
        O, LSE = spark_mha_fwd(Q, K, V, scale, causal)
        grads = spark_mha_bwd(Q, K, V, O, LSE, dO, scale, causal) if step else ()
    return (O, LSE) + tuple(grads)


def work(case):
    B, H, Nq, Nk, d = (case[k] for k in ("B", "H", "Nq", "Nk", "d"))
    pairs = float(Nq) * (Nq + 1) / 2 if case["causal"] else float(Nq) * Nk
    flops = 4.0 * B * H * pairs * d  # S = Q K^T and P V
    nbytes = B * H * (2.0 * d * (2 * Nq + 2 * Nk) + 4 * Nq)  # Q, O, K, V, LSE
    if case["pass"] == "step":
        # backward: the scores again, dP, dV, dK, dQ; dO read and dQ, dK, dV written besides
        flops *= 3.5
        nbytes += B * H * 2.0 * d * (2 * Nq + 2 * Nk)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # About four times the largest difference from the same problem in 64 bits (see _reference_error):
    # outputs are rounded once to the 16-bit type, P and dS once as operands, O once before the backward.
    # Measured: at most 2.5e-3 in bf16 and 3.8e-4 in fp16 over the listed cases.
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1.5e-3}


def _reference_error(case, seed=1):
    """Largest relative error (2-norm) over the outputs of one pass against the first and the last head
    evaluated in 64 bits; the basis of ``tolerance``.  Without dropout."""
    s = prepare(case, seed)
    outs = run(s)
    worst = {}
    for b, h in {(0, 0), (case["B"] - 1, case["H"] - 1)}:
        q, k, v, do = (s[n][b, h].double() for n in ("Q", "K", "V", "dO"))
        x = (q @ k.T) * s["scale"]
        if case["causal"]:
            x = x.masked_fill(torch.ones_like(x, dtype=torch.bool).triu(1), -math.inf)
        lse = torch.logsumexp(x, 1)
        P = torch.exp(x - lse[:, None])
        o = P @ v
        ref = [o, lse]
        if case["pass"] == "step":
            dS = P * (do @ v.T - (do * o).sum(1, keepdim=True)) * s["scale"]
            ref += [dS @ k, dS.T @ q, P.T @ do]
        for n, got, want in zip(("O", "LSE", "dQ", "dK", "dV"), outs, ref):
            e = float((got[b, h].double() - want).norm() / want.norm())
            worst[n] = max(worst.get(n, 0.0), e)
    return worst
