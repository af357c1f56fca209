"""The forward's loop, in which V runs one tile of 64 keys behind K: one, two and three tiles, an odd and an even number
of them where they are requested two at a time (256-row workgroups), ends inside a tile, causal waves that stop at
different tiles, rows of which the reference has to move in the first and in the second half of a tile.  First and last
head against 64-bit products, with and without dropout.
"""
import math

import pytest
import torch

from paper_2502_12784_amd import spark_dropout_mask, spark_mha_strided_fwd

pytestmark = pytest.mark.gpu

# heads, Nq, Nk, d, dtype, causal, dropout rate
CASES = [(300, 130, nk, d, dtype, False, p)
         for nk, d, dtype, p in [(1, 64, torch.float16, 0.0), (33, 128, torch.bfloat16, 0.0), (64, 96, torch.float16, 0.1),
                                 (65, 64, torch.bfloat16, 0.1), (127, 128, torch.float16, 0.0), (128, 64, torch.float16, 0.0),
                                 (129, 80, torch.bfloat16, 0.0), (192, 128, torch.float16, 0.1)]]
CASES += [(44, 700, 2048, 128, torch.bfloat16, False, 0.0), (44, 700, 2049, 128, torch.float16, False, 0.0),
          (44, 700, 2112, 96, torch.float16, False, 0.1)]  # 32, 33 and 33 tiles, two at a time
CASES += [(300, n, n, d, dtype, True, p)
          for n, d, dtype, p in [(1, 64, torch.float16, 0.0), (32, 128, torch.float16, 0.0), (65, 64, torch.float16, 0.1),
                                 (129, 128, torch.bfloat16, 0.1), (191, 64, torch.bfloat16, 0.0), (320, 96, torch.float16, 0.0)]]


@pytest.mark.parametrize("case", CASES)
def test_forward_rounds(case):
    bh, nq, nk, d, dtype, causal, p = case
    print(f"\n[rounds] {case}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6400 + nk)
    q, k, v = (torch.randn(1, bh, n, d, generator=g, device="cuda") for n in (nq, nk, nk))
    k *= 1.0 + 3.0 * (torch.arange(nk, device="cuda") % 64 >= 40)[:, None]  # the maximum grows late in a tile
    q, k, v = (t.to(dtype) for t in (q, k, v))
    scale = 1.0 / math.sqrt(d)
    drop = dict(p_drop=p, seed=11, offset=3) if p else {}
    O, LSE = spark_mha_strided_fwd(q, k, v, scale, causal, **drop)
    rescale = 256.0 / (256 - int(p * 256 + 0.5))
    keep = spark_dropout_mask(1, bh, nq, nk, p, 11, 3, "cuda")[0] if p else None
    u = 2.0 ** (-8 if dtype == torch.bfloat16 else -11)  # unit roundoff of P and of O
    for h in (0, bh - 1):
        x = (q[0, h].double() @ k[0, h].double().T) * scale
        if causal:
            x = x.masked_fill(torch.ones_like(x, dtype=torch.bool).triu(1), -math.inf)
        lse = torch.logsumexp(x, 1)
        P = torch.exp(x - lse[:, None])
        if p:
            P = P * keep[h].double() * rescale
        o = P @ v[0, h].double()
        # |sum of P V| changes by at most u max|V| (rescaled) with P rounded, and the result is rounded once
        tol = u * (float(o.abs().max()) + rescale * float(v[0, h].abs().max())) + 1e-5
        assert float((O[0, h].double() - o).abs().max()) <= tol
        assert float((LSE[0, h].double() - lse).abs().max()) <= 1e-4
