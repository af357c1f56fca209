"""Forward grids on both sides of the rule that takes 256-row workgroups at d > 64: one full round of them, just
beyond one, almost two, rows that end inside a tile.  First and last head against 64-bit products.
"""
import math

import pytest
import torch

from paper_2502_12784_amd import spark_mha_strided_fwd

pytestmark = pytest.mark.gpu

# heads, Nq, Nk, d, dtype, causal: workgroups of 256 / of 128 rows
CASES = [
    (32, 1987, 2050, 128, torch.bfloat16, False),   # 256 / 512: wide
    (43, 700, 2048, 96, torch.float16, False),      # 129 / 258: wide, the smallest
    (86, 300, 2111, 128, torch.float16, False),     # 172 / 258: wide, last tile mostly empty
    (256, 100, 2048, 128, torch.bfloat16, False),   # 256 / 256: narrow
    (257, 256, 2048, 128, torch.bfloat16, False),   # 257 / 514: narrow
    (112, 1000, 2100, 128, torch.bfloat16, False),  # 448 / 896: wide
    (64, 2048, 2048, 128, torch.bfloat16, True),    # 256 / 512, paired: wide
    (30, 2303, 2303, 104, torch.float16, True),     # 150 / 270, a middle tile alone: wide
]


@pytest.mark.parametrize("case", CASES)
def test_wide_forward(case):
    bh, nq, nk, d, dtype, causal = case
    print(f"\n[wide] {case}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(8100 + nq)
    q, k, v = (torch.randn(1, bh, n, d, generator=g, device="cuda").to(dtype) for n in (nq, nk, nk))
    scale = 1.0 / math.sqrt(d)
    O, LSE = spark_mha_strided_fwd(q, k, v, scale, causal)
    u = 2.0 ** (-8 if dtype == torch.bfloat16 else -11)  # unit roundoff of P and of O
    for h in (0, bh - 1):
        x = (q[0, h].double() @ k[0, h].double().T) * scale
        if causal:
            x = x.masked_fill(torch.ones_like(x, dtype=torch.bool).triu(1), -math.inf)
        lse = torch.logsumexp(x, 1)
        o = torch.exp(x - lse[:, None]) @ v[0, h].double()
        # |sum of P V| changes by at most u max|V| with P rounded, and the result is rounded once
        tol = u * (float(o.abs().max()) + float(v[0, h].abs().max())) + 1e-5
        assert float((O[0, h].double() - o).abs().max()) <= tol
        assert float((LSE[0, h].double() - lse).abs().max()) <= 1e-4
