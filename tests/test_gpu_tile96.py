"""The kernels of 96 columns (d = 72 to 96) beside those of 128: the same rows with columns of zeros appended up to
d = 104 run in the wider kernels, where those columns add zeros to the same sums in the same order.  So every output has to
be equal bit for bit, and the gradients of the appended columns are zero.  Grids of each route: the forward with
workgroups of 128 and of 256 rows, the backward as one grid and as two, with ragged last tiles and strided rows.
"""
import math

import pytest
import torch

from paper_2502_12784_amd import load_library, spark_mha_strided_bwd, spark_mha_strided_fwd

pytestmark = pytest.mark.gpu

# heads, Nq, Nk, d, dtype, causal, dropout rate, backward grids
CASES = [
    (40, 1025, 1025, 96, torch.bfloat16, True, 0.0, 2),
    (36, 1333, 1333, 80, torch.float16, False, 0.0, 2),
    (44, 700, 2079, 72, torch.bfloat16, False, 0.0, 2),   # 256-row workgroups
    (200, 511, 511, 88, torch.float16, True, 0.1, 2),      # dQ with 32-key tiles
    (64, 513, 770, 96, torch.bfloat16, False, 0.2, 2),
    (10, 1100, 1000, 80, torch.bfloat16, False, 0.0, 1),
    (12, 1030, 1030, 72, torch.float16, True, 0.1, 1),
    # causal 256-row workgroups, in pairs: nine tiles of them a head, the middle one alone; 36 and 35 tiles of 64 keys
    (30, 2303, 2303, 80, torch.float16, True, 0.0, 2),
    (30, 2303, 2303, 96, torch.bfloat16, True, 0.1, 2),
    (30, 2240, 2240, 96, torch.float16, True, 0.1, 2),
    (30, 2240, 2240, 72, torch.bfloat16, True, 0.0, 2),
]


def run(q, k, v, do, causal, p):
    drop = dict(p_drop=p, seed=77, offset=1) if p else {}
    scale = 1.0 / math.sqrt(96)
    o, lse = spark_mha_strided_fwd(q, k, v, scale, causal, **drop)
    return (o, lse) + tuple(spark_mha_strided_bwd(q, k, v, o, lse, do, scale, causal, **drop))


@pytest.mark.parametrize("case", CASES)
def test_same_bits_as_the_wider_kernels(case):
    bh, nq, nk, d, dtype, causal, p, grids = case
    print(f"\n[tile96] {case}", flush=True)
    for dim in (d, 104):
        assert load_library().spark_mha_bwd_grids(1, bh, nq, nk, dim, causal, p, int(dtype == torch.bfloat16)) == grids
    g = torch.Generator(device="cuda").manual_seed(9600 + nq)
    wide = [torch.zeros(1, bh, n, 104, dtype=dtype, device="cuda") for n in (nq, nk, nk, nq)]
    for t in wide:
        t[..., :d] = torch.randn(1, bh, t.shape[2], d, generator=g, device="cuda")
    exp = run(*wide, causal, p)
    for rows in ([t[..., :d] for t in wide], [t[..., :d].contiguous() for t in wide]):
        got = run(*rows, causal, p)
        for name, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), got, exp):
            if name == "LSE":
                assert torch.equal(a, b), name
            else:
                assert torch.equal(a, b[..., :d]), (name, float((a.float() - b[..., :d].float()).abs().max()))
                assert not b[..., d:].any()
