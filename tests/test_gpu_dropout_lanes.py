"""The rows of a block may be spread over the lanes in two ways by the dropout kernels of the backward's 128-row tiles, by
the strides of the operands' rows and the length of the loop (far_rows in csrc/spark_mha.hip).  Which lane holds a row does not
enter its arithmetic: the same problem with rows further apart gives the same bits."""
import math

import pytest

from paper_2502_12784_amd import load_library

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float16", "bfloat16"])
@pytest.mark.parametrize("heads, Nq, Nk, d, causal, grids", [
    (160, 203, 203, 64, False, 2), (160, 203, 203, 64, True, 2), (160, 203, 140, 48, False, 2), (160, 190, 190, 32, True, 2),
    (130, 140, 300, 40, False, 2), (40, 530, 520, 128, False, 2), (40, 1030, 1030, 128, True, 2), (40, 1030, 1030, 112, True, 2),
    (20, 530, 520, 64, False, 1), (50, 300, 300, 48, True, 1), (11, 700, 530, 128, False, 1), (20, 1030, 1030, 128, True, 1)])
def test_row_strides_do_not_change_the_bits(heads, Nq, Nk, d, causal, grids, dtype):
    import torch
    from paper_2502_12784_amd import spark_mha_strided_bwd, spark_mha_strided_fwd
    dt = getattr(torch, dtype)
    assert load_library().spark_mha_bwd_grids(1, heads, Nq, Nk, d, causal, 0.1, int(dtype == "bfloat16")) == grids
    print(f"\n[lanes] {heads} x {Nq} over {Nk}, d = {d}, {'causal' if causal else 'full'} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(11)
    src = [torch.randn(1, heads, n, d, generator=g, device="cuda").to(dt) for n in (Nq, Nk, Nk, Nq)]

    def run(pads):
        q, k, v, do = (torch.empty(1, heads, t.shape[2], d + p, device="cuda", dtype=dt)[..., :d].copy_(t)
                       for t, p in zip(src, pads))
        args = (1.0 / math.sqrt(d), causal, 0.1, 4711, 3)
        O, L = spark_mha_strided_fwd(q, k, v, *args, O=torch.empty_like(src[0]))
        return (O, L) + spark_mha_strided_bwd(q, k, v, O, L, do, *args, *(torch.empty_like(t) for t in src[:3]))

    want = run((0, 0, 0, 0))
    # rows of every residue of 128 bytes that decides, in all operands and in one of them
    for pads in [(8,) * 4, (16,) * 4, (128 - d % 64,) * 4, (0, 16, 0, 0), (0, 0, 0, 16), (16, 0, 8, 0)]:
        for name, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), want, run(pads)):
            assert torch.equal(a, b), (name, pads)
