"""The kernels of full grids (128-row forward, dQ, dK/dV; beyond the sizes that the split and, but for one case, the
joint grids take) on tensors of other layouts, with head dimensions below the tile width.  First and last head against
the oracle, the backward's route against the one stated.
"""
import math

import pytest

from paper_2502_12784_amd import load_library, synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# (B, H, Nq, Nk, d, dtype, causal, dropout threshold or 0, layout); forward tiles of 128 rows / of both backward sides
CASES = [
    (3, 12, 1333, 1333, 80, synth.BF16, True, 0, "packed"),     # 396 / 792
    (3, 12, 1333, 1333, 80, synth.F16, True, 26, "bnhd"),
    (2, 33, 300, 300, 40, synth.F16, False, 0, "packed"),       # 198 / 396
    (2, 33, 300, 300, 104, synth.BF16, False, 26, "padded"),
    (4, 27, 600, 600, 40, synth.BF16, True, 0, "padded"),       # 540 / 1080
    (4, 27, 600, 600, 56, synth.F16, True, 26, "packed"),       # 540 / 1080
    (4, 14, 600, 600, 104, synth.F16, True, 0, "bnhd"),         # 280 / 560
    (2, 30, 200, 700, 104, synth.BF16, False, 0, "bnhd"),       # 120 / 480
    (3, 40, 130, 400, 24, synth.F16, False, 26, "padded"),      # 240 / 720
]
ONE_GRID = (2, 27, 600, 600, 56, synth.F16, True, 26, "packed")  # 270 / 540


def _store(t, layout):
    """The same [B,H,N,d] values in other memory: [B,N,H,d], or rows padded by 8 elements (filled with 7)."""
    import torch
    B, H, N, d = t.shape
    if layout == "padded":
        s = torch.full((B, H, N, d + 8), 7.0, dtype=t.dtype, device=t.device)[..., :d]
    else:
        s = torch.empty(B, N, H, d, dtype=t.dtype, device=t.device).permute(0, 2, 1, 3)
    return s.copy_(t)


@pytest.mark.parametrize("case", CASES + [ONE_GRID])
def test_full_grids_on_other_layouts(case):
    import torch
    from paper_2502_12784_amd import spark_mha_strided_bwd, spark_mha_strided_fwd
    B, H, Nq, Nk, d, dtype, causal, thr, layout = case
    grids = load_library().spark_mha_bwd_grids(B, H, Nq, Nk, d, causal, thr / 256.0, int(dtype == synth.BF16))
    assert grids == (1 if case == ONE_GRID else 2)
    scale = 1.0 / math.sqrt(d)
    inp = synth.make_inputs(B, H, Nq, d, dtype, seed=9100 + Nq + d, Nk=Nk)
    dev = {n: pu.to_device(inp[n], dtype) for n in ("Q", "K", "V", "dO")}
    print(f"\n[full grid] {case}", flush=True)
    if layout == "packed":
        qkv = torch.stack([dev[n].permute(0, 2, 1, 3) for n in ("Q", "K", "V")], dim=2)
        Q, K, V = (qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3))
        dqkv = torch.empty_like(qkv)
        grads = [dqkv[:, :, i].permute(0, 2, 1, 3) for i in range(3)]
    else:
        Q, K, V = (_store(dev[n], layout) for n in ("Q", "K", "V"))
        grads = [_store(torch.zeros_like(t), layout) for t in (Q, K, V)]
    O, dO = _store(torch.zeros_like(dev["Q"]), layout), _store(dev["dO"], layout)
    drop = (thr / 256.0, 4711, 3)
    _, LSE = spark_mha_strided_fwd(Q, K, V, scale, causal, *drop, O=O)
    spark_mha_strided_bwd(Q, K, V, O, LSE, dO, scale, causal, *drop, dQ=grads[0], dK=grads[1], dV=grads[2])
    torch.cuda.synchronize()
    if layout == "padded":
        for t in [O] + grads:  # the eight elements behind each row are untouched
            assert t.as_strided(t.shape[:3] + (8,), t.stride(), d).eq(7.0).all()
    heads = [0, B * H - 1]
    ref = pu.run_oracle(inp, dtype, scale, causal, heads=heads, dropout=(thr, 4711, 3) if thr else None)
    gpu = dict(zip(("O", "LSE", "dQ", "dK", "dV"), [t.contiguous() for t in [O, LSE] + grads]))
    m = pu.compare(gpu, ref, dtype, heads=heads)
    print(f"[full grid] {case}: {m}", flush=True)
    pu.assert_within_tolerance(m, case)
