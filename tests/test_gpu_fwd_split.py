"""The forward for small grids (32 query rows per workgroup, keys split over its 8 waves) at the sizes
where it can go wrong: one query row and one row more or less than a tile, key counts that leave
waves without a tile or with a masked one, odd numbers of causal tiles, paired and unpaired causal
tiles, a head size between the tile widths; and few rows against long memories, where several workgroups
share the keys of a row (a short last part, a last part whose only tile is ragged).  Every element against the oracle.
"""
import math

import pytest

from paper_2502_12784_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# (B, H, Nq, Nk, d, dtype, causal, dropout threshold or 0)
CASES = [
    (1, 1, 1, 257, 64, synth.F16, False, 0), (2, 3, 1, 2048, 128, synth.BF16, False, 0),
    (1, 2, 31, 512, 128, synth.F16, False, 0), (1, 2, 33, 513, 64, synth.BF16, False, 26),
    (1, 2, 32, 1000, 72, synth.F16, False, 0), (1, 2, 300, 300, 128, synth.F16, False, 26),
    (1, 2, 257, 257, 64, synth.F16, True, 0), (1, 1, 321, 321, 128, synth.BF16, True, 0),
    (1, 2, 1037, 1037, 64, synth.BF16, True, 26),
    (4, 8, 290, 290, 64, synth.F16, True, 0), (4, 8, 290, 290, 128, synth.BF16, True, 26),  # paired, odd
    (1, 8, 2048, 2048, 64, synth.F16, False, 0), (2, 17, 300, 2050, 128, synth.BF16, False, 0),  # two rounds
    (1, 5, 4100, 4100, 64, synth.BF16, True, 0),
    # shared keys
    (1, 1, 1, 6200, 64, synth.F16, False, 0), (1, 3, 1, 16384, 128, synth.BF16, False, 0),
    (1, 2, 33, 5000, 72, synth.F16, False, 0), (2, 2, 7, 4097, 128, synth.F16, False, 26),
    (1, 4, 40, 8193, 64, synth.BF16, False, 26), (16, 8, 1, 6145, 40, synth.F16, False, 0),
]


@pytest.mark.parametrize("case", CASES)
def test_split_forward(case):
    B, H, Nq, Nk, d, dtype, causal, thr = case
    scale = 1.0 / math.sqrt(d)
    inp = synth.make_inputs(B, H, Nq, d, dtype, seed=6100 + Nq + Nk + d, Nk=Nk)
    print(f"\n[split] {case}", flush=True)
    gpu = pu.run_gpu(inp, dtype, scale, causal, dropout=(thr / 256.0, 4711, 3) if thr else None)
    ref = pu.run_oracle(inp, dtype, scale, causal, dropout=(thr, 4711, 3) if thr else None)
    m = pu.compare(gpu, ref, dtype)
    print(f"[split] {case}: {m}", flush=True)
    pu.assert_within_tolerance(m, case)


def test_workspace_is_optional_and_checked():
    import ctypes
    import torch
    import paper_2502_12784_amd as pkg
    lib = pkg.load_library()
    B, H, Nq, Nk, d = 1, 2, 3, 8000, 64
    need = lib.spark_mha_fwd_workspace_bytes(B, H, Nq, Nk, d, 0, 0)
    assert need > 0 and lib.spark_mha_fwd_workspace_bytes(B, H, Nk, Nk, d, 1, 0) == 0
    Q, K, V = (torch.randn(B, H, n, d, device="cuda").half() for n in (Nq, Nk, Nk))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    sq, sk = pkg.Strides(H * Nq * d, Nq * d, d), pkg.Strides(H * Nk * d, Nk * d, d)

    def call(pointer, size):
        O, L = torch.empty_like(Q), torch.empty(B, H, Nq, device="cuda")
        rc = lib.spark_mha_workspace_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), L.data_ptr(), sq, sk,
                                         sk, sq, pointer, size, B, H, Nq, Nk, d, 0.125, 0, 0.0, 0, 0, 0,
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        return rc, O, L

    assert call(ws.data_ptr(), need - 1)[0] == -5 and call(ws.data_ptr() + 4, need)[0] == -4
    rc, O, L = call(ws.data_ptr(), need)
    rc0, O0, L0 = call(None, 0)  # one workgroup per row: the same results up to rounding
    assert rc == rc0 == 0
    # P is rounded to fp16 (2^-11 relative) against another reference m: O = sum p v / sum p moves by at most
    # 2 * 2^-11 max|v|, and its own rounding by 2 * 2^-11 |O|
    torch.testing.assert_close(O, O0, rtol=2 ** -10, atol=2 ** -10 * float(V.abs().max()))
    torch.testing.assert_close(L, L0, rtol=1e-6, atol=1e-6)
    for x, y in zip((O, L), pkg.spark_mha_cross_fwd(Q, K, V, 0.125)):
        assert torch.equal(x, y)  # what the binding calls, bit for bit
