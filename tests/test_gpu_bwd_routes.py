"""The three routes of the backward beyond the smallest grids: both sides in one grid (unpaired, paired, an odd
tile in the middle, two and three tiles per head, unequal lengths, dropout) and, just above its limits,
one kernel per side.  Every element against the oracle, and the route of every case against the list it stands in.
"""
import math

import pytest

from paper_2502_12784_amd import load_library, synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# (B, H, Nq, Nk, d, dtype, causal, dropout threshold or 0); n = 128-row tiles of both sides
MERGED = [
    (1, 33, 128, 128, 64, synth.F16, False, 0), (2, 10, 250, 250, 128, synth.BF16, True, 0),    # n = 66, 80
    (2, 9, 100, 700, 64, synth.BF16, False, 0), (2, 9, 700, 100, 104, synth.F16, False, 26),    # 126
    (1, 20, 1100, 1100, 64, synth.F16, False, 0), (4, 14, 600, 600, 64, synth.F16, True, 26),  # 360, 560
    (4, 13, 600, 600, 64, synth.BF16, True, 0), (3, 13, 600, 600, 128, synth.F16, True, 26),    # 520, 390: paired, odd
    (3, 43, 250, 250, 64, synth.F16, True, 0), (2, 60, 250, 250, 64, synth.BF16, True, 0),      # 516, 480: two tiles
    (2, 60, 250, 250, 128, synth.F16, True, 0), (3, 20, 300, 300, 64, synth.F16, True, 26),     # 480; 360: three tiles
]
SEPARATE = [
    (1, 6, 1, 1600, 128, synth.F16, False, 0), (1, 3, 40, 2900, 104, synth.BF16, False, 26),     # long memories
    (2, 33, 250, 250, 64, synth.F16, False, 0), (2, 33, 250, 250, 128, synth.BF16, False, 26),  # n = 264
    (4, 27, 600, 600, 64, synth.BF16, True, 0), (4, 14, 600, 600, 128, synth.F16, True, 0),     # 1080, 560
    (2, 32, 257, 129, 40, synth.BF16, False, 26), (3, 60, 300, 300, 128, synth.BF16, True, 0),  # 320, 1080
    # causal with dropout, d <= 64: five tiles per head, four, three, two
    (4, 27, 600, 600, 64, synth.F16, True, 26), (4, 27, 600, 600, 64, synth.BF16, True, 26),    # 1080
    (3, 43, 500, 500, 56, synth.BF16, True, 26), (3, 30, 300, 300, 64, synth.F16, True, 26),    # 1032, 540
    (2, 140, 200, 200, 64, synth.BF16, True, 26),                                               # 1120
]


@pytest.mark.parametrize("case", MERGED + SEPARATE)
def test_backward_routes(case):
    B, H, Nq, Nk, d, dtype, causal, thr = case
    grids = load_library().spark_mha_bwd_grids(B, H, Nq, Nk, d, causal, thr / 256.0, int(dtype == synth.BF16))
    assert grids == (1 if case in MERGED else 2)
    scale = 1.0 / math.sqrt(d)
    inp = synth.make_inputs(B, H, Nq, d, dtype, seed=7300 + Nq + Nk + d, Nk=Nk)
    print(f"\n[routes] {case}", flush=True)
    gpu = pu.run_gpu(inp, dtype, scale, causal, dropout=(thr / 256.0, 4711, 3) if thr else None)
    ref = pu.run_oracle(inp, dtype, scale, causal, dropout=(thr, 4711, 3) if thr else None)
    m = pu.compare(gpu, ref, dtype)
    print(f"[routes] {case}: {m}", flush=True)
    pu.assert_within_tolerance(m, case)
