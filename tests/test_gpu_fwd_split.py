"""The forward for small grids (32 query rows per workgroup, keys split over its 8 waves) at the sizes
where it can go wrong: one query row and one row more or less than a tile, key counts that leave
waves without a tile or with a masked one, odd numbers of causal tiles, paired and unpaired causal
tiles, a head size between the tile widths.  Every element against the oracle.
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
