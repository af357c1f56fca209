"""The backward for small grids (32 rows per workgroup, the other dimension split over its waves, dQ and
dK/dV in one launch) at the sizes where it can go wrong: one row, one row more or less than a tile,
lengths that leave waves without a tile, with one, or with an odd number of them (both stages of the
double buffer), causal diagonals, dropout, head sizes between the tile widths, the largest grid the
rule takes.  Every element against the oracle.
"""
import math

import pytest

from paper_2502_12784_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# (B, H, Nq, Nk, d, dtype, causal, dropout threshold or 0).  Two keys at least with dropout: with one, P is 1
# and dS = P o (dP - D) vanishes, so dK is what the 16-bit rounding of O leaves in D, about
# sqrt(N d) 2^-9 |O| |dO| in bf16, and no relative bound exists.
CASES = [
    (1, 1, 1, 1, 64, synth.F16, False, 0), (1, 2, 1, 300, 128, synth.F16, False, 0),
    (2, 1, 300, 2, 64, synth.BF16, False, 26), (1, 2, 31, 33, 128, synth.BF16, False, 0),
    (1, 2, 33, 31, 64, synth.F16, False, 26), (1, 2, 128, 128, 64, synth.F16, False, 0),
    (1, 3, 257, 1000, 64, synth.F16, False, 0), (1, 3, 1000, 257, 128, synth.F16, False, 26),
    (1, 2, 129, 800, 72, synth.BF16, False, 0), (2, 2, 555, 555, 40, synth.F16, False, 0),
    (1, 2, 33, 33, 128, synth.F16, True, 0), (1, 2, 257, 257, 64, synth.F16, True, 0),
    (1, 2, 545, 545, 64, synth.BF16, True, 26), (1, 2, 161, 161, 128, synth.F16, True, 26),
    (1, 3, 1037, 1037, 128, synth.BF16, True, 0), (4, 8, 256, 256, 64, synth.F16, True, 0),
    (4, 8, 256, 256, 128, synth.F16, False, 0),
]


@pytest.mark.parametrize("case", CASES)
def test_split_backward(case):
    B, H, Nq, Nk, d, dtype, causal, thr = case
    scale = 1.0 / math.sqrt(d)
    inp = synth.make_inputs(B, H, Nq, d, dtype, seed=7100 + Nq + Nk + d, Nk=Nk)
    print(f"\n[split] {case}", flush=True)
    gpu = pu.run_gpu(inp, dtype, scale, causal, dropout=(thr / 256.0, 4711, 3) if thr else None)
    ref = pu.run_oracle(inp, dtype, scale, causal, dropout=(thr, 4711, 3) if thr else None)
    m = pu.compare(gpu, ref, dtype)
    print(f"[split] {case}: {m}", flush=True)
    pu.assert_within_tolerance(m, case)
