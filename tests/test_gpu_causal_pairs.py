"""Causal grids on both sides of the rule that pairs complementary tiles in one workgroup: with and
without a lone middle tile, two and three tiles per head, grids that just exceed one tile per CU.
Every element of every output against the oracle.
"""
import math

import pytest

from paper_2502_12784_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# (B, H, N, d, dtype): tiles per head = ceil(N / 128), paired above 256 tiles in all unless 2 or 3 per head
CASES = [
    (4, 13, 600, 64, synth.F16), (4, 13, 600, 128, synth.BF16),    # 260 tiles, 5 per head
    (2, 32, 512, 128, synth.F16), (1, 65, 512, 64, synth.BF16),    # 256 and 260 tiles, 4 per head
    (3, 43, 250, 64, synth.F16), (3, 43, 250, 128, synth.BF16),    # 258 tiles, 2 per head
    (5, 52, 130, 64, synth.BF16),                                  # 520 tiles, 2 per head
    (3, 30, 300, 128, synth.F16),                                  # 270 tiles, 3 per head
    (2, 47, 300, 128, synth.BF16), (2, 100, 270, 96, synth.F16),   # 282 and 600 tiles, 3 per head: dK/dV, forward paired
]


@pytest.mark.parametrize("case", CASES)
def test_causal_pairs(case):
    B, H, N, d, dtype = case
    scale = 1.0 / math.sqrt(d)
    inp = synth.make_inputs(B, H, N, d, dtype, seed=7200 + N + d)
    print(f"\n[pairs] {case}", flush=True)
    m = pu.compare(pu.run_gpu(inp, dtype, scale, True), pu.run_oracle(inp, dtype, scale, True), dtype)
    print(f"[pairs] {case}: {m}", flush=True)
    pu.assert_within_tolerance(m, case)
