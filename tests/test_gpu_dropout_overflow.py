"""Dropped entries whose dP = dO V^T is past fp32's range (bf16 holds such operands): they count for nothing, so O,
LSE and the gradients are finite and those of the oracle.  Each route of the backward and both tile widths.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2502_12784_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# (H, Nq, Nk, causal): split over waves, both sides in one grid, one kernel per side (both tile widths each)
SHAPES = [(2, 64, 96, False), (2, 96, 96, True), (20, 128, 640, False), (14, 400, 400, True), (60, 200, 300, False),
          (180, 200, 200, True)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", SHAPES)
def test_dropped_entries_past_the_range_of_fp32(shape, d):
    H, Nq, Nk, causal = shape
    thr, seed, offset = 128, 4711, 3
    inp = synth.make_inputs(1, H, Nq, d, synth.BF16, seed=8200 + Nq + d, Nk=Nk, sigma_v=1e-20, sigma_do=0.0)
    keep = oracle.dropout_mask(1, H, Nq, Nk, seed, offset, thr)
    row = Nq - 1  # the only query with a gradient; V of the first key it drops is 1e20, of all others about 1e-20
    for h in range(H):
        key = int(np.flatnonzero(keep[0, h, row, :row + 1 if causal else Nk] == 0)[0])
        inp["V"][0, h, key] = synth.round_to_bits(np.full(d, 1e20, np.float32), synth.BF16)
        inp["dO"][0, h, row] = synth.round_to_bits(np.full(d, 1e20, np.float32), synth.BF16)
    scale = 1.0 / math.sqrt(d)
    print(f"\n[overflow] {shape} d={d}", flush=True)
    gpu = pu.run_gpu(inp, synth.BF16, scale, causal, dropout=(thr / 256.0, seed, offset))
    ref = pu.run_oracle(inp, synth.BF16, scale, causal, dropout=(thr, seed, offset))
    for n in ("O", "LSE", "dQ", "dK", "dV"):
        got = pu.to_f64(gpu[n])
        assert np.isfinite(ref[n]).all() and np.isfinite(got).all(), n
        # the bar of every gradient here (O and LSE are held to it as well: O spans 40 orders of magnitude)
        assert np.linalg.norm(got - ref[n]) <= pu.TOL_REL_L2 * np.linalg.norm(ref[n]), n
