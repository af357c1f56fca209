"""Which kernels a call launches, at the edges of the rules that the timings beside them in csrc/spark_mha.hip draw: the
call is captured into a graph (nothing runs) and the grids of its kernel nodes are compared.
"""
import ctypes
import math

import pytest

pytestmark = pytest.mark.gpu


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint), ("y", ctypes.c_uint), ("z", ctypes.c_uint)]


class _KernelNode(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("smem", ctypes.c_uint)]


def _grids(call):
    """Grid sizes (in x) of the kernels that `call` launches, in order."""
    return [grid for grid, _ in _launches(call)]


def _launches(call):
    """(grid size, threads per workgroup) of the same."""
    import torch
    hip = ctypes.CDLL("libamdhip64.so")
    call()  # sets the kernels up, outside of the capture
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    stream, graph, n = ctypes.c_void_p(side.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    with torch.cuda.stream(side):
        assert hip.hipStreamBeginCapture(stream, 1) == 0
        try:
            call()
        finally:
            assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        out.append((p.grid.x, p.block.x))
    assert hip.hipGraphDestroy(graph) == 0
    return out


def _tensors(H, Nq, Nk, d):
    import torch
    def z(n):
        return torch.zeros(1, H, n, d, dtype=torch.float16, device="cuda")
    return z(Nq), z(Nk), z(Nk), z(Nq), torch.zeros(1, H, Nq, device="cuda"), z(Nq)


def _backward(H, Nq, Nk, d, causal, p):
    import torch
    from paper_2502_12784_amd import spark_mha_dropout_bwd
    Q, K, V, O, L, dO = _tensors(H, Nq, Nk, d)
    out = [torch.empty_like(t) for t in (Q, K, V)]
    ws = torch.empty(8 * H * Nq + 16, dtype=torch.uint8, device="cuda")
    return _grids(lambda: spark_mha_dropout_bwd(Q, K, V, O, L, dO, 1 / math.sqrt(d), causal, p, 1, 0, *out, ws))


def _stats(H, Nq, d):  # grid of the pass in front of the backward in one grid: 2048 elements per workgroup
    per = 2048 // (64 if d <= 64 else 128)
    return (H * Nq + per - 1) // per


# heads, N, d, dropout rate, whether both sides run in one grid (causal, one tile of 128 rows per head and side)
ONE_TILE = [(128, 64, 128, 0.0, True), (129, 64, 128, 0.0, False), (240, 128, 96, 0.0, False), (128, 128, 64, 0.1, True),
            (200, 100, 64, 0.1, False), (384, 128, 64, 0.0, True), (385, 128, 64, 0.0, False)]


@pytest.mark.parametrize("case", ONE_TILE)
def test_causal_heads_of_one_tile(case):
    H, N, d, p, one_grid = case
    assert _backward(H, N, N, d, True, p) == ([_stats(H, N, d), 2 * H] if one_grid else [H, H])


# heads, N, d, dropout rate, whether the dK/dV kernel pairs the two causal tiles of a head (beyond the merged grids)
TWO_TILES = [(140, 192, 64, 0.1, False), (256, 200, 64, 0.1, False), (257, 200, 64, 0.1, True), (130, 256, 128, 0.0, True), (257, 256, 64, 0.0, True)]


@pytest.mark.parametrize("case", TWO_TILES)
def test_causal_heads_of_two_tiles(case):
    H, N, d, p, paired = case
    assert _backward(H, N, N, d, True, p)[1] == (H if paired else 2 * H)


# the same for three tiles: paired (two workgroups per head) or not
THREE_TILES = [(88, 300, 128, 0.0, False), (89, 300, 128, 0.0, True), (128, 384, 128, 0.0, True), (129, 384, 128, 0.0, False),
               (200, 300, 64, 0.0, False), (90, 320, 64, 0.1, False), (130, 320, 64, 0.1, False)]


@pytest.mark.parametrize("case", THREE_TILES)
def test_causal_heads_of_three_tiles(case):
    H, N, d, p, paired = case
    assert _backward(H, N, N, d, True, p)[1] == (2 * H if paired else 3 * H)


def _forward(H, Nq, Nk, d, causal, p, launches=_grids):
    from paper_2502_12784_amd import spark_mha_dropout_fwd
    Q, K, V, O, L, _ = _tensors(H, Nq, Nk, d)
    return launches(lambda: spark_mha_dropout_fwd(Q, K, V, 1 / math.sqrt(d), causal, p, 1, 0, O, L))


# heads, d, dropout rate, whether the forward pairs the three causal tiles of a head
THREE_TILES_FWD = [(192, 128, 0.0, False), (193, 128, 0.0, True), (256, 96, 0.0, True), (257, 128, 0.0, False),
                   (220, 64, 0.0, False), (220, 128, 0.1, False)]


@pytest.mark.parametrize("case", THREE_TILES_FWD)
def test_forward_of_causal_heads_of_three_tiles(case):
    H, d, p, paired = case
    assert _forward(H, 300, 300, d, True, p) == [2 * H if paired else 3 * H]


# heads, N, d, dropout rate, whether the causal forward has workgroups of 8 waves for 256 rows
WIDE = [(30, 2303, 80, 0.0, True), (30, 2240, 96, 0.1, True), (30, 2303, 128, 0.0, True), (30, 2047, 96, 0.0, False),
        (30, 2303, 64, 0.0, False)]


@pytest.mark.parametrize("case", WIDE)
def test_causal_forward_of_wide_workgroups(case):
    H, N, d, p, wide = case
    tiles = (N + 255) // 256 if wide else (N + 127) // 128
    assert _forward(H, N, N, d, True, p, _launches) == [(H * ((tiles + 1) // 2), 512 if wide else 256)]


# heads, Nq, Nk, d, dropout rate, whether both sides run in one grid
FEW_QUERIES = [(8, 256, 1536, 128, 0.0, True), (8, 256, 1537, 96, 0.0, False), (6, 1, 1600, 128, 0.0, False),
               (4, 100, 5000, 64, 0.0, True), (8, 256, 2432, 128, 0.1, True), (8, 256, 2433, 128, 0.1, False),
               (4, 5000, 100, 128, 0.0, True)]


@pytest.mark.parametrize("case", FEW_QUERIES)
def test_backward_of_few_queries_over_many_keys(case):
    H, Nq, Nk, d, p, one_grid = case
    nq, nk = H * ((Nq + 127) // 128), H * ((Nk + 127) // 128)
    assert _backward(H, Nq, Nk, d, False, p) == ([_stats(H, Nq, d), nq + nk] if one_grid else [nq, nk])


# heads, Nq, Nk, d, dropout rate, whether the forward splits the keys over the 8 waves of 32-row workgroups, or has
# 4 waves for 128 rows
FEW_ROWS = [(256, 32, 2048, 128, 0.0, True), (257, 32, 2048, 128, 0.0, False), (319, 1, 3000, 128, 0.0, False),
            (320, 1, 3000, 128, 0.0, True), (300, 1, 3000, 120, 0.0, True), (300, 1, 3000, 128, 0.1, True),
            (150, 64, 2500, 128, 0.0, False), (150, 64, 2500, 112, 0.0, True), (240, 64, 2500, 120, 0.0, False),
            (100, 96, 8191, 128, 0.0, True), (100, 96, 8192, 128, 0.0, False), (104, 96, 10400, 104, 0.0, False),
            (70, 129, 2500, 128, 0.0, True), (256, 32, 384, 128, 0.0, False), (256, 32, 705, 128, 0.0, True),
            (224, 32, 384, 128, 0.0, True), (256, 32, 384, 96, 0.0, True)]


@pytest.mark.parametrize("case", FEW_ROWS)
def test_forward_of_few_rows(case):
    H, Nq, Nk, d, p, split = case
    want = (H * ((Nq + 31) // 32), 512) if split else (H * ((Nq + 127) // 128), 256)
    assert _forward(H, Nq, Nk, d, False, p, _launches) == [want]


def test_bwd_grids_reports_the_route():
    """spark_mha_bwd_grids against the launches: one kernel, or the statistics pass and one grid, or one kernel per side."""
    from paper_2502_12784_amd import load_library
    lib = load_library()
    for H, Nq, Nk, d, causal, p in ((2, 128, 128, 64, 0, 0.0), (128, 64, 64, 128, 1, 0.0), (129, 64, 64, 128, 1, 0.0),
                                    (20, 1100, 1100, 64, 0, 0.0), (20, 1100, 1100, 64, 0, 0.1), (8, 256, 1536, 128, 0, 0.0),
                                    (8, 256, 1537, 96, 0, 0.0), (140, 192, 192, 64, 1, 0.1)):
        got = _backward(H, Nq, Nk, d, bool(causal), p)
        one_grid = len(got) == 1 or got[0] == _stats(H, Nq, d)
        assert lib.spark_mha_bwd_grids(1, H, Nq, Nk, d, causal, p, 0) == (1 if one_grid else 2), (H, Nq, Nk, d, causal, p, got)
    assert lib.spark_mha_bwd_grids(1, 2, 8, 16, 64, 1, 0.0, 0) < 0  # causal needs a square
