"""The native marshalling of ordinary calls (csrc/host_binding.cpp) against the general ctypes path: the same
kernels, so the same bits, layouts and errors; and calls that it must leave to the general path."""
import pytest

pytestmark = pytest.mark.gpu


class _NotTaken:
    """Stands in for the extension: takes no call."""

    @staticmethod
    def fwd(*args):
        return None

    bwd = fwd


def _calls(kind, dtype):
    import torch
    import paper_2502_12784_amd as pkg
    g = torch.Generator(device="cuda").manual_seed(7)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dtype)
    if kind == "packed":
        qkv, dO = n(2, 77, 3, 3, 40), n(2, 77, 3, 40).permute(0, 2, 1, 3)
        Q, K, V = (qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3))
        O, L = pkg.spark_mha_strided_fwd(Q, K, V, 0.2, True, 0.1, -5, 1 << 40)
        return (O, L) + pkg.spark_mha_strided_bwd(Q, K, V, O, L, dO, 0.2, True, 0.1, -5, 1 << 40)
    if kind.startswith("few"):  # few queries, long memories: workgroups share the keys, through a workspace
        kv, q = n(2, 8000, 2, 2, 64), n(2, 3, 2, 64)
        Q, K, V = q.permute(0, 2, 1, 3), kv[:, :, 0].permute(0, 2, 1, 3), kv[:, :, 1].permute(0, 2, 1, 3)
        if kind == "few-strided":
            return pkg.spark_mha_strided_fwd(Q, K, V, 0.125) + pkg.spark_mha_strided_fwd(Q, K, V, 0.125, False, 0.1, 7, 1)
        Q, K, V = Q.contiguous(), K.contiguous(), V.contiguous()
        return pkg.spark_mha_cross_fwd(Q, K, V, 0.125) + pkg.spark_mha_dropout_fwd(Q, K, V, 0.125, False, 0.1, 7, 1)
    if kind == "long":
        return pkg.spark_mha_fwd(*(n(1, 1, 3000, 128) for _ in range(3)), 0.088, False)
    Nk = 130 if kind == "cross" else 70
    Q, dO, K, V = n(2, 3, 70, 64), n(2, 3, 70, 64), n(2, 3, Nk, 64), n(2, 3, Nk, 64)
    if kind == "self":
        O, L = pkg.spark_mha_fwd(Q, K, V, 0.125, True)
        return (O, L) + pkg.spark_mha_bwd(Q, K, V, O, L, dO, 0.125, True)
    if kind == "given":  # outputs of the caller
        O, L, dQ, dK, dV = (torch.full_like(Q, 9.0) for _ in range(5))
        L = torch.full((2, 3, 70), 9.0, device="cuda")
        out = pkg.spark_mha_fwd(Q, K, V, 0.125, False, O, L)
        grads = pkg.spark_mha_bwd(Q, K, V, O, L, dO, 0.125, False, dQ, dK, dV)
        assert out[0].data_ptr() == O.data_ptr() and grads[2].data_ptr() == dV.data_ptr()
        return out + grads
    if kind == "dropout":
        O, L = pkg.spark_mha_dropout_fwd(Q, K, V, 0.125, False, 0.1, 12345678901234, 3)
        return (O, L) + pkg.spark_mha_dropout_bwd(Q, K, V, O, L, dO, 0.125, False, 0.1, 12345678901234, 3)
    O, L = pkg.spark_mha_cross_fwd(Q, K, V, 0.125)
    return (O, L) + pkg.spark_mha_cross_bwd(Q, K, V, O, L, dO, 0.125)


@pytest.mark.parametrize("dtype", ["float16", "bfloat16"])
@pytest.mark.parametrize("kind", ["self", "given", "cross", "dropout", "packed", "few", "few-strided", "long"])
def test_native_and_general_path_agree(kind, dtype, monkeypatch):
    import torch
    from paper_2502_12784_amd import binding
    binding.load_library()
    dt = getattr(torch, dtype)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # the current stream, not the default one
        got = _calls(kind, dt)
    side.synchronize()
    monkeypatch.setattr(binding, "_host", _NotTaken)
    want = _calls(kind, dt)
    for a, b in zip(got, want):
        assert a.shape == b.shape and a.stride() == b.stride() and a.dtype == b.dtype
        assert torch.equal(a, b)


def test_unusual_calls_take_the_general_path():
    import torch
    from paper_2502_12784_amd import SparkError, binding, spark_mha_fwd
    binding.load_library()
    q = torch.randn(1, 2, 33, 64, device="cuda").half()
    host = binding._host
    args = (None, None, 0.125, False, 0.0, 0, 0, 0)
    assert host.fwd(q, q, q, *args) is not None
    for bad in (q.cpu(), q[0], q.float(), q.transpose(2, 3), torch.nn.Parameter(q).to_sparse(), q[:, :, :32], "q"):
        assert host.fwd(q, bad, q, *args) is None
    assert host.fwd(q, q, q, None, None, 1, False, 0.0, 0, 0, 0) is None  # an int for the scale
    O, _ = spark_mha_fwd(q, q, q, 1, 0)                                   # ... which the general path converts
    assert torch.equal(O, spark_mha_fwd(q, q, q, 1.0, False)[0])
    with pytest.raises(ValueError):
        spark_mha_fwd(q, q[:, :, :32], q, 0.125, False)
    with pytest.raises(SparkError):
        spark_mha_fwd(q, q, q, float("nan"), False)
    with pytest.raises(SparkError):
        spark_mha_fwd(q.float(), q.float(), q.float(), 0.125, False)


@pytest.mark.parametrize("watched", ["not", "profiler", "inference"])
def test_allocated_outputs_are_those_of_empty_like(watched, monkeypatch):
    """Outputs that the call allocates by itself: the layout of empty_like, and nobody who watches allocations misses one.
    The dispatcher reports an allocation to a profiler, the device's allocation kernel by itself does not."""
    import contextlib
    import torch
    from paper_2502_12784_amd import binding, spark_mha_strided_bwd, spark_mha_strided_fwd
    binding.load_library()
    dense = torch.randn(2, 3, 40, 64, device="cuda").half()
    views = [dense, dense.transpose(0, 1).contiguous().transpose(0, 1), dense.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3),
             dense[:, :1], dense[:1, :, :, :32], dense.as_strided((1, 3, 40, 64), (8, 2560, 64, 1)), dense[:, :, :1]]
    host, taken = binding._host, []

    class Seen:
        fwd = staticmethod(lambda *a: taken.append(host.fwd(*a)) or taken[-1])
        bwd = staticmethod(lambda *a: taken.append(host.bwd(*a)) or taken[-1])

    monkeypatch.setattr(binding, "_host", Seen)
    for q in views:
        grad = torch.empty_like(q).copy_(q)
        watch = {"not": contextlib.nullcontext, "inference": torch.inference_mode,
                 "profiler": lambda: torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU])}[watched]()
        with watch:
            O, L = spark_mha_strided_fwd(q, q, q, 0.125)
            out = (O,) + spark_mha_strided_bwd(q, q, q, O, L, grad, 0.125)
        for t in out:
            assert t.stride() == torch.empty_like(q).stride() and t.device == q.device and not t.requires_grad
        assert L.stride() == torch.empty(L.shape).stride() and L.dtype == torch.float32
        assert all(t.is_inference() == (watched == "inference") for t in out + (L,))
        if watched == "profiler":  # O, LSE, dQ, dK, dV and the workspace
            names = [e.name for e in watch.events()]
            assert sum(n in ("aten::empty", "aten::empty_like", "aten::empty_strided") for n in names) >= 6
    assert len(taken) == 2 * len(views) and all(t is not None for t in taken)


@pytest.mark.filterwarnings("ignore:Named tensors")
@pytest.mark.parametrize("layout", ["contiguous", "permuted"])
def test_allocated_outputs_keep_the_names_of_named_inputs(layout):
    """As torch.empty_like: O is named as Q, dQ, dK, dV as Q, K, V."""
    import torch
    from paper_2502_12784_amd import spark_mha_bwd, spark_mha_fwd, spark_mha_strided_bwd, spark_mha_strided_fwd
    names, memory = ("B", "H", "N", "d"), ("B", "H", "M", "d")
    x = torch.randn(2, 3, 40, 64, device="cuda").half()
    if layout == "permuted":
        x = x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    q, k = x.refine_names(*names), x.refine_names(*memory)
    entries = [(spark_mha_strided_fwd, spark_mha_strided_bwd)]
    if layout == "contiguous":
        entries.append((spark_mha_fwd, spark_mha_bwd))
    for fwd, bwd in entries:
        O, L = fwd(q, k, k, 0.125, False)
        outs = (O,) + tuple(bwd(q, k, k, O, L, q, 0.125, False))
        assert [t.names for t in outs] == [names, names, memory, memory] and L.names == (None,) * 3
        assert torch.equal(O.rename(None), fwd(x, x, x, 0.125, False)[0])
