"""Checks on the compiled device code that need no GPU."""
import os
import re

import pytest

from paper_2502_12784_amd import build


@pytest.fixture(scope="module")
def asm():
    return build.device_assembly()[0]


def test_every_direct_lds_load_carries_its_hazard_guard(asm):
    """The global->LDS loads are inline assembly, invisible to the compiler's hazard handling: each
    must be preceded by the five wait states that separate it from a VALU write of the scalar
    registers (descriptor, offset, M0) it reads."""
    loads = re.findall(r"buffer_load_dword(?:x4)? .* lds", asm)
    assert len(loads) > 500          # every attention kernel uses them
    assert build.unguarded_lds_loads(asm) == []


def test_no_packed_fp32_arithmetic(asm):
    """The library is built with packed fp32 operations switched off."""
    assert not re.search(r"\bv_pk_(add|mul|fma)_f32\b", asm)


def test_tile_loops_do_not_spill():
    table = build.kernel_resources()
    rows = [l.split() for l in table.splitlines() if l.startswith("mha_")]
    assert len(rows) > 60
    assert all(r[-1] == "0" for r in rows), [r for r in rows if r[-1] != "0"]


def test_waits_without_a_barrier_are_compiler_fences():
    """In the split kernels a wave reads LDS that its own direct loads filled, with no barrier between.  Nothing but a
    memory clobber keeps the compiler from moving such a read in front of the wait: the bare wait_vmem_all()
    belongs in front of a barrier, these kernels wait with wait_vmem<N>() and wait_lds_all()."""
    def code(name):
        return re.sub(r"//.*", "", open(os.path.join(build.CSRC, name)).read())
    for name in ("fwd_split_kernel.hpp", "bwd_split_kernel.hpp"):
        assert "load16_to_lds" in code(name) or ".template tile<" in code(name)
        assert "wait_vmem<" in code(name) and "wait_vmem_all" not in code(name), name
    helpers = code("mma_gfx950.hpp")
    for asm_text in (r's_waitcnt vmcnt\(%0\)" ::"n"\(N\)', r's_waitcnt lgkmcnt\(0\)" ::'):
        assert re.search(asm_text + r'[^;]*: "memory"\)', helpers)


def test_host_binding_needs_no_compiler_but_hipccs(monkeypatch, tmp_path):
    """Without g++ the host extension is compiled with the clang++ of the ROCm toolchain."""
    seen = []

    def run(cmd, **_):
        seen.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return type("Done", (), {"returncode": 0, "stdout": ""})

    monkeypatch.setattr(build, "HOST_EXT", str(tmp_path / "_spark_host.so"))
    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    monkeypatch.delenv("CXX", raising=False)
    build.build_host_binding()
    assert os.path.exists(seen[0][0]) and seen[0][0].endswith("clang++")
    monkeypatch.setenv("CXX", "some-c++")
    build.build_host_binding()
    assert seen[1][0] == "some-c++"
