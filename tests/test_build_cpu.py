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


class Flow:
    """Order of memory events in one compiled kernel: 'row' (a load to registers), 'tile' (a direct global->LDS load),
    ('wait', N) (at most N vector memory operations outstanding), 'barrier' and 'mfma', with the branches between them."""

    def __init__(self, body):
        self.at, self.events, self.next = {}, [], []
        jumps = []
        for line in (l.split("//")[0].split(";")[0].strip() for l in body.split("\n")):
            op = line.split()[0] if line else ""
            if re.match(r"\.LBB\w+:", line):
                self.at[op[:-1]] = len(self.events)
                continue
            event = None
            if re.match(r"(buffer|global|flat)_load", op):
                event = "tile" if line.endswith(" lds") else "row"
            elif op == "s_waitcnt" and "vmcnt" in line:
                event = ("wait", int(re.search(r"vmcnt\((\d+)\)", line).group(1)))
            elif "mfma" in op or op in ("s_barrier", "s_endpgm"):
                event = "mfma" if "mfma" in op else op[2:]
            elif re.match(r"s_c?branch", op):
                event = "jump"
                jumps.append((len(self.events), line.split()[1], op == "s_branch"))
            if event:
                self.events.append(event)
                self.next.append([len(self.events)] if event != "endpgm" else [])
        for i, label, always in jumps:
            self.next[i] = [self.at[label]] + ([] if always else [i + 1])

    def behind(self, event, *ends):
        """Numbers of the events that can follow event number `event` with none of the kind `ends` before them."""
        seen, todo = set(), list(self.next[event])
        while todo:
            i = todo.pop()
            if i not in seen and i < len(self.events):
                seen.add(i)
                if self.events[i] not in ends:
                    todo += self.next[i]
        return seen


def kernel_flows(asm, name):
    for m in re.finditer(r"\n(_ZN5spark\d+%sI\w+):" % name, asm):
        body = asm[m.end():]
        yield m.group(1), Flow(body[:body.index("\n.Lfunc_end")])


def test_split_backward_does_not_wait_for_the_tile_it_has_requested(asm):
    """In the loops of the split backward a wave requests the next tile (and, for dK/dV, its row of O) and then works on
    the present one: up to the first matrix instruction nothing may wait for what has been requested."""
    kernels = list(kernel_flows(asm, "mha_bwd_split_kernel"))
    assert len(kernels) == 16
    for name, flow in kernels:
        runs = [i for i, e in enumerate(flow.events) if e == "tile" and (i == 0 or flow.events[i - 1] != "tile")]
        loops = [i for i in runs if i in flow.behind(i)]
        assert len(loops) >= 2, name  # dQ and dK/dV
        for i in loops:
            best = {}  # event -> most operations requested on a way to it
            todo = [(i, 0)]
            while todo:
                k, n = todo.pop()
                if best.get(k, -1) >= n or flow.events[k] == "mfma":
                    continue
                best[k] = n
                if isinstance(flow.events[k], tuple):
                    assert flow.events[k][1] >= n, (name, flow.events[k], n)
                todo += [(j, n + (flow.events[k] in ("tile", "row"))) for j in flow.next[k]]


@pytest.mark.parametrize("name, kernels", [("mha_bwd_dq_kernel", r"Li\d+ELb0E"), ("mha_bwd_dkdv_pipe_kernel", r"Li(64|96)ELb0E"),
                                           ("mha_bwd_merged_kernel", r"Li(64|96)ELb0E")])
def test_rows_and_first_tile_are_requested_together(asm, name, kernels):
    """Without a mask a backward workgroup requests its rows of Q, K, V, O and dO and its first tile, and only then waits:
    with a wait in between, the latencies of memory add up at its head."""
    flows = [(k, f) for k, f in kernel_flows(asm, name) if re.search(kernels, k)]
    assert len(flows) in (8, 12) and all("row" in f.events for _, f in flows)
    for kernel, flow in flows:
        for i in (i for i, e in enumerate(flow.events) if e == "row"):
            for w in (w for w in flow.behind(i, "tile", "mfma", "barrier") if isinstance(flow.events[w], tuple)):
                assert "tile" not in {flow.events[k] for k in flow.behind(w, "mfma", "barrier")}, kernel


@pytest.mark.parametrize("name", ["mha_fwd_kernel", "mha_bwd_dq_kernel", "mha_bwd_dkdv_pipe_kernel", "mha_bwd_merged_kernel"])
def test_loops_wait_at_their_barrier_only(asm, name):
    """A loop over tiles requests the next tile at its top and awaits it at the barrier that ends the round: no wait for
    vector memory (a spilled value's reload, for one) with products still to come before that barrier."""
    flows = list(kernel_flows(asm, name))
    assert len(flows) >= 24
    for kernel, flow in flows:
        for i, e in enumerate(flow.events):
            if e != "tile" or i not in flow.behind(i):
                continue
            for w in flow.behind(i, "barrier"):
                if isinstance(flow.events[w], tuple):
                    assert "mfma" not in {flow.events[k] for k in flow.behind(w, "barrier")}, kernel


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


@pytest.mark.parametrize("name", ["mha_bwd_dq_far_kernel", "mha_bwd_dkdv_pipe_far_kernel", "mha_bwd_merged_far_kernel"])
def test_kernels_of_rows_far_apart_wait_no_earlier(asm, name):
    """The two orders above in the dropout kernels whose rows are spread over the lanes: with the loop's wait at its
    barrier, and, without a mask, rows and first tile requested before anything is waited for."""
    flows = list(kernel_flows(asm, name))
    assert len(flows) == 8  # two types, 64 and 128 columns, causal or not
    for kernel, flow in flows:
        loops = [i for i, e in enumerate(flow.events) if e == "tile" and i in flow.behind(i)]
        assert loops, kernel
        for w in (w for i in loops for w in flow.behind(i, "barrier") if isinstance(flow.events[w], tuple)):
            assert "mfma" not in {flow.events[k] for k in flow.behind(w, "barrier")}, kernel
        rows = [i for i, e in enumerate(flow.events) if e == "row"]
        if not re.search(r"Li\d+ELb0E" if "_dq_" in name else r"Li64ELb0E", kernel):
            continue
        assert rows, kernel
        for w in (w for i in rows for w in flow.behind(i, "tile", "mfma", "barrier") if isinstance(flow.events[w], tuple)):
            assert "tile" not in {flow.events[k] for k in flow.behind(w, "mfma", "barrier")}, kernel


def test_split_backward_loops_load_no_argument(asm):
    """A kernel argument loaded inside a loop over tiles is awaited there, in every round, with the wave's only chain of
    work behind it: the arguments of the split backward fit the scalar registers it has."""
    seen = 0
    for m in re.finditer(r"\n(_ZN5spark20mha_bwd_split_kernelI\w+):", asm):
        body = asm[m.end():]
        body = body[:body.index("\n.Lfunc_end")]
        parts = re.split(r"\n(\.LBB[0-9_]+):", body)
        labels, blocks = ["entry"] + parts[1::2], [parts[0]] + parts[2::2]
        loops = [(labels.index(t), i) for i, b in enumerate(blocks) for t in re.findall(r"s_c?branch\w* (\.LBB[0-9_]+)", b)
                 if t in labels and labels.index(t) <= i]
        inner = [l for l in loops if not any(o != l and l[0] <= o[0] and o[1] <= l[1] for o in loops)]
        tiles = [b for a, z in inner for b in ["\n".join(blocks[a:z + 1])] if "v_mfma" in b]
        assert len(tiles) >= 2, m.group(1)  # dQ and dK/dV
        assert not any("s_load" in b or "scratch_" in b for b in tiles), m.group(1)
        seen += 1
    assert seen == 16
