"""The matrix instructions that the kernels issue as assembly statements: the compiler leaves no wait states behind those,
so no accumulator may be read between a kernel's last one and the wait that the source puts there, and none of these
kernels may spill registers."""
import os
import re
import subprocess

import pytest

from paper_2505_13345_amd import build


def _kernels(source, tmp_path, tag):
    out = os.path.join(tmp_path, source + ".s")
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "-w", "-S", "--cuda-device-only", os.path.join(build.CSRC, source),
                    "-o", out], check=True, capture_output=True)
    kernels, name = {}, None
    for line in open(out):
        label = re.match(r"(_Z\w+):", line)
        if label:
            name = label.group(1)
            kernels[name] = []
        elif name and line.strip():
            kernels[name].append(line.strip())
    return {n: lines for n, lines in kernels.items() if tag in n and any(l.startswith("v_mfma") for l in lines)}


@pytest.mark.parametrize("source,tag", [("ffn.hip", "t256"), ("wgrad.hip", "wgd")])
def test_accumulators_are_read_behind_the_wait_states(source, tag, tmp_path):
    kernels = _kernels(source, str(tmp_path), tag)
    assert kernels
    for name, lines in kernels.items():
        waits = [i for i in range(len(lines) - 1) if lines[i] == lines[i + 1] == "s_nop 15"]
        assert waits, name
        for i in waits:
            last = max(j for j in range(i) if lines[j].startswith("v_mfma"))
            early = [l for l in lines[last + 1:i] if not l.startswith(";") and re.search(r"\ba(\d|\[)", l)]
            assert not early, (name, early[:3])


@pytest.mark.parametrize("source,tag,changes", [
    ("coact.hip", "coact_lds", ["write add", "add read", "read write"]),   # one buffer: cleared, counted, read, cleared
    ("wgrad.hip", "wgd", ["write read"]),   # two halves in turn: written, read
    ("wgrad.hip", "wgs", ["write read"])])
def test_lds_accesses_of_a_wave_are_held_in_order(source, tag, changes, tmp_path):
    """Where lanes read LDS that other lanes of their wave wrote, a barrier of the block or of the wave (which emits no
    instruction, only its mark) stands between."""
    kernels = _kernels(source, str(tmp_path), tag)
    assert kernels
    for name, lines in kernels.items():
        last, held, seen = None, True, set()
        for l in lines:
            if l.startswith(("; wave barrier", "s_barrier")):
                held = True
            access = re.match(r"ds_(write|add|read)", l)
            if access:
                change = f"{last} {access.group(1)}"
                if change in changes:
                    assert held, (name, l)
                    seen.add(change)
                last, held = access.group(1), False
        assert seen == set(changes), (name, seen)


@pytest.mark.parametrize("tag", ["t256", "t128", "wgd"])
def test_build_refuses_kernels_that_spill(tag, tmp_path, monkeypatch):
    """A kernel of that name whose registers do not suffice does not build."""
    (tmp_path / "spills.hip").write_text("""
        #include <hip/hip_runtime.h>
        namespace %s {
        __global__ __launch_bounds__(1024) void kernel(const float* in, float* out, int n) {
          float v[300];
          for (int i = 0; i < 300; ++i) v[i] = in[i * n];
          for (int r = 0; r < n; ++r)
            for (int i = 0; i < 300; ++i) v[i] += v[(i + r) %% 300];
          for (int i = 0; i < 300; ++i) out[i * n] = v[i];
        }
        }""" % tag)
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path))
    with pytest.raises(RuntimeError, match="scratch"):
        build._compile("spills.hip")
