"""The matrix instructions that the kernels issue as assembly statements: the compiler leaves no wait states behind those,
so no accumulator may be read between a kernel's last one and the wait that the source puts there."""
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
