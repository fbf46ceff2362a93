"""The order of loads that the tiled kernel's counted waits rely on, read from
the assembly that the compiler makes of its translation units (CPU only).

`s_waitcnt vmcnt(N)` before a barrier leaves the N newest vector-memory loads
in flight, so a load to LDS is in place behind it only if N younger loads
follow it.  Two waits have N > 0: that of the main loop's stages in the
fidelity kernels (the N youngest are the dense head's loads to registers) and
the one before the first stage (they are stage 1's loads to LDS).  Each must
have a scheduling barrier between the loads that have to be in place and the
youngest N, so that no pass of the compiler can move one past the other, and
the youngest N must be there.
"""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2608_02703_amd import build


def _assembly(name, tmp_path):
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = str(tmp_path / (name + ".s"))
    subprocess.run([hipcc, *build.HIP_FLAGS, f"-I{build.INCLUDE}", "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, name), "-o", out],
                   check=True, capture_output=True, text=True)
    with open(out) as f:
        return f.read().split("\n")


def _waits(lines):
    """Per kernel the counted waits before barriers: (N, what lies between the
    last scheduling barrier and it, as 'L' loads to LDS and 'r' other vector
    loads; None without such a barrier since the wait before)."""
    kernels, name, since, wait = {}, None, None, None
    for line in lines:
        s = line.strip()
        m = re.match(r"(_Z\w+):", line)
        if m:
            name, since, wait = m.group(1), None, None
            kernels[name] = []
        elif name is None:
            continue
        elif s.startswith("; sched_barrier mask(0x00000000)"):
            since = ""
        elif re.match(r"(buffer|global|flat)_load", s):
            if since is not None:
                since += "L" if re.search(r"\blds\b", s) else "r"
        elif re.match(r"s_waitcnt vmcnt\(\d+\) lgkmcnt\(0\)$", s):
            wait = int(re.search(r"\d+", s).group())
        elif s == "s_barrier":
            if wait is not None:
                kernels[name].append((wait, since))
                since = None
            wait = None
        elif s and not s.startswith(";"):
            wait = None
    return {k: v for k, v in kernels.items() if "6k_mfma" in k}


@pytest.mark.parametrize("tu,fidelity", [("k_fid_mfma.hip", 2), ("k_mfma.hip", 0)])
def test_loads_that_a_counted_wait_passes_are_the_youngest(tu, fidelity, tmp_path):
    kernels = _waits(_assembly(tu, tmp_path))
    assert kernels
    in_loop = 0
    for name, waits in kernels.items():
        counted = [w for w in waits if w[0] > 0]
        assert counted, f"{name}: no counted wait"
        first, rest = counted[0], counted[1:]
        assert first[1] is not None and first[1].count("L") >= first[0], f"{name}: {first}"
        for n, since in rest:
            assert since is not None, f"{name}: vmcnt({n}) without a scheduling barrier before its loads"
            assert "L" not in since and since.count("r") >= n, f"{name}: vmcnt({n}) after '{since}'"
        in_loop += bool(rest)
    assert in_loop == fidelity
