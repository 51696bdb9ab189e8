"""What the compiler reports of the kernels' registers: a spill in a loop over tiles costs 5 to 20 % of a call and no other test shows it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2310_03294_amd import build as B


def _spills(source, tmp_path):
    """VGPRs spilled by each kernel of a source file."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    r = subprocess.run([hipcc, *B.HIP_FLAGS, "-w", "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-I", B.INCLUDE,
                        "-I", B.CSRC, "-c", os.path.join(B.CSRC, source), "-o", str(tmp_path / "x.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    counts = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert names and len(names) == len(counts)
    return dict(zip(names, counts))


def test_bf16_backward_spills_nothing(tmp_path):
    assert {k: n for k, n in _spills("dfa_bwd_bf16.hip", tmp_path).items() if n} == {}
