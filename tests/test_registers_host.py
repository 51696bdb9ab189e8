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


def test_bf16_forward_spills_nothing(tmp_path):
    """The 256-row form of lists of pairs stands at 254 of 256 registers."""
    assert {k: n for k, n in _spills("dfa_fwd_bf16.hip", tmp_path).items() if n} == {}


def test_f32_sums_are_for_sequences_alone(tmp_path):
    """dk, dv as sums of 32 rows (7 % of a backward at d = 128) in kernels of their own, and no form of theirs spills."""
    spills = {k: n for k, n in _spills("dfa_attn_f32.hip", tmp_path).items() if "k_bwd_f32" in k}
    flags = {k: tuple(re.findall(r"Lb([01])E", k)) for k in spills}          # (SHARED, SUMS) of the mangled name
    assert {f[1] for f in flags.values()} == {"0", "1"}
    assert all(n == 0 for k, n in spills.items() if flags[k][1] == "1")
