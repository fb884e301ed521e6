"""The compiler's resource report of the attention kernels that hold many tile places: nothing may spill."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2401_06706_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
@pytest.mark.parametrize("source", ["tree_attn.hip", "tree_attn_shared.hip", "tree_attn_any.hip"])
def test_no_register_spills(source, tmp_path):
    flags = [f for f in B.HIPCC_FLAGS if f != "-shared"]
    res = subprocess.run([HIPCC] + flags + ["-c", "-Rpass-analysis=kernel-resource-usage", os.path.join(B.CSRC, source), "-o", str(tmp_path / "x.o")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert res.returncode == 0, res.stdout[-2000:]
    kernels = res.stdout.split("Function Name: ")[1:]
    assert kernels
    for k in kernels:
        spills = [int(n) for n in re.findall(r"[SV]GPRs Spill: (\d+)", k)]
        assert len(spills) == 2 and not any(spills), k[:2000]


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
@pytest.mark.parametrize("source,most", [("verify_sample.hip", 8), ("draft_sample.hip", 0)])
def test_vector_registers_put_aside_by_the_row_kernels(source, most, tmp_path):
    """A thread of the verification rows holds up to 32 float4 of one row and 14 of the other and fills its registers: the few that it puts
    aside stay few (a branch in the wrong place makes the compiler copy a row, 50 and more)."""
    flags = [f for f in B.HIPCC_FLAGS if f != "-shared"]
    res = subprocess.run([HIPCC] + flags + ["-c", "-Rpass-analysis=kernel-resource-usage", os.path.join(B.CSRC, source), "-o", str(tmp_path / "x.o")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert res.returncode == 0, res.stdout[-2000:]
    spills = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", res.stdout)]
    assert spills and max(spills) <= most, res.stdout[-4000:]
