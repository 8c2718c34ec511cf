"""Checks of the gfx950 code of the lifting kernels beyond test_codegen.py (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2405_12631_amd import build as B


def _listing(src, tmp_path):
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("hipcc not available")
    out = str(tmp_path / (src + ".s"))
    subprocess.run([B.HIPCC, "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", out] +
                   [f for f in B.HIP_FLAGS if f != "-fPIC"], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.mark.slow
@pytest.mark.parametrize("src,kernels", [("wv_lift_rows.hip", 1), ("wv_lift_fused.hip", 3)])
def test_no_scalar_spills(src, kernels, tmp_path):
    """A spilled scalar is read back with vector instructions in the row loop, whose issue bounds these
    kernels."""
    spills = re.findall(r"\.sgpr_spill_count:\s*(\d+)", _listing(src, tmp_path))
    assert spills == ["0"] * kernels, spills


@pytest.mark.slow
def test_split_kernel_uses_global_memory_and_no_scratch(tmp_path):
    """Both strip forms of the split kernel sit at the edge of the register file (251 and 255 VGPRs)."""
    asm = _listing("wv_lift_split.hip", tmp_path)
    assert re.findall(r"; ScratchSize: (\d+)", asm) == ["0", "0"]
    assert re.findall(r"\.(?:v|s)gpr_spill_count:\s*(\d+)", asm) == ["0"] * 4
    assert asm.count("global_load") > 20 and not re.search(r"^\s*(flat|scratch)_", asm, flags=re.M)
