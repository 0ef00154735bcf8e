"""CPU check of the compiled attention kernels: register spills of the tile loop.  (hipcc cross-compiles; no GPU needed.)"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_08862_amd import build as BLD


def test_wide_attention_kernel_does_not_spill(tmp_path):
    """The eight waves of a workgroup have 256 registers each and the tile loop needs about 200: what the epilogues and the
    chunk merge derive from the thread index must not live across it (43 spilled registers cost 3 .. 6 us per launch)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    r = subprocess.run([hipcc, *BLD.FLAGS, "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(BLD.CSRC, "attention.hip"), "-o", str(tmp_path / "attention.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    spills = {}
    for name, spill in re.findall(r"Function Name: (\S+).*?VGPRs Spill: (\d+)", r.stderr, re.S):
        if "attn_wide_kernel" in name:
            spills[name] = int(spill)
    assert len(spills) == 2 and not any(spills.values()), spills
