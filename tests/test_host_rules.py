"""CPU check of host/device-shared launch rules: a small C++ program compiled against the library's own header
(no GPU needed; hipcc compiles it like any other translation unit of the library)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_08862_amd import build as BLD

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_slab_rule_is_consistent_for_every_row_count(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "slab_rule_check")
    src = os.path.join(ROOT, "tests", "host", "slab_rule_check.cpp")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-result", src, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr


def test_attention_chunk_rule_compares_times_and_avoids_second_rounds(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "chunk_rule_check")
    src = os.path.join(ROOT, "tests", "host", "chunk_rule_check.cpp")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-result", src, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr


def test_tile_rules_fit_their_grids_and_follow_few_rows(tmp_path):
    """(The rules are the library's own: the program is linked against it.)"""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "tile_rule_check")
    src = os.path.join(ROOT, "tests", "host", "tile_rule_check.cpp")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-result", src, "-L" + os.path.dirname(BLD.LIB), "-l:" + os.path.basename(BLD.LIB),
                        "-Wl,-rpath," + os.path.dirname(BLD.LIB), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr


@pytest.mark.parametrize("source, kernel, limit, kernels", [("gemm.hip", r"slab_(alt_)?kernel|glu_w\d_kernel", 320, 14), ("elementwise.hip", r"rmsnorm_(rows_)?kernel|rope_append_kernel", 200, 11),
                                                            ("qkv_rope.hip", r"qkv_many_kernel", 200, 1)])
def test_launch_rules_are_not_evaluated_in_front_of_the_loads(tmp_path, source, kernel, limit, kernels):
    """The K splits and row tiles of a step are decided once, by the embedding kernel: a GEMM or a consumer of its slabs that evaluates the rule
    itself has 280 .. 1500 instructions in front of its first operand load, one that reads the choice at most 310 (with eight waves, whose addresses of seven tiles are set up first)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    out = tmp_path / "kernels.s"
    r = subprocess.run([hipcc, *BLD.FLAGS, "--offload-device-only", "-S", os.path.join(BLD.CSRC, source), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    seen = 0
    for name, body in re.findall(r"\n(_Z\S+):\s*; @.*?\n(.*?)\n\.Lfunc_end", out.read_text(), re.S):
        if re.search(kernel, name):
            ops = [line.strip() for line in body.split("\n") if line.startswith("\t") and not line.strip().startswith((".", ";"))]
            first = next(i for i, op in enumerate(ops) if re.match(r"buffer_load_dwordx4|global_load_dwordx4|buffer_load.* lds$", op))
            assert first <= limit, (name, first)
            seen += 1
    assert seen == kernels, seen
