"""The lattice passes' barriers, on the CPU: a workgroup of the kernels themselves, compiled as host
code (tests/workgroup_emulation), with its waves run in every order that the barriers allow a wave
to be ahead of the others in."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CLANG = next((c for c in ("/opt/rocm/lib/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)


@pytest.mark.skipif(CLANG is None, reason="needs clang++")
def test_workgroup_without_a_tile_sums_nothing_in_any_wave_order(tmp_path):
    """Its sums (zero) and the pending test that it takes do not share LDS without a barrier between."""
    exe = str(tmp_path / "empty_workgroup")
    src = os.path.join(HERE, "workgroup_emulation")
    subprocess.check_call([CLANG, "-O1", "-std=c++17", "-x", "c++", "-Wno-unknown-attributes", "-Wno-ignored-attributes",
                           "-I", src, "-I", os.path.join(ROOT, "paper_2603_24370_amd", "csrc"),
                           os.path.join(src, "empty_workgroup.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
