"""The workgroup shapes behind waves_per_wg and wg_per_cu (launch_plan.hpp),
compiled for the host: the automatic shape spelled out, as the autotuner
returns it, is launched as the automatic one."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_automatic_shape_spelled_out(tmp_path):
    exe = str(tmp_path / "launch_plan")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2603_01915_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "launch_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "0 failures" in r.stdout
