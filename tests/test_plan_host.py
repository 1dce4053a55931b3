"""The cut of a call into launches, built on its own with the host compiler and
driven by tests/c/plan_checks.cpp.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_launch_plan_on_random_tables(tmp_path):
    exe = tmp_path / "plan_checks"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2104_05588_amd", "csrc"), "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "c", "plan_checks.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300, env=env)
    assert res.returncode == 0, res.stderr[-3000:]
    assert "plan checks ok" in res.stdout
