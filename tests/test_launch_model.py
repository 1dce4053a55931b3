"""The library's launches of calls with statistics, run against a HIP runtime and a
model of the kernels in host memory (tests/c/launch_model.cpp): every bucket's
statistics come from its own partials, whatever the table, in every scratch.  No GPU."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2104_05588_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    if not os.path.exists(B.LIB):
        B.build()
    exe = tmp_path_factory.mktemp("model") / "launch_model"
    # -rdynamic: the library's HIP calls find this program's definitions
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2104_05588_amd", "csrc"), "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "c", "launch_model.cpp"), "-o", str(exe), "-ldl"],
                   check=True, capture_output=True, text=True)
    return str(exe)


def run(model, scenario):
    res = subprocess.run([model, B.LIB, scenario], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    assert "launch model ok" in res.stdout
    return res.stdout


def test_random_tables(model):
    run(model, "random_tables")


def test_a_long_table_keeps_its_passes_and_its_scratch_bounded(model):
    run(model, "long_table")


def test_captured_calls_find_room_after_a_warm_up_of_their_size(model):
    run(model, "capture")


def test_the_fixed_array_keeps_its_size_whatever_the_call(model):
    run(model, "fixed_array")


def test_the_bench_probes_take_the_shape_that_the_library_launches(model):
    lines = [ln.split() for ln in run(model, "shapes").splitlines() if ln.startswith("shape")]
    assert len(lines) == 20
    for _, g, P, threads, lds in lines:
        assert (int(threads) // 64, int(lds)) == bench.step_split(int(g), int(P)), (g, P)


def test_short_calls_take_workgroups_of_four_and_no_cap(model):
    lines = [ln.split() for ln in run(model, "shapes").splitlines() if ln.startswith("short")]
    assert len(lines) == 10
    for _, g, P, threads, lds in lines:
        assert (int(threads), int(lds)) == (256, 0), (g, P)
