"""The cut of a call into work items and LDS (paper_2607_06731_amd/csrc/
run_shape.h) on the host: tests/run_shape_harness.cpp walks the items of random
calls, whatever the fitness, widths, lengths and tuning."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("shape") / "run_shape_harness")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "paper_2607_06731_amd", "csrc"),
                           os.path.join(ROOT, "tests", "run_shape_harness.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("seed", [1, 2, 3, 4])
def test_items_cover_the_work_and_fit(harness, seed):
    r = subprocess.run([harness, str(seed), "4000"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    assert int(r.stdout.split()[0]) == 4000
