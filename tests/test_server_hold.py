"""When a ready request waits for the launches in flight (Core::hold): small
launches are shared, but nothing waits longer than 0.3 ms for one launch,
however few node evaluations it has."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def runs(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("hold") / "server_hold_harness")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "paper_2607_06731_amd", "csrc"),
                           os.path.join(ROOT, "tests", "server_hold_harness.cpp"), "-o", exe])
    out = {}
    for line in subprocess.check_output([exe], text=True, timeout=60).splitlines():
        name, *req = line.split()
        out[name] = [tuple(int(v) for v in r.split(":")) for r in req]
    return out


def test_a_long_launch_is_not_waited_for(runs):
    (first, _), (second, waited) = runs["long_launch"]
    assert second == first + 1
    assert waited <= 300


def test_small_launches_are_shared(runs):
    launches = [n for n, _ in runs["small_launches"]]
    assert launches[0] == 0 and len(set(launches[1:])) == 1
    assert max(w for _, w in runs["small_launches"]) <= 110


def test_large_requests_do_not_wait(runs):
    assert runs["large_request"][1] == (1, 0)


def test_one_launch_per_request_never_waits_for_company(runs):
    assert [n for n, _ in runs["one_each"]] == [0, 1, 2]
