"""The threaded words (paper_2607_06731_amd/csrc/threaded.h) against the
flag words of the same staging walk, on the host: every instruction names
the handler of its operator and stack depth, block 0 marks the last word
only, and no depth leaves the program's class table."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2607_06731_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("threaded") / "threaded_harness")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2607_06731_amd", "csrc"),
                           "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "threaded_harness.cpp"), "-o", exe])
    return exe


def _comb(n_leaves, var):
    """n_leaves leaves, then n_leaves - 1 additions: depth n_leaves."""
    leaf = synth.LOAD if var else synth.CONST
    return [leaf] * n_leaves + [synth.ADD] * (n_leaves - 1)


@pytest.mark.parametrize("law,n_vars,p_var", [("u32", 3, 0.5), ("u64", 5, 0.5), ("u128", 20, 0.9),
                                              ("short", 1, 0.5), ("u64", 2, 0.1)])
def test_words_name_the_same_instructions(harness, tmp_path, law, n_vars, p_var):
    rng = np.random.default_rng(11)
    hi = {"u32": 32, "u64": 64, "u128": 128, "short": 4}[law]
    pop = synth.sample_programs(rng, rng.integers(1 if law == "short" else 3, hi + 1, 4000), n_vars,
                                synth.UNARY_2, p_var=p_var)
    # every depth up to the limit, over variables and over constants
    extra = [_comb(d, v) for d in range(1, 33) for v in (True, False)]
    extra += [e + [synth.SIN] for e in extra] + [e + [synth.LOAD, synth.DIV] for e in extra[:62]]
    nodes = np.concatenate([pop.nodes] + [np.array(e, np.uint32) for e in extra])
    offsets = np.concatenate([pop.offsets, pop.offsets[-1] + np.cumsum([len(e) for e in extra])])
    consts = pop.consts if pop.consts.size else np.ones(1, np.float32)
    f = str(tmp_path / "in.bin")
    with open(f, "wb") as h:
        np.array([offsets.size - 1, nodes.size, consts.size, n_vars], np.int64).tofile(h)
        nodes.astype(np.uint32).tofile(h)
        offsets.astype(np.int64).tofile(h)
        consts.astype(np.float32).tofile(h)
    valid, words, bad = map(int, subprocess.check_output([harness, f]).split())
    assert bad == -1
    assert valid == offsets.size - 1 and words > valid
