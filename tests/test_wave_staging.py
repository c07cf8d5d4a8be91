"""The staging that the library runs (paper_2607_06731_amd/csrc/stage_waves.h:
one wavefront per program, constant folding, Sethi-Ullman order) on the host:
tests/wave_harness.cpp gives it 64 lanes, runs the words it makes and compares
them bit for bit with a plain stack machine over the nodes.  Statuses are the
oracle's, outputs of correctly rounded commands the oracle's fp32 bits; no
program stores a word outside its range, neither in the order written nor
packed to exactly the words it needs (as after offsets that decrease).  Built
twice: optimized, and under AddressSanitizer + UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from oracle import ABS, ADD, CUBE, DIV, MUL, SIGN, SQUARE, SUB
from paper_2607_06731_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
L, C = synth.LOAD, synth.CONST
REORDERED = 2048            # cases from which programs are reordered


@pytest.fixture(scope="module", params=[False, True], ids=["O1", "asan-ubsan"])
def harness(request, tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("wave") / "wave_harness")
    san = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-g"] if request.param else []
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__"] + san +
                          ["-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2607_06731_amd", "csrc"),
                           "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "wave_harness.cpp"), "-o", exe])
    return exe, request.param


def _run(exe, tmp, nodes, offsets, consts, X, data_cases, mask, seed=1):
    nodes = np.ascontiguousarray(nodes, np.uint32)
    offsets = np.ascontiguousarray(offsets, np.int64)
    consts = np.ascontiguousarray(consts, np.float32)
    X = np.ascontiguousarray(X, np.float32)
    P = offsets.size - 1
    ext = int((mask & ~oracle.MASK_BENCH) != 0)
    fin, fout = str(tmp / "in.bin"), str(tmp / "out.bin")
    with open(fin, "wb") as f:
        np.array([P, nodes.size, consts.size, X.shape[0], X.shape[1], data_cases, ext, mask, seed],
                 np.int64).tofile(f)
        nodes.tofile(f)
        offsets.tofile(f)
        consts.tofile(f)
        X.tofile(f)
    r = subprocess.run([exe, fin, fout], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    raw = np.fromfile(fout, np.uint8)
    info = raw[:P * 72].view(np.int64).reshape(P, 9)
    return info, raw[P * 72:].view(np.float32).reshape(P, X.shape[1])


def _check(info, nodes, offsets, n_consts, n_vars, mask, data_cases):
    st, md = oracle.validate(nodes, offsets, n_consts, n_vars, mask)
    assert np.array_equal(info[:, 0], st)
    ok = st == 0
    assert info[ok, 4].all(), "words outside the program's range"
    assert info[ok, 5].all(), "a word without a handler"
    assert not info[ok, 6].any(), "values"
    assert info[ok, 7].all(), "packed words"
    assert (info[np.diff(offsets) > 0, 8] != 0).all(), "staged by one lane"
    cls = np.where(md <= 8, 0, np.where(md <= 16, 1, 2))
    if data_cases < REORDERED:
        assert np.array_equal(info[ok, 1], cls[ok]) and not info[ok, 3].any()
    else:
        # the summation unit of a program with more than 16 cells stays
        assert np.array_equal(info[ok, 1] == 2, cls[ok] == 2)
        assert (info[ok, 1] <= cls[ok]).all()
    return ok


def _pack(progs):
    nodes = np.concatenate([np.array(p, np.uint32) for p in progs])
    at = np.nonzero(nodes == C)[0]
    nodes[at] |= np.arange(at.size, dtype=np.uint32) << 8
    consts = np.random.default_rng(1).uniform(-2, 2, max(1, at.size)).astype(np.float32)
    return nodes, np.concatenate([[0], np.cumsum([len(p) for p in progs])]).astype(np.int64), consts


def _right_leaning(depth, ops, tail=()):
    """depth variables, then depth - 1 operators: a cell each in the order
    written, two in Sethi-Ullman order, where every leaf joins its operator."""
    return [L | ((k % 3) << 8) for k in range(depth)] + [ops[k % len(ops)] for k in range(depth - 1)] + list(tail)


@pytest.mark.parametrize("data_cases", [REORDERED - 1, REORDERED])
def test_right_leaning_programs(harness, tmp_path, data_cases):
    """The words of the order written outnumber those of the reordered program
    by nearly two to one: none of them lies outside the packed range."""
    exe, san = harness
    progs = []
    for ops in ([SUB], [DIV, ADD, SUB]) if san else ([ADD], [SUB], [DIV], [MUL], [SUB, DIV], [DIV, ADD, SUB], [SUB, MUL]):
        for d in (9, 17, 32) if san else (1, 2, 8, 9, 10, 16, 17, 31, 32):
            progs.append(_right_leaning(d, ops))
            progs.append(_right_leaning(d, ops, [synth.SIN, synth.ABS]))
            progs.append(_right_leaning(d, ops, [C, SUB]))
            progs.append([C, L] + _right_leaning(d - 2, ops) + [DIV, SUB] if d > 3 else [L])
    # constants and functions of leaves among them
    for d in (9, 17, 30):
        progs.append(sum([[L, synth.SIN] if k % 3 else [L | 256] for k in range(d)], []) + [SUB, DIV] * 15)
        progs[-1] = progs[-1][:len(progs[-1]) - 30 + d - 1]
        progs.append([C if k % 2 else L for k in range(d)] + ([DIV, SUB] * 15)[:d - 1])
    nodes, offsets, consts = _pack(progs)
    X = np.random.default_rng(2).uniform(-2, 2, (3, 7)).astype(np.float32)
    info, out = _run(exe, tmp_path, nodes, offsets, consts, X, data_cases, oracle.MASK_BENCH)
    ok = _check(info, nodes, offsets, consts.size, 3, oracle.MASK_BENCH, data_cases)
    assert ok.all()
    if data_cases >= REORDERED:
        assert (info[:, 2] * 2 <= np.diff(offsets) + 2).sum() > (6 if san else 50)    # about half the words are left


@pytest.mark.parametrize("data_cases", [REORDERED - 1, REORDERED])
@pytest.mark.parametrize("law,p_var", [("short", 0.5), ("u64", 0.5), ("u128", 0.9), ("u128", 0.1), ("long", 0.5)])
def test_programs_of_every_length(harness, tmp_path, law, p_var, data_cases):
    exe, san = harness
    rng = np.random.default_rng(len(law))
    lo, hi, n = {"short": (1, 5, 200), "u64": (3, 64, 200), "u128": (65, 130, 100), "long": (120, 260, 40)}[law]
    pop = synth.sample_programs(rng, rng.integers(lo, hi + 1, n // 5 if san else n), 4, (ABS,),
                                binary=(ADD, SUB, MUL, DIV), p_var=p_var)
    X = rng.uniform(-3, 3, (4, 9)).astype(np.float32)
    consts = pop.consts if pop.consts.size else np.ones(1, np.float32)
    info, out = _run(exe, tmp_path, pop.nodes, pop.offsets, consts, X, data_cases, oracle.MASK_BENCH)
    assert _check(info, pop.nodes, pop.offsets, consts.size, 4, oracle.MASK_BENCH, data_cases).all()
    for p in range(0, pop.n_programs, 3):
        want = oracle.program_outputs(pop.nodes[pop.offsets[p]:pop.offsets[p + 1]], consts, X,
                                      allowed_mask=oracle.MASK_BENCH, mode=oracle.M32E).astype(np.float32)
        assert np.array_equal(out[p].view(np.uint32)[~np.isnan(want)], want.view(np.uint32)[~np.isnan(want)])
        assert np.array_equal(np.isnan(out[p]), np.isnan(want))


@pytest.mark.parametrize("data_cases", [REORDERED - 1, REORDERED])
def test_the_whole_command_table(harness, tmp_path, data_cases):
    exe, san = harness
    rng = np.random.default_rng(5)
    pop = synth.sample_gcl_programs(rng, rng.integers(3, 150, 20 if san else 120), 4)
    # and programs of the table that move nothing, so that they are reordered
    flat = synth.sample_gcl_programs(rng, rng.integers(3, 129, 40 if san else 200), 4,
                                     unary=(ABS, SQUARE, SIGN, CUBE, synth.SIN, synth.TANH), p_pow=0.2)
    moves = np.isin(flat.nodes & 0xFF, (synth.DUP, synth.SWAP, synth.DEL, synth.COPY, synth.PASTE))
    keep = [p for p in range(flat.n_programs) if not moves[flat.offsets[p]:flat.offsets[p + 1]].any()]
    X = rng.uniform(-2, 2, (4, 5)).astype(np.float32)
    for q in (pop, flat.take(np.array(keep)) if keep else pop):
        info, _ = _run(exe, tmp_path, q.nodes, q.offsets, q.consts, X, data_cases, oracle.MASK_GCL)
        assert _check(info, q.nodes, q.offsets, q.consts.size, 4, oracle.MASK_GCL, data_cases).all()


def test_right_leaning_programs_with_powers(harness, tmp_path):
    """POW takes its operands in the order written, the operators around it do
    not."""
    exe, _ = harness
    progs = []
    for d in (9, 12, 17, 31):
        for ops in ([synth.POW, SUB], [SUB, SUB, synth.POW], [DIV, synth.POW, ADD, SUB]):
            progs.append(_right_leaning(d, ops, [SQUARE]))
            progs.append([C] + _right_leaning(d, ops) + [synth.POW])
    nodes, offsets, consts = _pack(progs)
    X = np.random.default_rng(2).uniform(0.2, 2, (3, 7)).astype(np.float32)
    info, _ = _run(exe, tmp_path, nodes, offsets, consts, X, REORDERED, oracle.MASK_GCL)
    assert _check(info, nodes, offsets, consts.size, 3, oracle.MASK_GCL, REORDERED).all()


def test_long_runs_of_constants(harness, tmp_path):
    """Runs of up to 31 held constants across the 64-node chunks."""
    exe, san = harness
    progs = []
    for run in (17, 31) if san else (15, 16, 17, 31):
        for pad in (1, 62, 90) if san else (0, 1, 40, 62, 63, 64, 90):
            progs.append([C] * run + [synth.SIN] * pad + [ADD, SUB] * 15)
            progs[-1] = progs[-1][:run + pad + run - 1]
            progs.append([C] * (run - 1) + [synth.COS] * pad + [L] + [MUL] * (run - 1))
    nodes, offsets, consts = _pack(progs)
    X = np.random.default_rng(2).uniform(-2, 2, (1, 3)).astype(np.float32)
    for data_cases in (1, REORDERED):
        info, _ = _run(exe, tmp_path, nodes, offsets, consts, X, data_cases, oracle.MASK_BENCH)
        assert _check(info, nodes, offsets, consts.size, 1, oracle.MASK_BENCH, data_cases).all()


def test_broken_programs(harness, tmp_path):
    exe, san = harness
    rng = np.random.default_rng(8)
    n = 80 if san else 400
    for mask, w in ((oracle.MASK_BENCH, synth.sample_programs(rng, rng.integers(1, 150, n), 4, synth.UNARY_2)),
                    (oracle.MASK_GCL, synth.sample_gcl_programs(rng, rng.integers(3, 150, n), 4))):
        nodes = w.nodes.copy()
        at = rng.choice(nodes.size, n // 2, replace=False)
        half = at.size // 2
        nodes[at[:half]] = (nodes[at[:half]] & ~np.uint32(0xFF)) | rng.integers(0, 40, half).astype(np.uint32)
        nodes[at[half:]] = (nodes[at[half:]] & 0xFF) | (rng.integers(0, 1 << 24, at.size - half).astype(np.uint32) << 8)
        X = rng.uniform(-2, 2, (4, 2)).astype(np.float32)
        info, _ = _run(exe, tmp_path, nodes, w.offsets, w.consts, X, REORDERED, mask)
        ok = _check(info, nodes, w.offsets, w.consts.size, 4, mask, REORDERED)
        assert (~ok).sum() > n // 8
