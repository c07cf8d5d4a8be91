"""Programs that need more than 8 stack cells are staged in another order on
datasets of 2,048 cases and more: their outputs there are, bit for bit, those of
the same programs over the same cases in calls too short for that, and for
correctly rounded operators the oracle's float32 values."""
import numpy as np
import pytest

import oracle
from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu
L, C = synth.LOAD, synth.CONST
N = 2048


def _gp():
    import paper_2607_06731_amd as gp
    return gp


def _forms():
    """Right-leaning programs around every reversed form: - and / of two cells, of
    a constant and of a variable with the top as the left operand."""
    progs = []
    for op in (synth.ADD, synth.SUB, synth.MUL, synth.DIV):
        for d in (9, 10, 16, 17, 18, 31):
            leaves = [L | ((k % 3) << 8) for k in range(d)]
            tail = [op] * (d - 1)
            progs.append(leaves + tail)                                   # a variable op the rest
            progs.append([C] + leaves + tail + [op])                      # a constant op the rest
            progs.append([L | 256, synth.SIN, L, synth.SUB] + leaves[:d - 2] + [op] * (d - 3) + [op])    # cells op cells
            progs.append(sum([[v, synth.ABS] for v in leaves], []) + tail)
            progs.append(leaves + [synth.SUB, op] * ((d - 1) // 2) + [op] * ((d - 1) % 2))
    nodes = np.concatenate([np.array(p, np.uint32) for p in progs])
    at = np.nonzero(nodes == C)[0]
    nodes[at] |= np.arange(at.size, dtype=np.uint32) << 8
    consts = np.random.default_rng(0).uniform(-2, 2, at.size).astype(np.float32)
    return nodes, np.concatenate([[0], np.cumsum([len(p) for p in progs])]).astype(np.int64), consts


def _same(a, b):
    nan = np.isnan(b)
    return np.array_equal(np.isnan(a), nan) and np.array_equal(a.view(np.uint32)[~nan], b.view(np.uint32)[~nan])


def _below_and_from(gp, nodes, offsets, consts, X, mask):
    whole = gp.predict(nodes, offsets, consts, X, mask)
    head = gp.predict(nodes, offsets, consts, X[:, :N - 1], mask)
    tail = gp.predict(nodes, offsets, consts, X[:, N - 1:], mask)
    assert _same(whole, np.concatenate([head, tail], axis=1))
    return whole


def test_every_reversed_form():
    gp = _gp()
    nodes, offsets, consts = _forms()
    X = np.random.default_rng(1).uniform(-2, 2, (3, N)).astype(np.float32)
    out = _below_and_from(gp, nodes, offsets, consts, X, synth.MASK_2)
    sines = np.add.reduceat((nodes & 0xFF) == synth.SIN, offsets[:-1]) > 0
    for p in np.nonzero(~sines)[0]:
        want = oracle.program_outputs(nodes[offsets[p]:offsets[p + 1]], consts, X[:, ::16].copy(),
                                      allowed_mask=oracle.MASK_BENCH, mode=oracle.M32E).astype(np.float32)
        assert _same(out[p, ::16], want), p


@pytest.mark.parametrize("law", ["u64", "u128", "geom"])
@pytest.mark.parametrize("values", ["ordinary", "edges"])
def test_sampled_programs(law, values):
    gp = _gp()
    rng = np.random.default_rng(len(law) + len(values))
    lens = {"u64": rng.integers(3, 65, 3000), "u128": rng.integers(60, 131, 1500),
            "geom": np.clip(rng.geometric(1 / 24, 3000), 3, 128)}[law]
    pop = synth.sample_programs(rng, lens, 4, synth.UNARY_2, p_var=0.8)
    X = rng.normal(0, 2, (4, N)).astype(np.float32)
    if values == "edges":
        odd = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-45, 3e38, -3e38, 1e-3, 2.0 ** 17, 88.0, -104.0], np.float32)
        at = rng.random(X.shape) < 0.2
        X[at] = rng.choice(odd, at.sum())
    _below_and_from(gp, pop.nodes, pop.offsets, pop.consts, X, synth.MASK_2)


def test_the_whole_command_table():
    gp = _gp()
    rng = np.random.default_rng(3)
    pop = synth.sample_gcl_programs(rng, rng.integers(3, 130, 2000), 4, p_pow=0.1)
    X = rng.uniform(-2, 2, (4, N)).astype(np.float32)
    _below_and_from(gp, pop.nodes, pop.offsets, pop.consts, X, synth.MASK_GCL)


def test_scores_of_deep_programs():
    """Programs of every class by the order written, scored below and from the
    limit: the sums' grouping is the class's, so a score over the same cases (the
    rest without weight) stays within the order of two float32 sums."""
    gp = _gp()
    nodes, offsets, consts = _forms()
    rng = np.random.default_rng(5)
    X = rng.uniform(-2, 2, (3, N)).astype(np.float32)
    y = rng.uniform(-2, 2, N).astype(np.float32)
    out = gp.predict(nodes, offsets, consts, X, synth.MASK_2).astype(np.float64)
    want = ((out - y) ** 2).mean(axis=1)
    F = gp.evaluate(nodes, offsets, consts, X, y, 0.0, synth.MASK_2)
    fin = np.isfinite(want) & (want < 1e30)
    assert fin.sum() > 0.8 * want.size
    np.testing.assert_allclose(F[fin], want[fin], rtol=2.0 ** -21)
