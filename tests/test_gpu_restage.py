"""Calls whose offsets step back somewhere: that pair is BAD_OFFSETS, and the
programs, whose node ranges overlap, are staged apart, each in exactly the words
it needs.  Here on datasets long enough that programs are reordered, with
programs whose words in the order written are nearly twice those.  Scores and
outputs equal those of the same programs in a call without the step, bit for
bit; when the words outnumber the call's nodes, nothing is staged."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LOAD


def _gp():
    import paper_2607_06731_amd as gp
    return gp


def _combs(n, rng):
    """n programs of `depth` variables and depth - 1 operators after them."""
    ops = [synth.SUB, synth.DIV, synth.ADD, synth.MUL]
    progs = []
    for k in range(n):
        d = int(rng.integers(9, 33))
        progs.append([L | (int(v) << 8) for v in rng.integers(0, 3, d)] + [ops[int(o)] for o in rng.integers(0, 4, d - 1)])
    return progs


def _calls(n, spare):
    rng = np.random.default_rng(n)
    progs = _combs(n, rng)
    nodes = np.concatenate([np.array(p, np.uint32) for p in progs])
    o = np.concatenate([[0], np.cumsum([len(p) for p in progs])]).astype(np.int64)
    # twice the programs: twice `depth` words each, 2 depth - 1 nodes
    words = int(sum(len(p) + 1 for p in progs))
    full = np.concatenate([nodes, np.zeros(words - nodes.size + spare, np.uint32)])
    return nodes, o, full, np.concatenate([o, o])


@pytest.mark.parametrize("n_cases", [2047, 2048, 5000])
@pytest.mark.parametrize("n", [1, 40, 9000])
def test_deep_programs_are_packed_apart(n, n_cases):
    gp = _gp()
    rng = np.random.default_rng(7)
    X = rng.uniform(-2, 2, (3, n_cases)).astype(np.float32)
    y = rng.uniform(-2, 2, n_cases).astype(np.float32)
    consts = np.ones(1, np.float32)
    # in the order written (2,047 cases) as many words as nodes less one per operator
    spare = 0 if n_cases >= 2048 else 2 * int(sum(len(p) for p in _combs(n, np.random.default_rng(n))))
    nodes, o, full, offsets = _calls(n, spare)
    ref = gp.evaluate(nodes, o, consts, X, y, 0.0, synth.MASK_2)
    F, st = gp.evaluate(full, offsets, consts, X, y, 0.0, synth.MASK_2, return_status=True)
    assert st[n] == 8 and (np.delete(st, n) == 0).all()
    assert np.isnan(F[n])
    assert np.array_equal(np.delete(F, n).view(np.uint64), np.concatenate([ref, ref]).view(np.uint64))
    if n <= 40:
        a = gp.predict(nodes, o, consts, X, synth.MASK_2).view(np.uint32)
        b = gp.predict(full, offsets, consts, X, synth.MASK_2).view(np.uint32)
        assert np.array_equal(np.delete(b, n, axis=0), np.concatenate([a, a]))


@pytest.mark.parametrize("n", [1, 40, 9000])
def test_one_word_too_many(n):
    gp = _gp()
    rng = np.random.default_rng(7)
    X = rng.uniform(-2, 2, (3, 2048)).astype(np.float32)
    _, _, full, offsets = _calls(n, -1)
    F, st = gp.evaluate(full, offsets, np.ones(1, np.float32), X, X[0], 0.0, synth.MASK_2, return_status=True)
    assert (st == 8).all() and np.isnan(F).all()


def test_requests_that_step_back(n_cases=3000):
    """Two requests of one launch, one of them with the step."""
    import torch
    gp = _gp()
    rng = np.random.default_rng(9)
    X = rng.uniform(-2, 2, (3, n_cases)).astype(np.float32)
    y = rng.uniform(-2, 2, n_cases).astype(np.float32)
    consts = np.ones(1, np.float32)
    data = gp.DeviceDataset(X, y)
    nodes, o, full, offsets = _calls(300, 0)
    pops = [gp.DevicePopulation(full, offsets, consts), gp.DevicePopulation(nodes, o, consts)]
    outs = [(torch.empty(p.n_programs, dtype=torch.float64, device="cuda"),
             torch.empty(p.n_programs, dtype=torch.int32, device="cuda")) for p in pops]
    gp.gp_eval_batched(gp.table_tensor([gp.request_entry(p, 0, *q) for p, q in zip(pops, outs)]),
                       gp.table_tensor([gp.dataset_entry(data)]), sum(p.n_programs for p in pops),
                       sum(p.nodes.numel() for p in pops), 3, n_cases, synth.MASK_2)
    torch.cuda.synchronize()
    ref = gp.evaluate(nodes, o, consts, X, y, 0.0, synth.MASK_2)
    F, st = outs[0][0].cpu().numpy(), outs[0][1].cpu().numpy()
    assert st[300] == 8 and (np.delete(st, 300) == 0).all()
    assert np.array_equal(np.delete(F, 300).view(np.uint64), np.concatenate([ref, ref]).view(np.uint64))
    assert np.array_equal(outs[1][0].cpu().numpy().view(np.uint64), ref.view(np.uint64))
