"""Calls of many short programs, whose programs are staged by one lane each:
scores and statuses equal, bit for bit, those of the same programs in calls too
small for that (a wavefront stages each), whatever is left to the wavefronts
among them: long and deep programs, long runs of constants, broken ones."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu
L, C = synth.LOAD, synth.CONST


def _gp():
    import paper_2607_06731_amd as gp
    return gp


def _mixed(rng, P, gcl, broken):
    """P programs, most of them short, and every kind that lanes leave."""
    lens = rng.integers(1, 9, P)
    lens[rng.random(P) < 0.02] = 63
    lens[rng.random(P) < 0.02] = 65
    lens[rng.random(P) < 0.01] = 200
    if gcl:
        pop = synth.sample_gcl_programs(rng, np.maximum(lens, 3), 3)
    else:
        pop = synth.sample_programs(rng, lens, 3, synth.UNARY_2)
    deep = [[L | ((k % 3) << 8) for k in range(d)] + [synth.SUB, synth.DIV] * ((d - 1) // 2) for d in (9, 17, 31)]
    runs = [[C] * r + [synth.ADD] * (r - 1) for r in (8, 9, 20)]
    extra = [p for p in deep + runs for _ in range(20)]
    nodes = np.concatenate([pop.nodes] + [np.array(p, np.uint32) for p in extra])
    offsets = np.concatenate([pop.offsets, pop.offsets[-1] + np.cumsum([len(p) for p in extra])])
    if broken:
        at = rng.choice(nodes.size, nodes.size // 50, replace=False)
        nodes = nodes.copy()
        nodes[at] = rng.integers(0, 40, at.size).astype(np.uint32) | (rng.integers(0, 9, at.size).astype(np.uint32) << 8)
    order = rng.permutation(offsets.size - 1)
    lens = np.diff(offsets)[order]
    nodes = np.concatenate([nodes[offsets[p]:offsets[p + 1]] for p in order])
    return nodes, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), pop.consts


def _takes_lanes(nodes, offsets):
    P = offsets.size - 1
    return P * P >= 4000 * nodes.size


@pytest.mark.parametrize("n_cases", [37, 2048])
@pytest.mark.parametrize("gcl,broken", [(False, False), (False, True), (True, False), (True, True)])
def test_scores_equal_those_of_small_calls(gcl, broken, n_cases):
    gp = _gp()
    rng = np.random.default_rng(1 + gcl + 2 * broken)
    nodes, offsets, consts = _mixed(rng, 60000, gcl, broken)
    P = offsets.size - 1
    mask = synth.MASK_GCL if gcl else synth.MASK_2
    X = rng.uniform(-2, 2, (3, n_cases)).astype(np.float32)
    y = rng.uniform(-2, 2, n_cases).astype(np.float32)
    assert _takes_lanes(nodes, offsets)
    F, st = gp.evaluate(nodes, offsets, consts, X, y, 1e-3, mask, return_status=True)
    want, _, _ = gp.gp_validate(nodes, offsets, consts.size, 3, mask)
    assert np.array_equal(st, want) and (want != 0).any() == broken
    for b in range(0, P, 4000):
        e = min(P, b + 4000)
        o = offsets[b:e + 1] - offsets[b]
        sub = nodes[offsets[b]:offsets[e]]
        assert not _takes_lanes(sub, o)
        ref, s2 = gp.evaluate(sub, o, consts, X, y, 1e-3, mask, return_status=True)
        nan = np.isnan(ref)
        assert np.array_equal(s2, st[b:e])
        assert np.array_equal(np.isnan(F[b:e]), nan)
        assert np.array_equal(F[b:e].view(np.uint64)[~nan], ref.view(np.uint64)[~nan])


@pytest.mark.parametrize("n_cases", [37, 2048])
@pytest.mark.parametrize("gcl", [False, True])
def test_offsets_that_step_back(gcl, n_cases):
    gp = _gp()
    rng = np.random.default_rng(5)
    nodes, offsets, consts = _mixed(rng, 60000, gcl, False)
    mask = synth.MASK_GCL if gcl else synth.MASK_2
    P = offsets.size - 1
    X = rng.uniform(-2, 2, (3, n_cases)).astype(np.float32)
    ref = gp.evaluate(nodes, offsets, consts, X, X[1], 0.0, mask)
    full = np.concatenate([nodes, np.zeros(400, np.uint32)])
    F, st = gp.evaluate(full, np.concatenate([offsets, offsets[:41]]), consts, X, X[1], 0.0, mask,
                        return_status=True)
    assert st[P] == 8 and (np.delete(st, P) == 0).all()
    got, want = np.delete(F, P), np.concatenate([ref, ref[:40]])
    assert np.array_equal(got.view(np.uint64), want.view(np.uint64))


def test_blocks_of_more_programs_than_a_round():
    """Over 1,024 programs per staging block: k_stage_waves looks them through in
    rounds."""
    gp = _gp()
    rng = np.random.default_rng(8)
    nodes, offsets, consts = _mixed(rng, 120000, False, True)
    k = 11
    lens = np.tile(np.diff(offsets), k)
    all_nodes, all_off = np.tile(nodes, k), np.concatenate([[0], np.cumsum(lens)])
    assert all_off.size - 1 > 1024 * 1024
    X = rng.uniform(-2, 2, (3, 37)).astype(np.float32)
    ref, s0 = gp.evaluate(nodes, offsets, consts, X, X[1], 0.0, synth.MASK_2, return_status=True)
    F, st = gp.evaluate(all_nodes, all_off, consts, X, X[1], 0.0, synth.MASK_2, return_status=True)
    assert np.array_equal(st, np.tile(s0, k))
    want = np.tile(ref, k)
    nan = np.isnan(want)
    assert np.array_equal(np.isnan(F), nan)
    assert np.array_equal(F.view(np.uint64)[~nan], want.view(np.uint64)[~nan])


def test_requests_of_one_launch():
    import torch
    gp = _gp()
    rng = np.random.default_rng(6)
    X = rng.uniform(-2, 2, (3, 300)).astype(np.float32)
    y = rng.uniform(-2, 2, 300).astype(np.float32)
    data = gp.DeviceDataset(X, y)
    reqs, refs = [], []
    for n in (30000, 1, 20000, 7):
        nodes, offsets, consts = _mixed(rng, n, False, n == 20000)
        pop = gp.DevicePopulation(nodes, offsets, consts if consts.size else np.ones(1, np.float32))
        out = torch.empty(pop.n_programs, dtype=torch.float64, device="cuda")
        st = torch.empty(pop.n_programs, dtype=torch.int32, device="cuda")
        reqs.append((pop, out, st))
        b = 3000
        refs.append([gp.evaluate(nodes[offsets[k]:offsets[min(k + b, offsets.size - 1)]],
                                 offsets[k:k + b + 1] - offsets[k], consts if consts.size else np.ones(1, np.float32),
                                 X, y, 0.0, synth.MASK_2, return_status=True) for k in range(0, offsets.size - 1, b)])
    total, nn = sum(r[0].n_programs for r in reqs), sum(r[0].nodes.numel() for r in reqs)
    assert total * total >= 4000 * nn
    gp.gp_eval_batched(gp.table_tensor([gp.request_entry(p, 0, o, s) for p, o, s in reqs]),
                       gp.table_tensor([gp.dataset_entry(data)]), total, nn, 3, 300, synth.MASK_2)
    torch.cuda.synchronize()
    for (_, out, st), ref in zip(reqs, refs):
        F, S = np.concatenate([r[0] for r in ref]), np.concatenate([r[1] for r in ref])
        assert np.array_equal(st.cpu().numpy(), S)
        nan = np.isnan(F)
        got = out.cpu().numpy()
        assert np.array_equal(np.isnan(got), nan)
        assert np.array_equal(got.view(np.uint64)[~nan], F.view(np.uint64)[~nan])
