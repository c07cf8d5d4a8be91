"""gp_timing_read's phases: each depth class's evaluation in its own, and a timed
call's scores are the untimed call's."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LOAD


@pytest.mark.parametrize("depth,phase", [(3, "eval_d8"), (12, "eval_d16"), (24, "eval_d32")])
def test_every_depth_class_has_its_phase(depth, phase):
    import torch
    import paper_2607_06731_amd as gp
    rng = np.random.default_rng(depth)
    P, n = 20000, 2000
    prog = [L | ((k % 3) << 8) for k in range(depth)] + [synth.ADD] * (depth - 1) + [synth.SIN] * 30
    nodes = np.tile(np.array(prog, np.uint32), P)
    X = rng.uniform(-2, 2, (3, n)).astype(np.float32)
    y = rng.uniform(-2, 2, n).astype(np.float32)
    pop = gp.DevicePopulation(nodes, np.arange(P + 1) * len(prog), np.ones(1, np.float32))
    data = gp.DeviceDataset(X, y)
    out = torch.empty(P, dtype=torch.float64, device="cuda")

    def step():
        gp.gp_eval(pop.nodes, pop.offsets, pop.consts, data.X, data.y, 0.0, out, None, synth.MASK_2)

    step()
    plain = out.clone()
    gp.timing_reset()
    gp.timing_enable(True)
    for _ in range(3):
        step()
    torch.cuda.synchronize()
    gp.timing_enable(False)
    ms, calls = gp.timing_read()
    gp.timing_reset()
    assert calls == 3
    evals = {k: ms[k] for k in ("eval_d8", "eval_d16", "eval_d32")}
    assert max(evals, key=evals.get) == phase
    assert evals[phase] > 0.8 * sum(evals.values()), evals
    assert torch.equal(out, plain)


def test_the_phases_add_up_over_mixed_depths():
    import torch
    import paper_2607_06731_amd as gp
    w = synth.make_workload("generation", n_programs=20000, n_cases=1000)
    pop = gp.DevicePopulation(w.pop.nodes, w.pop.offsets, w.pop.consts)
    data = gp.DeviceDataset(w.data.X, w.data.y)
    want = gp.evaluate(w.pop.nodes, w.pop.offsets, w.pop.consts, w.data.X, w.data.y, w.tax, w.allowed_mask)
    out = torch.empty(pop.n_programs, dtype=torch.float64, device="cuda")
    gp.timing_reset()
    gp.timing_enable(True)
    for _ in range(4):
        gp.gp_eval(pop.nodes, pop.offsets, pop.consts, data.X, data.y, w.tax, out, None, w.allowed_mask)
    torch.cuda.synchronize()
    gp.timing_enable(False)
    ms, calls = gp.timing_read()
    gp.timing_reset()
    assert calls == 4 and all(v > 0 for v in ms.values())
    parts = sum(v for k, v in ms.items() if k != "total")
    assert abs(parts - ms["total"]) < 0.05 * ms["total"]
    nan = np.isnan(want)
    assert np.array_equal(out.cpu().numpy().view(np.uint64)[~nan], want.view(np.uint64)[~nan])
