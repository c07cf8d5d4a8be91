"""Batched calls of 1 to 4,096 requests (the request tables are made by a run of
requests per thread), empty requests among them: scores equal, bit for bit,
those of the same programs and dataset in one call."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_req", [1, 2, 3, 255, 256, 257, 513, 4096])
def test_scores_of_many_requests(n_req):
    import torch
    import paper_2607_06731_amd as gp
    rng = np.random.default_rng(n_req)
    sizes = np.where(rng.random(n_req) < 0.2, 0, rng.integers(1, 9, n_req))
    sizes[rng.integers(0, n_req)] = 300
    data = []
    for n, v in ((1, 1), (200, 3), (1500, 2), (4099, 5)):
        data.append((rng.uniform(-3, 3, (v, n)).astype(np.float32), rng.uniform(-3, 3, n).astype(np.float32)))
    dev = [gp.DeviceDataset(X, y) for X, y in data]
    which = rng.integers(0, len(data), n_req)
    P = int(sizes.sum())
    pop = synth.sample_programs(rng, rng.integers(1, 100, P), 1, synth.UNARY_2)
    big = gp.DevicePopulation(pop.nodes, pop.offsets, pop.consts)
    F = torch.full((P,), -1.0, dtype=torch.float64, device="cuda")
    st = torch.full((P,), -1, dtype=torch.int32, device="cuda")
    entries, nodes, at = [], 0, 0
    keep = []
    for r in range(n_req):
        k = int(sizes[r])
        o = pop.offsets[at:at + k + 1]
        p = gp.DevicePopulation(pop.nodes[o[0]:o[-1]], o - o[0], pop.consts)
        keep.append(p)
        entries.append(gp.request_entry(p, int(which[r]), F[at:at + k], st[at:at + k]))
        nodes += int(o[-1] - o[0])
        at += k
    gp.gp_eval_batched(gp.table_tensor(entries), gp.table_tensor([gp.dataset_entry(d, 1e-3) for d in dev]), P, nodes,
                       5, 4099, synth.MASK_2)
    torch.cuda.synchronize()
    F, st = F.cpu().numpy(), st.cpu().numpy()
    assert (st == 0).all()
    of = np.repeat(which, sizes)
    for d, (X, y) in enumerate(data):
        ref = gp.evaluate(pop.nodes, pop.offsets, pop.consts, X, y, 1e-3, synth.MASK_2)
        assert np.array_equal(F[of == d].view(np.uint64), ref[of == d].view(np.uint64))
