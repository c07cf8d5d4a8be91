"""What one call of one population may hold on the device: never more than 8
bytes per node, 25 per program with the counts of two partition passes over
blocks of 128 programs (24 keys of 4 bytes each, twice, and two sums), and 9 per
(program, case tile), with the sections' alignment.  Callers budget for that,
and calls that fit the fixed workspace of gp_eval_noalloc with it have to go on
fitting."""
import numpy as np
import pytest
import torch

CASES = [(1, 1), (100, 1), (128, 1), (129, 2), (4096, 32), (1 << 20, 32)]      # cases, most tiles


def _bytes(P, N, tiles):
    blocks = -(-P // 128)
    total = 0
    for size in ((N + 1) * 8, P * 16, P, P * 4, 96 * blocks, 96 * blocks, 8 * blocks, 8 * blocks, 24, 12, 12,
                 8 * P * tiles, P * tiles, 96, 80, 4, 16, 12, 12, 24, 4 * P, 8, 4):
        total += -(-size // 256) * 256
    return total


@pytest.mark.parametrize("cases,tiles", CASES)
def test_workspace_of_one_population(cases, tiles):
    import paper_2607_06731_amd as gp
    rng = np.random.default_rng(cases)
    sizes = [1, 7, 8, 9, 127, 128, 129, 4095, 8185, 8192, 8193, 60000, 100000, 10 ** 6, 10 ** 7]
    sizes += [int(np.exp(v)) for v in rng.uniform(0, np.log(2e6), 300)]
    for P in sizes:
        for N in (P, 20 * P + 3):
            need = gp.workspace_size(P, N, 1, 1, 3, cases) * 4 // 5
            assert need <= _bytes(P, N, tiles), (P, N)


@pytest.mark.gpu
@pytest.mark.parametrize("P,cases,tiles", [(8192, 100, 1), (4000, 100, 1), (8192, 4096, 32), (300, 1000, 8)])
def test_the_fixed_workspace_takes_what_fits(P, cases, tiles):
    import paper_2607_06731_amd as gp
    from paper_2607_06731_amd import synth
    room = gp.GP_NOALLOC_WORKSPACE_BYTES
    N = (room - _bytes(P, 0, tiles)) // 8
    while _bytes(P, N, tiles) > room:
        N -= 16
    rng = np.random.default_rng(P)
    pop = synth.sample_programs(rng, rng.integers(3, 60, P), 3, synth.UNARY_2)
    X = rng.uniform(-2, 2, (3, cases)).astype(np.float32)
    y = rng.uniform(-2, 2, cases).astype(np.float32)
    want = gp.evaluate(pop.nodes, pop.offsets, pop.consts, X, y, 1e-3, synth.MASK_2)
    # nodes beyond the last program's count for the workspace only
    nodes = np.concatenate([pop.nodes, np.zeros(N - pop.nodes.size, np.uint32)])
    p, d = gp.DevicePopulation(nodes, pop.offsets, pop.consts), gp.DeviceDataset(X, y)
    out = torch.empty(P, dtype=torch.float64, device="cuda")
    gp.gp_eval_noalloc(p.nodes, p.offsets, p.consts, d.X, d.y, 1e-3, out, None, synth.MASK_2)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint64), want.view(np.uint64))
