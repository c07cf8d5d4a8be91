"""gp_predict of few programs over very many cases, whose tiles are as small as a
window of the staged inputs, and beyond that: sums of
variables, bit for bit against torch's float32 additions."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LOAD


@pytest.mark.parametrize("n_programs,n_cases,n_vars", [
    (1, 1000003, 2), (7, 300001, 5), (8, 1000000, 20), (3, 65537, 60), (2, 40000, 130), (100, 65536, 5),
    (1, 2048 * 24576 + 5, 1)])
def test_sums_of_variables(n_programs, n_cases, n_vars):
    import torch
    import paper_2607_06731_amd as gp
    g = torch.Generator(device="cuda").manual_seed(n_cases)
    X = torch.rand((n_vars, n_cases), generator=g, device="cuda", dtype=torch.float32)
    out = torch.full((n_programs, n_cases), -1.0, device="cuda", dtype=torch.float32)
    progs, use = [], []
    for p in range(n_programs):
        d = (2, 9, 17)[p % 3]                    # a program of each stack class
        use.append([(p + k) % n_vars for k in range(d)])
        progs.append([L | (v << 8) for v in use[-1]] + [synth.ADD] * (d - 1))
    nodes = np.concatenate([np.array(p, np.uint32) for p in progs])
    pop = gp.DevicePopulation(nodes, np.concatenate([[0], np.cumsum([len(p) for p in progs])]), np.ones(1, np.float32))
    gp.gp_predict(pop.nodes, pop.offsets, pop.consts, X, out, allowed_op_mask=synth.MASK_2)
    for p in range(n_programs):
        f = X[use[p][-1]]
        for v in use[p][-2::-1]:
            f = X[v] + f
        assert torch.equal(out[p], f)


def test_the_output_rows_are_only_written():
    """Rows of programs and the columns beyond the cases: what the buffer held
    does not matter, and stays where nothing is written."""
    import torch
    import paper_2607_06731_amd as gp
    n, ld = 5000, 5120
    X = torch.rand((2, n), device="cuda", dtype=torch.float32)
    nodes = np.array([L, L | 256, synth.ADD, L], np.uint32)
    pop = gp.DevicePopulation(nodes, np.array([0, 3, 4]), np.ones(1, np.float32))
    for fill in (float("nan"), float("inf"), 7.0):
        buf = torch.full((2, ld), fill, device="cuda", dtype=torch.float32)
        gp.gp_predict(pop.nodes, pop.offsets, pop.consts, X, buf, allowed_op_mask=synth.MASK_2)
        assert torch.equal(buf[0, :n], X[0] + X[1]) and torch.equal(buf[1, :n], X[0])
        rest = torch.full((2, ld - n), fill, device="cuda")
        assert torch.equal(buf[:, n:].nan_to_num(1.5), rest.nan_to_num(1.5))


def test_programs_without_variables():
    import torch
    import paper_2607_06731_amd as gp
    X = torch.empty((0, 300), device="cuda", dtype=torch.float32)
    pop = gp.DevicePopulation(np.array([synth.CONST, synth.CONST | 256, synth.SUB], np.uint32), np.array([0, 3]),
                              np.array([3.5, 1.25], np.float32))
    out = torch.empty((1, 300), device="cuda", dtype=torch.float32)
    gp.gp_predict(pop.nodes, pop.offsets, pop.consts, X, out, allowed_op_mask=synth.MASK_2, n_cases=300)
    assert torch.equal(out, torch.full_like(out, 2.25))
