"""The interpreter's division inside its fast range is the IEEE quotient: every
significand of the divisor (2^23 of them) under several dividends, and dense
random pairs over the range's exponents, bit for bit against NumPy's float32."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LOAD


def _quotients(a, b):
    import torch
    import paper_2607_06731_amd as gp
    X = torch.from_numpy(np.stack([a, b])).cuda()
    nodes = np.array([L, L | 256, synth.DIV], np.uint32)
    pop = gp.DevicePopulation(nodes, np.array([0, 3]), np.ones(1, np.float32))
    out = torch.empty((1, a.size), dtype=torch.float32, device="cuda")
    gp.gp_predict(pop.nodes, pop.offsets, pop.consts, X, out, allowed_op_mask=synth.MASK_2)
    return out.cpu().numpy()[0]


@pytest.mark.parametrize("dividend", [1.0, 3.0, 1.9999999, 1.3333334, 16777215.0, 0.1, -7.0])
@pytest.mark.parametrize("exponent", [-9, 0, 59])
def test_every_divisor_significand(dividend, exponent):
    bits = (np.uint32(127 + exponent) << 23) + np.arange(1 << 23, dtype=np.uint32)
    b = bits.view(np.float32)
    a = np.full(b.size, dividend, np.float32)
    assert np.array_equal(_quotients(a, b).view(np.uint32), (a / b).view(np.uint32))


@pytest.mark.parametrize("seed", range(6))
def test_dense_random_pairs(seed):
    rng = np.random.default_rng(seed)
    n = 1 << 23

    def draw(lo, hi):
        e = rng.integers(127 + lo, 127 + hi, n).astype(np.uint32)
        return ((rng.integers(0, 2, n).astype(np.uint32) << 31) | (e << 23) | rng.integers(0, 1 << 23, n).astype(np.uint32)).view(np.float32)
    a, b = draw(-60, 60), draw(-9, 60)
    assert np.array_equal(_quotients(a, b).view(np.uint32), (a / b).view(np.uint32))
