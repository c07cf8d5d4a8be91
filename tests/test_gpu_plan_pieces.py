"""Plans whose window budget is no multiple of the running sums' alignment, on
datasets whose tiles are staged in pieces (running sums in LDS between them):
scores equal gp_eval's up to the rounding of a differently grouped compensated
sum, 2^-21 each."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_lds", [4096, 40 * 1024, 65536])
@pytest.mark.parametrize("n_vars,max_tiles", [(2, 1), (3, 32), (60, 2), (140, 2)])
def test_tiles_in_pieces(tile_lds, n_vars, max_tiles):
    import torch
    import paper_2607_06731_amd as gp
    rng = np.random.default_rng(tile_lds + n_vars)
    n = 40001 if max_tiles < 32 else 500003
    pop = synth.sample_programs(rng, rng.integers(3, 100, 150), n_vars, (synth.ABS,))
    X = rng.uniform(-2, 2, (n_vars, n)).astype(np.float32)
    y = rng.uniform(-2, 2, n).astype(np.float32)
    p, d = gp.DevicePopulation(pop.nodes, pop.offsets, pop.consts), gp.DeviceDataset(X, y)
    out = torch.empty(p.n_programs, dtype=torch.float64, device="cuda")
    plan = gp.Plan(p, d, 0.0, out, None, synth.MASK_2,
                   tuning={"tile_lds_bytes": tile_lds, "max_tiles": max_tiles, "programs_per_item": 13})
    plan.launch()
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    plan.close()
    ref = gp.evaluate(pop.nodes, pop.offsets, pop.consts, X, y, 0.0, synth.MASK_2)
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin) and fin.sum() > 50
    np.testing.assert_allclose(got[fin], ref[fin], rtol=2.0 ** -20)
