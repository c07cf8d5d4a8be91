"""A program beyond the node count whose words the interpreter can address is
refused by its status; its neighbours are scored."""
import numpy as np
import pytest

from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu


def test_a_program_of_too_many_nodes_is_refused():
    import torch
    import paper_2607_06731_amd as gp
    limit = (1 << 29) - 16
    nodes = torch.zeros(limit + 9, dtype=torch.int32, device="cuda").view(torch.uint32)     # LOAD 0 throughout
    offsets = torch.tensor([0, 1, limit + 2, limit + 3], dtype=torch.int64, device="cuda")
    consts = torch.ones(1, dtype=torch.float32, device="cuda")
    X = torch.rand((1, 300), device="cuda")
    y = torch.rand(300, device="cuda")
    out = torch.empty(3, dtype=torch.float64, device="cuda")
    st = torch.empty(3, dtype=torch.int32, device="cuda")
    gp.gp_eval(nodes, offsets, consts, X, y, 0.0, out, st, synth.MASK_2)
    torch.cuda.synchronize()
    assert st.tolist() == [0, 8, 0]
    F = out.cpu().numpy()
    assert np.isnan(F[1]) and F[0] == F[2] and np.isfinite(F[0])
