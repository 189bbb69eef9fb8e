"""Site temperatures on grids much thinner than the fused kernel's tile, on both sides of its rule, against the oracle bit for
bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


# one row of tiles: one round of them and one tile more; a quarter and three eighths full and less; columns
@pytest.mark.parametrize("H,W", [(1, 32768), (1, 32769), (8, 32832), (7, 32832), (12, 32832), (11, 32832),
                                 (33, 16448), (16385, 1), (16416, 24), (16416, 23)])
@pytest.mark.parametrize("r_s,n_s", [(1, 1), (1, 7), (2, 4)])
def test_thin_grids(H, W, r_s, n_s):
    lb = (3, 50)
    T = np.random.default_rng(H).uniform(0.0, 1.0, -(-H // lb[0]) * -(-W // lb[1])).astype(np.float32)
    g = M.mpr_sst_temperatures(torch.from_numpy(T).cuda(), H, W, *lb, r_s, n_s)
    assert np.array_equal(g.cpu().numpy(), oracle.sst_temperatures(T, H, W, *lb, r_s, n_s))
