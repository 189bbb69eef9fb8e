"""Block energies in each form of the kernel (eight realizations a wave, one a wave, a workgroup per realization, from the gaps
of narrow blocks) and on both sides of the rules between them, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


# columns: height and width around the rule, a grid too narrow for it; wide rows; few and many waves; R with a remainder
@pytest.mark.parametrize("H,W,R,lb", [
    (130, 17, 3, (128, 1)), (130, 17, 3, (127, 1)), (260, 16, 2, (256, 2)), (260, 16, 2, (255, 2)), (260, 15, 2, (256, 2)),
    (300, 21, 2, (300, 1)), (300, 1, 2, (300, 1)), (127, 40, 2, (500, 1)), (128, 40, 2, (500, 1)), (2, 5000, 3, (1, 5000)),
    (5, 3000, 9, (5, 3000)), (64, 64, 33, (8, 8)), (200, 200, 77, (4, 4)), (60, 70, 5, (16, 16)), (60, 70, 5, (16, 17)), (100, 100, 12, (3, 3)),
    (80, 90, 4, (31, 33)), (80, 90, 4, (32, 32)), (512, 260, 400, (16, 32)), (200, 200, 61, (5, 3)), (1, 1, 1, (1, 1))])
def test_block_energy(H, W, R, lb):
    rng = np.random.default_rng(H + W + R)
    m = (rng.random((H, W)) < 0.4).astype(np.uint8)
    st = rng.random((R, H, W)).astype(np.float32)
    st = np.where(m > 0, st[0], st).astype(np.float32)
    o = np.stack([oracle.block_energy(s, m, *lb) for s in st])
    g = M.mpr_block_energy(torch.from_numpy(st).cuda(), torch.from_numpy(m).cuda(), *lb).cpu().numpy()
    # sums of bond energies of at most one: any order, and a cosine's last bits
    n = 4 * min(lb[0], H) * min(lb[1], W)
    assert np.abs(g - o).max() <= n * n * 2.0 ** -53 + n * 2.0 ** -50
