"""The fused site-temperature passes against the oracle, bit for bit: grid sides around the tile and its ring, window radii
on both sides of the fused kernel's rule, pass counts around the number of passes of a launch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,lb,r_s,n_s", [
    (32, 64, (8, 8), 1, 1), (33, 65, (16, 5), 1, 6), (31, 63, (7, 9), 1, 7), (70, 131, (16, 16), 1, 13),
    (32, 64, (8, 8), 2, 3), (45, 140, (5, 16), 2, 4), (100, 10, (32, 3), 2, 7), (1, 1, (4, 4), 1, 5), (3, 200, (2, 9), 2, 2),
    (20, 20, (4, 4), 3, 2), (20, 20, (4, 4), 0, 3), (20, 20, (4, 4), 1, 0)])
def test_site_temperatures_match_oracle(H, W, lb, r_s, n_s):
    nb = (-(-H // lb[0]), -(-W // lb[1]))
    T = np.exp(np.random.default_rng(H * W).uniform(-5, 1, nb)).astype(np.float32)
    o = oracle.sst_temperatures(T, H, W, *lb, r_s, n_s)
    g = M.mpr_sst_temperatures(torch.from_numpy(T).cuda(), H, W, *lb, r_s, n_s)
    assert np.array_equal(g.cpu().numpy(), o)


def test_site_temperatures_with_infinities():
    """An infinite block temperature spreads as an infinity, and its neighbours' finite means are untouched."""
    T = np.full((3, 5), 0.25, np.float32)
    T[1, 2] = np.inf
    o = oracle.sst_temperatures(T, 48, 80, 16, 16, 1, 5)
    g = M.mpr_sst_temperatures(torch.from_numpy(T).cuda(), 48, 80, 16, 16, 1, 5)
    assert np.array_equal(g.cpu().numpy(), o)
