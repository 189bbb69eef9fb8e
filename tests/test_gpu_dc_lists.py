"""The double checkerboard's update lists against the oracle, bit for bit: pairs inside a block, over two blocks and over the
grid's edge, grids around the list builder's workgroup, realizations with and without a remainder of a thread's share."""
import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,lb,R,p", [
    (1, 1, (2, 2), 1, 1.0), (1, 7, (1, 1), 2, 0.7), (9, 5, (3, 1), 3, 0.6), (33, 31, (5, 3), 2, 0.5), (64, 64, (16, 16), 4, 0.5),
    (40, 103, (7, 10), 3, 0.9), (130, 66, (33, 64), 2, 0.2), (600, 500, (16, 24), 17, 0.5)])
def test_chain_matches_oracle(H, W, lb, R, p):
    rng = np.random.default_rng(H * W)
    m = (rng.random((H, W)) >= p).astype(np.uint8)
    t = rng.random((H, W)).astype(np.float32) * m
    T = rng.uniform(0.02, 0.5, -(-H // lb[0]) * -(-W // lb[1])).astype(np.float32)
    T[::5] = 0.0
    kw = dict(n_real=R, init_mode=0, stop_mode=0, n_eq=3, n_samp=2, seed=8)
    o = oracle.simulate(t, m, T, *lb, OCfg(scene=4, order=1, **kw))
    g = M.mpr_simulate(*(torch.from_numpy(a).cuda() for a in (t, m, T)), *lb, M.SimConfig(scene_id=4, order=M.ORDER_DC, **kw))
    assert np.array_equal(g.state.cpu().numpy(), o.state)
    assert np.array_equal(g.acc.cpu().numpy(), o.acc)
    assert np.allclose(g.energy.cpu().numpy(), o.energy, rtol=0, atol=1e-5)
