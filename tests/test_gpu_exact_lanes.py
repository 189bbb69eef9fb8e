"""The exact decisions that several lanes of a wave make together: temperatures so low that most downhill proposals need one, T = 0,
ordinary ones, on both sweep kernels and for the directional coupling, on grids with fewer active lanes than a decision takes and
on larger ones, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


def _scene(H, W, seed):
    rng = np.random.default_rng(seed)
    m = (rng.random((H, W)) < 0.4).astype(np.uint8)
    return rng.random((H, W)).astype(np.float32) * m, m


@pytest.mark.parametrize("T", [0.0, 1e-7, 3e-6, 2e-5, 3e-4, 0.1])
@pytest.mark.parametrize("kernel,R", [(M.SWEEP_TILES, 3), (M.SWEEP_LANES, 5), (M.SWEEP_LANES, 64)])
@pytest.mark.parametrize("H,W", [(1, 1), (2, 5), (37, 70)])
def test_cold_chains_match_oracle(kernel, R, T, H, W):
    t, m = _scene(H, W, 7 * H + W)
    T = np.full(-(-H // 16) * -(-W // 16), T, np.float32)
    kw = dict(n_real=R, init_mode=0, stop_mode=0, n_eq=4, n_samp=1, seed=12)
    o = oracle.simulate(t, m, T, 16, 16, OCfg(scene=2, **kw))
    g = M.mpr_simulate(*(torch.from_numpy(a).cuda() for a in (t, m, T)), 16, 16, M.SimConfig(sweep_kernel=kernel, scene_id=2, **kw))
    assert np.array_equal(g.state.cpu().numpy(), o.state)


@pytest.mark.parametrize("T", [0.0, 1e-3, 5e-3])
@pytest.mark.parametrize("R", [5, 64])
def test_cold_directional_chains_match_oracle(R, T):
    t, m = _scene(37, 70, 3)
    T = np.full(2 * 3 * 5, T, np.float32)
    kw = dict(n_real=R, init_mode=0, stop_mode=0, n_eq=4, n_samp=1, seed=12)
    o = oracle.simulate(t, m, T, 16, 16, OCfg(scene=2, directional=1, **kw))
    g = M.mpr_simulate(*(torch.from_numpy(a).cuda() for a in (t, m, T)), 16, 16,
                       M.SimConfig(coupling=M.COUPLING_DIRECTIONAL, scene_id=2, **kw))
    assert np.array_equal(g.state.cpu().numpy(), o.state)
