"""A batch below the lane sweep: scenes around the edges of the sweep's tile, block sizes with and without the temperature table,
check intervals around the sweeps of a launch, scenes that stop at different checks, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 70), (33, 65), (32, 64), (31, 129), (66, 3), (97, 130)]


@pytest.mark.parametrize("lb,R,kw", [
    ((16, 16), 3, dict(stop_mode=0, n_eq=7, n_samp=2)),
    ((2, 1), 1, dict(stop_mode=0, n_eq=1, n_samp=0)),
    ((16, 16), 5, dict(stop_mode=1, n_fit=20, n_f=5, n_max=200, n_samp=3)),
    ((2, 1), 2, dict(stop_mode=1, n_fit=2, n_f=7, n_max=40, n_samp=1)),
    ((5, 40), 63, dict(stop_mode=1, n_fit=6, n_f=1, n_max=9, n_samp=1))])
def test_scenes_match_oracle(lb, R, kw):
    kw = dict(n_real=R, init_mode=1, seed=21, **kw)
    scenes, host = [], []
    for i, (H, W) in enumerate(SHAPES):
        rng = np.random.default_rng(10 * i + R)
        m = (rng.random((H, W)) < 0.2 + 0.1 * i).astype(np.uint8)
        m.ravel()[0] = 1
        t = rng.random((H, W)).astype(np.float32) * m
        T = rng.uniform(0.02, 0.5, -(-H // lb[0]) * -(-W // lb[1])).astype(np.float32)
        host.append((t, m, T))
        t, m, T = (torch.from_numpy(a).cuda() for a in (t, m, T))
        scenes.append(dict(t=t, mask=m, T_blocks=T, block=lb, scene_id=30 + i))
    b = M.mpr_simulate_batched(scenes, M.SimConfig(**kw), want_energy=True)
    for i, (g, a) in enumerate(zip(b.outputs, host)):
        o = oracle.simulate(*a, *lb, OCfg(scene=30 + i, **kw))
        assert g.sweeps == o.k_star
        assert np.array_equal(g.state.cpu().numpy(), o.state)
        assert np.array_equal(g.acc.cpu().numpy(), o.acc)
        assert np.allclose(g.energy.cpu().numpy(), o.energy[:o.k_star + 1], rtol=0, atol=1e-5)
