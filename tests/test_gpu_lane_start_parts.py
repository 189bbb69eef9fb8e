"""The energy of a start on the lane layouts at grid sizes around its parts (32 sites each for a random start, 2048 for one
that every realization shares), with a second group of realizations."""
import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("shape", [(1, 31), (4, 8), (3, 11), (45, 46), (32, 65), (1, 1, 1), (4, 2, 4), (3, 1, 11), (13, 13, 13)])
def test_energy_of_the_start(shape, mode):
    rng = np.random.default_rng(sum(shape))
    m = (rng.random(shape) < 0.5).astype(np.uint8)
    m.ravel()[0] = 1
    t = rng.random(shape).astype(np.float32) * m
    lb = (5,) * len(shape)
    T = rng.uniform(0.02, 0.5, int(np.prod([-(-n // 5) for n in shape]))).astype(np.float32)
    kw = dict(n_real=65, init_mode=mode, stop_mode=0, n_eq=0, n_samp=0, seed=9)
    plane = len(shape) == 2
    o = (oracle.simulate if plane else oracle.simulate3)(t, m, T, *lb, OCfg(scene=2, **kw))
    g = (M.mpr_simulate if plane else M.mpr_simulate3d)(*(torch.from_numpy(a).cuda() for a in (t, m, T)), *lb,
                                                        M.SimConfig(scene_id=2, sweep_kernel=M.SWEEP_LANES, **kw))
    assert np.array_equal(g.state.cpu().numpy(), o.state)
    # (the GPU's energy rounds each bond to 2^-24 and uses the FP32 cosine)
    assert np.allclose(g.energy.cpu().numpy(), o.energy, rtol=0, atol=1e-5)
