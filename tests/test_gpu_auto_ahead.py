"""The automatic stop with sweeps queued ahead of the checks: the same stopping sweep, states and sums as the oracle on both
sweep kernels, for windows and check intervals around the sweeps of a launch, stops at a check, at n_max between checks and at
n_max on a check, several threads with a stream each, and more sweeps than the host block holds."""
import threading

import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _scene(H, W, seed):
    rng = np.random.default_rng(seed)
    m = (rng.random((H, W)) < 0.5).astype(np.uint8)
    t = rng.random((H, W)).astype(np.float32) * m
    T = rng.uniform(0.05, 0.4, -(-H // 16) * -(-W // 16)).astype(np.float32)
    return t, m, T


@pytest.mark.parametrize("kernel,R", [(M.SWEEP_TILES, 3), (M.SWEEP_LANES, 64)])
@pytest.mark.parametrize("n_fit,n_f,n_max,mode", [(20, 5, 200, 0), (4, 3, 60, 1), (6, 7, 33, 0), (3, 1, 40, 1), (5, 12, 17, 0), (8, 4, 11, 0)])
def test_stop_matches_oracle(kernel, R, n_fit, n_f, n_max, mode):
    t, m, T = _scene(70, 90, n_fit + n_f)
    kw = dict(n_real=R, init_mode=mode, stop_mode=1, n_fit=n_fit, n_f=n_f, n_max=n_max, n_samp=2, seed=3)
    o = oracle.simulate(t, m, T, 16, 16, OCfg(scene=5, **kw))
    g = M.mpr_simulate(dev(t), dev(m), dev(T), 16, 16, M.SimConfig(sweep_kernel=kernel, scene_id=5, **kw))
    assert g.sweeps == o.k_star
    assert np.array_equal(g.state.cpu().numpy(), o.state)
    assert np.array_equal(g.acc.cpu().numpy(), o.acc)
    assert np.allclose(g.energy.cpu().numpy(), o.energy[:o.k_star + 1], rtol=0, atol=1e-5)


def test_more_sweeps_than_the_host_block():
    t, m, T = _scene(20, 30, 1)
    kw = dict(n_real=2, init_mode=0, stop_mode=1, n_samp=1, seed=3, n_fit=10, n_f=5)
    a = M.mpr_simulate(dev(t), dev(m), dev(T), 16, 16, M.SimConfig(n_max=5000, **kw))
    b = M.mpr_simulate(dev(t), dev(m), dev(T), 16, 16, M.SimConfig(n_max=1000, **kw))
    assert a.sweeps == b.sweeps and torch.equal(a.state, b.state) and torch.equal(a.energy, b.energy)


def test_threads_with_their_own_streams():
    scenes = [_scene(64, 96, i) for i in range(4)]
    cfg = lambda i: M.SimConfig(n_real=4, init_mode=0, stop_mode=1, n_max=100, n_samp=1, seed=3, scene_id=i)
    args = [(dev(t), dev(m), dev(T)) for t, m, T in scenes]
    alone = [M.mpr_simulate(*a, 16, 16, cfg(i)) for i, a in enumerate(args)]
    torch.cuda.synchronize()
    got = [None] * 4

    def run(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(3):
                got[i] = M.mpr_simulate(*args[i], 16, 16, cfg(i))
            s.synchronize()

    threads = [threading.Thread(target=run, args=(i,)) for i in range(4)]
    [x.start() for x in threads]
    [x.join() for x in threads]
    for a, b in zip(alone, got):
        assert a.sweeps == b.sweeps and torch.equal(a.state, b.state) and torch.equal(a.acc, b.acc)
