"""Calls of few sweeps on the tile path take a launch a sweep without update lists from a plan: on both sides of the rule that
decides so (sweeps of the call, tiles times realizations, rows), against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


def _scene(H, W, lb, p, site=False):
    rng = np.random.default_rng(H + W)
    m = (rng.random((H, W)) >= p).astype(np.uint8)
    t = rng.random((H, W)).astype(np.float32) * m
    T = rng.uniform(0.02, 0.5, H * W if site else -(-H // lb[0]) * -(-W // lb[1])).astype(np.float32)
    T[::7] = 0.0
    return t, m, T


def _check(H, W, R, lb, n, p=0.5, site=False):
    t, m, T = _scene(H, W, lb, p, site)
    kw = dict(n_real=R, init_mode=0, stop_mode=0, seed=12, t_mode=int(site))
    o = oracle.simulate(t, m, T, *lb, OCfg(scene=3, n_eq=n, n_samp=0, **kw), parallel=True)
    dev = [torch.from_numpy(a).cuda() for a in (t, m, T)]
    cfg = dict(scene_id=3, sweep_kernel=M.SWEEP_TILES, **kw)
    st = M.mpr_simulate(*dev, *lb, M.SimConfig(n_eq=0, n_samp=0, **cfg)).state
    e = M.mpr_sweep(st, dev[1], dev[2], *lb, M.SimConfig(**cfg), 1, n, want_energy=True)
    assert np.array_equal(st.cpu().numpy(), o.state)
    assert np.allclose(e.cpu().numpy(), o.energy[1:], rtol=0, atol=1e-5)
    g = M.mpr_simulate(*dev, *lb, M.SimConfig(n_eq=n, n_samp=0, **cfg))
    assert np.array_equal(g.state.cpu().numpy(), o.state)
    assert np.allclose(g.energy.cpu().numpy(), o.energy, rtol=0, atol=1e-5)


# four tiles, three of them nearly empty; two tiles of one row
@pytest.mark.parametrize("H,W,R,n", [
    (33, 65, 127, 2), (33, 65, 128, 2), (33, 65, 159, 3), (33, 65, 160, 3), (33, 65, 3, 1), (33, 65, 4095, 4),
    (33, 65, 4096, 4), (33, 65, 12287, 6), (33, 65, 12288, 6), (1, 65, 4095, 4), (1, 65, 4096, 4), (7, 65, 2, 3), (8, 65, 2, 3)])
def test_sides_of_the_rule(H, W, R, n):
    _check(H, W, R, (16, 16), n)


# one tile and its edges; blocks in and outside the table; all gaps, few; workgroups of several realizations with a remainder
@pytest.mark.parametrize("H,W,R,lb,p,site", [
    (1, 1, 2, (1, 1), 1.0, False), (32, 64, 3, (16, 16), 0.6, False), (31, 63, 3, (33, 33), 0.6, False),
    (34, 66, 3, (4, 4), 0.9, False), (70, 131, 3, (16, 16), 0.5, True), (70, 131, 3, (8, 6), 1.0, False),
    (70, 131, 700, (16, 16), 0.1, False), (33, 65, 701, (7, 12), 0.5, False)])
def test_one_sweep(H, W, R, lb, p, site):
    _check(H, W, R, lb, 1, p, site)


@pytest.mark.parametrize("n_eq,n_samp", [(0, 1), (0, 2), (1, 1), (1, 2), (0, 3), (2, 1), (3, 1)])
def test_few_sweeps_sample_as_the_oracle(n_eq, n_samp):
    lb = (16, 16)
    for R in (2, 320):                            # with a plan from two sweeps on, and without up to three
        t, m, T = _scene(45, 70, lb, 0.5)
        kw = dict(n_real=R, init_mode=1, stop_mode=0, n_eq=n_eq, n_samp=n_samp, seed=4)
        o = oracle.simulate(t, m, T, *lb, OCfg(**kw))
        g = M.mpr_simulate(*(torch.from_numpy(a).cuda() for a in (t, m, T)), *lb, M.SimConfig(sweep_kernel=M.SWEEP_TILES, **kw))
        assert np.array_equal(g.state.cpu().numpy(), o.state) and np.array_equal(g.acc.cpu().numpy(), o.acc)
        assert np.allclose(g.energy.cpu().numpy(), o.energy, rtol=0, atol=1e-5)
