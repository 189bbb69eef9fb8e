"""Several realizations in one workgroup of the tile sweeps and in one thread of the double checkerboard, with a remainder,
against the oracle bit for bit: what is kept from one realization to the next (angles requested ahead, cells beyond the tile)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


def _scene(H, W, lb, site, p=0.5):
    rng = np.random.default_rng(H + W)
    m = (rng.random((H, W)) >= p).astype(np.uint8)
    t = rng.random((H, W)).astype(np.float32) * m
    T = rng.uniform(0.02, 0.5, H * W if site else -(-H // lb[0]) * -(-W // lb[1])).astype(np.float32)
    T[::7] = 0.0
    return t, m, T


def _check(t, m, T, lb, site, gpu, **kw):
    o = oracle.simulate(t, m, T, *lb, OCfg(scene=4, t_mode=int(site), order=gpu.get("order", 0), **kw), parallel=True)
    g = M.mpr_simulate(*(torch.from_numpy(a).cuda() for a in (t, m, T)), *lb,
                       M.SimConfig(scene_id=4, t_mode=M.T_SITE if site else M.T_BLOCK, **gpu, **kw))
    assert np.array_equal(g.state.cpu().numpy(), o.state)
    assert np.array_equal(g.acc.cpu().numpy(), o.acc)
    assert np.allclose(g.energy.cpu().numpy(), o.energy, rtol=0, atol=1e-5)


# with and without the temperature table; with the states of several sampling sweeps, and one sampling sweep
@pytest.mark.parametrize("lb,site,R,n_eq,n_samp", [
    ((16, 16), False, 61, 6, 3), ((33, 33), False, 61, 6, 3), ((16, 16), True, 61, 6, 2), ((16, 16), False, 181, 3, 1),
    ((33, 33), False, 61, 2, 1), ((16, 16), True, 95, 4, 0)])
def test_tile_sweeps_several_realizations_a_workgroup(lb, site, R, n_eq, n_samp):
    H, W = 197, 300
    chunk = -(-H // 32) * -(-W // 64) * R // 1024
    assert chunk >= 2 and R % chunk != 0
    t, m, T = _scene(H, W, lb, site)
    _check(t, m, T, lb, site, dict(sweep_kernel=M.SWEEP_TILES), n_real=R, init_mode=0, stop_mode=0, n_eq=n_eq, n_samp=n_samp,
           seed=5)


@pytest.mark.parametrize("H,W,lb,site,R", [
    (600, 500, (16, 24), False, 29), (600, 500, (16, 24), True, 29), (700, 900, (16, 16), False, 30),
    (700, 900, (5, 7), False, 57)])
def test_double_checkerboard_several_realizations_a_thread(H, W, lb, site, R):
    chunk = min(8, H * -(-W // 4) // 2 * R // (256 * 2048))
    assert chunk >= 2 and R % chunk != 0
    t, m, T = _scene(H, W, lb, site)
    _check(t, m, T, lb, site, dict(order=M.ORDER_DC), n_real=R, init_mode=0, stop_mode=0, n_eq=1, n_samp=1, seed=5)
