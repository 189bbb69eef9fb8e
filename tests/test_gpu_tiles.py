"""The tile sweeps (several sweeps per launch on a 64 x 32 tile with a ring) against the oracle: chains bit for bit and
energies within 1e-5 per bond, at grid sides around the tile and ring edges, with block layouts on both sides of the
temperature table's rule, and at sweep counts around the number of sweeps of a launch."""
import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M
from paper_2212_01317_amd import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def _scene(H, W, p, lb, seed=5):
    sc = synth.random_small(H, W, p, seed=seed)
    t, _ = oracle.map_angles(sc.z_obs, sc.mask)
    B = (-(-H // lb[0])) * (-(-W // lb[1]))
    T = np.exp(np.random.default_rng(seed).uniform(np.log(0.01), np.log(0.6), B)).astype(np.float32)
    T[::7] = 0.0
    return t, sc.mask, T


# blocks: in the table; at its limit (columns of four); too many for it; columns that split a pair
@pytest.mark.parametrize("H,W,lb,p,R,n_eq,n_samp", [
    (32, 64, (16, 16), 0.6, 3, 5, 0), (33, 65, (8, 8), 0.5, 2, 6, 1), (64, 128, (64, 128), 0.9, 2, 11, 2),
    (43, 74, (8, 4), 0.7, 2, 4, 1), (75, 131, (4, 4), 0.5, 2, 5, 1), (41, 139, (33, 33), 0.6, 3, 7, 1),
    (97, 70, (1, 1), 0.4, 2, 3, 1), (3, 300, (2, 12), 0.8, 2, 9, 1), (200, 2, (10, 8), 0.5, 5, 1, 1)])
def test_tile_sweeps_match_oracle(H, W, lb, p, R, n_eq, n_samp):
    print(f"[tiles] {H}x{W} blocks {lb} R={R} sweeps {n_eq}+{n_samp}", flush=True)
    t, mask, T = _scene(H, W, p, lb)
    kw = dict(n_real=R, init_mode=0, stop_mode=0, n_eq=n_eq, n_samp=n_samp, seed=12)
    o = oracle.simulate(t, mask, T, *lb, OCfg(scene=3, **kw))
    g = M.mpr_simulate(dev(t), dev(mask), dev(T), *lb, M.SimConfig(sweep_kernel=M.SWEEP_TILES, scene_id=3, **kw))
    assert np.array_equal(host(g.state), o.state)
    assert np.array_equal(host(g.acc), o.acc)
    assert np.allclose(host(g.energy), o.energy, rtol=0, atol=1e-5)


@pytest.mark.parametrize("n_fit,n_f,n_max", [(4, 3, 60), (6, 7, 60), (20, 5, 27), (3, 1, 9)])
def test_tile_sweeps_stop_where_the_oracle_stops(n_fit, n_f, n_max):
    t, mask, T = _scene(50, 90, 0.5, (16, 16))
    kw = dict(n_real=4, init_mode=1, stop_mode=1, n_fit=n_fit, n_f=n_f, n_max=n_max, n_samp=3, seed=8)
    o = oracle.simulate(t, mask, T, 16, 16, OCfg(**kw))
    g = M.mpr_simulate(dev(t), dev(mask), dev(T), 16, 16, M.SimConfig(sweep_kernel=M.SWEEP_TILES, **kw))
    assert (g.sweeps, g.converged) == (o.k_star, o.converged)
    assert np.array_equal(host(g.state), o.state) and np.array_equal(host(g.acc), o.acc)
    assert np.allclose(host(g.energy), o.energy, rtol=0, atol=1e-5)


@pytest.mark.parametrize("n", [1, 2, 5, 6, 8, 10, 11])
def test_continued_sweeps_leave_the_last_two_states_in_the_two_buffers(n):
    """Sweep by sweep the buffers alternate, so after n sweeps one holds the state after n and the other after n - 1."""
    lb, R = (16, 16), 3
    t, mask, T = _scene(70, 140, 0.5, lb)
    cfg = M.SimConfig(n_real=R, seed=3)
    start = M.mpr_simulate(dev(t), dev(mask), dev(T), *lb,
                           M.SimConfig(n_real=R, init_mode=M.INIT_RANDOM, stop_mode=M.STOP_FIXED, n_eq=2, n_samp=0,
                                       seed=3)).state
    one, two = start.clone(), start.clone()
    energies = []
    for i in range(n):
        if i == n - 1:
            two.copy_(one)
        energies.append(host(M.mpr_sweep(one, dev(mask), dev(T), *lb, cfg, 3 + i, 1, want_energy=True))[0])
    st, alt = start.clone(), start.clone()
    e = M.mpr_sweep(st, dev(mask), dev(T), *lb, cfg, 3, n, want_energy=True, state_alt=alt)
    assert np.array_equal(host(st), host(one))
    assert np.array_equal(host(e), np.array(energies))
    # (an odd count ends in state_alt, from which the binding copies the result back)
    assert np.array_equal(host(alt), host(one if n % 2 else two))


@pytest.mark.parametrize("n_eq,n_samp", [(0, 2), (3, 5), (1, 6), (5, 11)])
def test_sampling_sweeps_of_one_launch_match_oracle(n_eq, n_samp):
    t, mask, T = _scene(45, 99, 0.5, (16, 16))
    kw = dict(n_real=3, init_mode=0, stop_mode=0, n_eq=n_eq, n_samp=n_samp, seed=21)
    o = oracle.simulate(t, mask, T, 16, 16, OCfg(**kw))
    g = M.mpr_simulate(dev(t), dev(mask), dev(T), 16, 16, M.SimConfig(sweep_kernel=M.SWEEP_TILES, **kw))
    assert np.array_equal(host(g.state), o.state) and np.array_equal(host(g.acc), o.acc)
