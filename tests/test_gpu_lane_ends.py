"""The start and the end of the chains in the lane layout against the oracle: odd sites and rows, groups of realizations with a
remainder, block-mean and random starts, no sweep at all, several sampling sweeps, energies of more sweeps than are reduced
together, on the plane and on the cubic lattice."""
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


def same(g, o):
    assert np.array_equal(g.state.cpu().numpy().reshape(o.state.shape), o.state)
    assert np.array_equal(g.acc.cpu().numpy().reshape(o.acc.shape), o.acc)
    assert np.allclose(g.energy.cpu().numpy(), o.energy[:len(g.energy)], rtol=0, atol=1e-5)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("H,W,lb,R,n_eq,n_samp", [
    (1, 1, (4, 4), 64, 2, 1), (3, 5, (2, 2), 65, 0, 0), (9, 67, (4, 16), 70, 0, 1), (33, 31, (8, 5), 128, 9, 2),
    (40, 64, (16, 16), 100, 17, 3), (5, 130, (64, 64), 192, 3, 0)])
def test_plane(H, W, lb, R, n_eq, n_samp, mode):
    rng = np.random.default_rng(H * W + R)
    z = rng.normal(size=(H, W)).astype(np.float32)
    m = (rng.random((H, W)) < 0.45).astype(np.uint8)
    m[0, 0] = 1
    t, _ = oracle.map_angles(z, m)
    T = rng.uniform(0.02, 0.5, -(-H // lb[0]) * -(-W // lb[1])).astype(np.float32)
    kw = dict(n_real=R, init_mode=mode, stop_mode=0, n_eq=n_eq, n_samp=n_samp, seed=6)
    o = oracle.simulate(t, m, T, *lb, OCfg(scene=2, **kw))
    g = M.mpr_simulate(dev(t), dev(m), dev(T), *lb, M.SimConfig(sweep_kernel=M.SWEEP_LANES, scene_id=2, **kw))
    same(g, o)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("D,H,W,lb,R,n_eq,n_samp", [
    (1, 1, 1, (2, 2, 2), 3, 1, 1), (3, 5, 7, (2, 2, 3), 65, 0, 0), (5, 4, 10, (8, 8, 8), 70, 10, 2), (9, 3, 17, (4, 2, 16), 64, 0, 1)])
def test_cube(D, H, W, lb, R, n_eq, n_samp, mode):
    rng = np.random.default_rng(D * H * W + R)
    t = rng.random((D, H, W)).astype(np.float32)
    m = (rng.random((D, H, W)) < 0.4).astype(np.uint8)
    m[0, 0, 0] = 1
    t *= m
    B = -(-D // lb[0]) * -(-H // lb[1]) * -(-W // lb[2])
    T = rng.uniform(0.02, 0.5, B).astype(np.float32)
    kw = dict(n_real=R, init_mode=mode, stop_mode=0, n_eq=n_eq, n_samp=n_samp, seed=6)
    o = oracle.simulate3(t, m, T, *lb, OCfg(scene=2, **kw))
    g = M.mpr_simulate3d(dev(t), dev(m), dev(T), *lb, M.SimConfig(scene_id=2, **kw))
    same(g, o)


@pytest.mark.parametrize("mode", [0, 1])
def test_batch(mode):
    rng = np.random.default_rng(mode)
    scenes, ref = [], []
    for i, (H, W) in enumerate([(20, 37), (64, 32), (9, 130)]):
        m = (rng.random((H, W)) < 0.5).astype(np.uint8)
        t = rng.random((H, W)).astype(np.float32) * m
        T = rng.uniform(0.05, 0.4, -(-H // 16) * -(-W // 16)).astype(np.float32)
        scenes.append(dict(t=dev(t), mask=dev(m), T_blocks=dev(T), block=(16, 16), scene_id=i))
        ref.append((t, m, T))
    kw = dict(n_real=66, init_mode=mode, stop_mode=0, n_eq=4, n_samp=2, seed=6)
    outputs = M.mpr_simulate_batched(scenes, M.SimConfig(**kw), want_energy=True).outputs
    for g, (t, m, T), s in zip(outputs, ref, scenes):
        o = oracle.simulate(t, m, T, 16, 16, OCfg(scene=s["scene_id"], **kw))
        same(g, o)
