"""The steps around the chains against the oracle where their kernels divide the work: sites four at a time or one by one,
blocks over several chunks, curves on both sides of the points held in memory next to the core, medians between equal and
different values, and the mean of all samples over more blocks than one chunk of its sum."""
import math

import numpy as np
import pytest
import torch

import oracle
from oracle import SimConfig as OCfg
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def off(a, shift):
    """The same values in memory that begins `shift` elements into an allocation."""
    a = np.ascontiguousarray(a)
    return dev(np.concatenate([np.zeros(shift, a.dtype), a.ravel()]))[shift:].reshape(a.shape)


@pytest.mark.parametrize("H,W,shift", [(1, 1, 0), (2, 2, 0), (33, 31, 0), (64, 48, 0), (64, 48, 1), (64, 48, 2), (700, 900, 0)])
def test_map_predict_validate(H, W, shift):
    rng = np.random.default_rng(H * W + shift)
    z = rng.normal(3.0, 7.0, (H, W)).astype(np.float32)
    m = (rng.random((H, W)) < 0.6).astype(np.uint8)
    m[0, 0] = 1
    to, ro = oracle.map_angles(z, m)
    tg, rg = M.mpr_map_angles(off(z, shift), off(m, shift))
    assert np.array_equal(host(tg), to) and np.array_equal(host(rg), ro)
    acc = rng.random((H, W)) * 11
    zo = oracle.predict(acc, z, m, 11, ro)
    zg = M.mpr_predict(off(acc, shift), off(z, shift), off(m, shift), 11, rg)
    assert np.array_equal(host(zg), zo)
    truth = rng.normal(3.0, 7.0, (H, W)).astype(np.float32)
    vo = oracle.validate(zo, truth, 1 - m)
    vg = host(M.mpr_validate(off(zo, shift), off(truth, shift), off(1 - m, shift)))
    assert np.allclose(vg, vo, rtol=1e-12, atol=0)            # two sums of H W positive FP64 terms in another order


def _exact_bond_sums(t, m, lb, q):
    """Bond energies of each block, FP64 terms summed without rounding (the oracle's running sum of 1.2 million bonds is
    off by 3e-9, more than the bound below)."""
    H, W = t.shape
    d, k = t.astype(np.float64), 2 * np.pi * np.float64(np.float32(q))
    cx, mx = np.cos(k * (d[:, :-1] - d[:, 1:])), (m[:, :-1] & m[:, 1:]) == 1
    cy, my = np.cos(k * (d[:-1] - d[1:])), (m[:-1] & m[1:]) == 1
    S = []
    for y in range(0, H, lb[0]):
        for x in range(0, W, lb[1]):
            ys, xs = slice(y, y + lb[0]), slice(x, x + lb[1])
            S.append(-math.fsum(np.concatenate([cx[ys, xs][mx[ys, xs]], cy[ys, xs][my[ys, xs]]])))
    return np.array(S)


@pytest.mark.parametrize("H,W,lb", [(128, 128, (128, 128)), (90, 300, (90, 17)), (1500, 800, (1500, 800)), (5, 3000, (4, 2000)),
                                    (130, 129, (2, 2)), (67, 61, (1, 1)), (2100, 2050, (32, 32))])
def test_block_stats_over_chunks(H, W, lb):
    rng = np.random.default_rng(H * W)
    t = rng.random((H, W)).astype(np.float32)
    m = (rng.random((H, W)) < 0.55).astype(np.uint8)
    for q in (0.5, 0.3):
        _, No, To, Oo = oracle.block_stats(t, m, *lb, q)
        So = _exact_bond_sums(t, m, lb, q)
        Sg, Ng, Tg, Og = (host(x) for x in M.mpr_block_stats(dev(t), dev(m), *lb, q))
        assert np.array_equal(Ng, No) and np.array_equal(Og, Oo)
        assert np.allclose(Sg, So, rtol=0, atol=2e-16 * H * W) and np.allclose(Tg, To, rtol=1e-12, atol=0)


def _curve(n, kind):
    cT = np.geomspace(1e-3, 5.0, n)
    ce = -1.0 + 0.95 * np.linspace(0.02, 1.0, n)
    if kind == "noisy":                                       # falls back now and then: the running maximum is used
        ce = ce + np.random.default_rng(n).normal(0, 0.05, n)
    if kind == "gaps":
        ce[1::5] = np.nan
    if kind == "no first point":
        ce[0] = np.nan
    return cT, ce


@pytest.mark.parametrize("n,kind", [(1, ""), (2, "noisy"), (64, "noisy"), (121, ""), (257, "gaps"), (300, "no first point"),
                                    (1024, "noisy"), (1025, "noisy"), (1025, "gaps")])
def test_calibrate_curves(n, kind):
    H, W, lb = 120, 200, (7, 9)
    rng = np.random.default_rng(n)
    t = (0.3 * rng.random((H, W)) * np.linspace(0.01, 3.0, W)[None]).astype(np.float32) % 1.0
    m = (rng.random((H, W)) < 0.8).astype(np.uint8)
    cT, ce = _curve(n, kind)
    To, _, No = oracle.calibrate_temperature(t, m, *lb, cT, ce)
    Tg, _, Ng = M.mpr_calibrate_temperature(dev(t), dev(m), *lb, dev(cT), dev(ce))
    assert np.array_equal(host(Ng), No)
    # two FP64 exp/log of a few ulp each before the rounding to FP32: at most its last place
    np.testing.assert_array_max_ulp(host(Tg), To, 1)


@pytest.mark.parametrize("have,equal", [(1, False), (2, False), (2, True), (3, False), (6, True), (40, False), (41, False), (48, False)])
def test_median_of_the_blocks_with_bonds(have, equal):
    """48 blocks of 6 x 6, `have` of them with bonds; the others take the median."""
    H, W = 36, 48
    rng = np.random.default_rng(have)
    t = rng.random((H, W)).astype(np.float32)
    if equal:
        t = np.tile(rng.random((6, 6)).astype(np.float32), (6, 8))
    m = np.zeros((6, 6, 8, 6), np.uint8)
    for i, b in enumerate(rng.permutation(48)):
        m[b // 8, :5, b % 8, :5] = i < have
    m = m.reshape(H, W)
    cT, ce = _curve(121, "")
    To, _, No = oracle.calibrate_temperature(t, m, 6, 6, cT, ce)
    Tg, _, Ng = M.mpr_calibrate_temperature(dev(t), dev(m), 6, 6, dev(cT), dev(ce))
    assert np.array_equal(host(Ng), No) and (No > 0).sum() == have
    np.testing.assert_array_max_ulp(host(Tg), To, 1)


@pytest.mark.parametrize("H,W,lb", [(12, 20, (3, 4)), (128, 64, (2, 2)), (130, 66, (2, 2)), (200, 100, (1, 2))])
def test_start_of_blocks_without_samples(H, W, lb):
    """No sweep: the sum of one realization's start, gaps of empty blocks at the mean of all samples."""
    rng = np.random.default_rng(H)
    t = rng.random((H, W)).astype(np.float32)
    m = (rng.random((H, W)) < 0.3).astype(np.uint8)
    t *= m
    B = -(-H // lb[0]) * -(-W // lb[1])
    T = np.full(B, 0.1, np.float32)
    kw = dict(n_real=1, init_mode=1, stop_mode=0, n_eq=0, n_samp=1, seed=4)
    o = oracle.simulate(t, m, T, *lb, OCfg(scene=1, **kw))
    g = M.mpr_simulate(dev(t), dev(m), dev(T), *lb, M.SimConfig(scene_id=1, **kw))
    assert np.array_equal(host(g.state), o.state)
