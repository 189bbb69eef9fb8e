"""Block energies and the gradient against the oracle where their kernels divide the work: one or eight realizations per wave,
counts that leave a remainder, blocks over several chunks, sites four at a time or one by one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("H,W,lb,R,q", [
    (1, 1, (4, 4), 2, 0.5), (7, 13, (3, 5), 3, 0.3), (64, 64, (64, 64), 9, 0.5), (90, 75, (90, 8), 12, 0.5),
    (128, 96, (2, 2), 17, 0.45), (130, 130, (2, 3), 15, 0.5), (200, 330, (16, 16), 131, 0.5), (1100, 1000, (700, 600), 2, 0.5)])
def test_block_energy_and_gradient(H, W, lb, R, q):
    rng = np.random.default_rng(H * W + R)
    state = rng.random((R, H, W)).astype(np.float32)
    m = (rng.random((H, W)) < 0.5).astype(np.uint8)
    Ho = np.stack([oracle.block_energy(state[r], m, *lb, q) for r in range(R)])
    Hg = M.mpr_block_energy(dev(state), dev(m), *lb, q)
    n = 2 * min(lb[0], H) * min(lb[1], W)                     # bonds of a block: n roundings of a running sum of at most n
    assert np.abs(Hg.cpu().numpy().reshape(Ho.shape) - Ho).max() <= 1.2e-16 * n * (n + 8)
    gz = rng.standard_normal((H, W)).astype(np.float32)
    rg = np.array([-1.5, 2.25])
    T = rng.uniform(0.05, 0.5, Ho.shape[1]).astype(np.float32)
    T[0] = 0.0
    Hh = Hg.cpu().numpy().reshape(Ho.shape)
    do = oracle.temperature_grad(state, Hh, np.where(m == 0, gz.astype(np.float64) * (rg[1] - rg[0]), 0.0), T)
    dg = M.mpr_temperature_grad(dev(state), Hg, dev(gz), dev(m), dev(rg), dev(T)).cpu().numpy().ravel()
    assert np.allclose(dg, do, rtol=1e-9, atol=1e-12 * np.abs(do).max())
    # memory that begins one element into an allocation
    off = lambda a: dev(np.concatenate([np.zeros(1, a.dtype), a.ravel()]))[1:].reshape(a.shape)
    d1 = M.mpr_temperature_grad(off(state), Hg, off(gz), off(m), dev(rg), dev(T)).cpu().numpy().ravel()
    assert np.allclose(d1, do, rtol=1e-9, atol=1e-12 * np.abs(do).max())
