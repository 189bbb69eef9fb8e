"""The covariance of the temperature gradient on both sides of the rule that gives a block a thread or 32 lanes, against the
same sums in NumPy."""
import numpy as np
import pytest
import torch

from paper_2212_01317_amd import _lib as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,R", [(1, 2), (7, 40), (65535, 32), (65536, 32), (65536, 33), (65536, 2), (196607, 33), (196608, 33),
                                 (196609, 40)])
def test_covariance(B, R):
    rng = np.random.default_rng(B + R)
    H, W = 6, 10
    m = (rng.random((H, W)) < 0.4).astype(np.uint8)
    st = rng.random((R, H, W)).astype(np.float32)
    gz = rng.normal(size=(H, W)).astype(np.float32)
    Hb = rng.normal(-20.0, 3.0, (R, B))
    T = rng.uniform(0.05, 1.0, B).astype(np.float32)
    T[::9] = 0.0
    lo, hi = -1.5, 2.0
    w = np.where(m == 0, gz.astype(np.float64) * (hi - lo), 0.0)
    g = (w * st).reshape(R, -1).sum(1)
    hm = Hb.mean(0)
    T2 = np.where(T > 0, T.astype(np.float64) ** 2, 1.0)
    ref = np.where(T > 0, ((g - g.mean())[:, None] * (Hb - hm)).sum(0) / (R - 1) / T2, 0.0)
    # every sum in any order: at most (terms) eps of the sum of the magnitudes, of g, of the means and of the covariance
    mag = np.abs(w * st).reshape(R, -1).sum(1).max()
    tol = (H * W + 4 * R) * 2.0 ** -52 * 2 * mag * (np.abs(Hb) + np.abs(hm)).sum(0) / (R - 1) / T2
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    d = M.mpr_temperature_grad(dev(st), dev(Hb), dev(gz), dev(m), torch.tensor([lo, hi], dtype=torch.float64, device="cuda"),
                               dev(T)).cpu().numpy()
    assert (np.abs(d - ref) <= tol).all()
    assert (d[T == 0] == 0).all()
