"""The 3D sweep's deferred exact decisions against the oracle: with a small q and T = 0 every energy change lies inside
the FP32 filter's band, so every update is noted and settled by the exact test (the notes of a wave overflow within a
few planes); and odd rows, ragged bands and segments of the row-pair layout with a mixture of temperatures."""
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


@pytest.mark.parametrize("D,H,W,lb,R,q,zero_T", [
    (21, 6, 13, (30, 30, 30), 66, 1e-4, True), (9, 5, 8, (4, 2, 8), 64, 1e-4, True), (10, 7, 17, (3, 2, 5), 70, 0.5, False),
    (5, 1, 9, (2, 1, 4), 64, 0.5, False), (1, 3, 16, (1, 2, 8), 65, 0.25, False), (33, 2, 1, (8, 1, 1), 64, 0.5, False)])
def test_sweep3_matches_oracle(D, H, W, lb, R, q, zero_T):
    print(f"[3d settle] {D}x{H}x{W} blocks {lb} R={R} q={q}", flush=True)
    rng = np.random.default_rng(D * 100 + W)
    t = rng.random((D, H, W)).astype(np.float32)
    mask = (rng.random((D, H, W)) < 0.4).astype(np.uint8)
    mask[0, 0, 0] = 1
    nb = [-(-n // l) for n, l in zip((D, H, W), lb)]
    T = np.zeros(nb, np.float32) if zero_T else np.exp(rng.uniform(-4, 0, nb)).astype(np.float32)
    if not zero_T:
        T.ravel()[::5] = 0.0
    kw = dict(q=q, n_real=R, init_mode=0, stop_mode=0, n_eq=5, n_samp=1, seed=9)
    o = oracle.simulate3(t, mask, T, *lb, OCfg(**kw))
    g = M.mpr_simulate3d(dev(t), dev(mask), dev(T), *lb, M.SimConfig(**kw))
    assert np.array_equal(host(g.state), o.state)
    assert np.array_equal(host(g.acc), o.acc)
    assert np.allclose(host(g.energy), o.energy, rtol=0, atol=1e-5)
