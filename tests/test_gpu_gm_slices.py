"""The global-motion fit at the edges of its slices: one slice more or less, a slice longer than the
lanes hold at a time, and frames whose normal equations are pivoted on each of their rows (wide,
tall, and so small that the constant row is the largest).

Bar: that of the fit on identical samples -- the FP64 oracle's model within 1e-9, relative to the
motion it predicts at the frame corners (both sum at most 3e5 samples in FP64: 3e5 x 1.1e-16 x a
condition below 30 is under 1e-9)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf

pytestmark = pytest.mark.gpu


def _corners(A, W, H):
    c = np.array([[x, y, 1.0] for x in (-0.5 * (W - 1), 0.5 * (W - 1)) for y in (-0.5 * (H - 1), 0.5 * (H - 1))])
    return c @ np.asarray(A).reshape(2, 3).T


@pytest.mark.parametrize("n,W,H", [(511, 1242, 375), (512, 1242, 375), (513, 375, 1242), (1025, 375, 1242),
                                   (700, 2, 2), (131073, 640, 480), (262145, 480, 640), (300001, 2, 2)])
def test_fit_at_slice_edges(n, W, H):
    rng = np.random.default_rng(n)
    pts = np.stack([rng.uniform(0, W - 1, n), rng.uniform(0, H - 1, n)], 1).astype(np.float32)
    x = np.c_[pts.astype(np.float64) - [0.5 * (W - 1), 0.5 * (H - 1)], np.ones(n)]
    mot = x @ np.array([[0.02, -0.01, 12.5], [0.005, 0.03, -4.0]]).T + rng.normal(0, 0.3, (n, 2))
    out = rng.random(n) < 0.2
    mot[out] = rng.uniform(-80, 80, (int(out.sum()), 2))
    mot = mot.astype(np.float32)
    st = np.where(rng.random(n) < 0.1, rng.integers(1, 4, n), 0).astype(np.uint8)
    mot[n // 2, 0] = np.nan
    st[n // 2] = 0
    mot[n - 1, 1] = np.inf
    use = (st == 0) & np.all(np.isfinite(mot), 1)
    o, kind = oracle.gm_fit(pts.astype(np.float64), mot.astype(np.float64), use.astype(np.uint8),
                            (0.5 * (W - 1), 0.5 * (H - 1)), 2.0)
    assert kind == 2
    want = _corners(o, W, H)
    for _ in range(2):
        g = dgf.gm_fit(torch.from_numpy(pts).cuda(), torch.from_numpy(mot).cuda(), torch.from_numpy(st).cuda(), W, H, 2.0)
        err = np.abs(_corners(g.cpu().numpy(), W, H) - want).max() / (1.0 + np.abs(want).max())
        print(f"n={n} {W}x{H} rel={err:.2e}", flush=True)
        assert err <= 1e-9
