"""The global-motion fit at the edges of its forms (one workgroup up to 4096 points) and slices: one slice more or less, a slice longer than the
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
                                   (700, 2, 2), (1023, 640, 480), (4096, 375, 1242), (4097, 640, 480), (131073, 640, 480), (262145, 480, 640), (300001, 2, 2)])
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


def test_plan_with_pairs_on_both_sides():
    rng = np.random.default_rng(3)
    pairs = []
    for W, H, stride in ((320, 240, 5), (400, 320, 5), (331, 203, 3), (90, 70, 5)):
        I0 = rng.integers(0, 256, (H // 4 + 2, W // 4 + 2)).astype(np.uint8).repeat(4, 0).repeat(4, 1)[:H + 3, :W + 2]
        a, b = torch.from_numpy(I0[:H, :W].copy()).cuda(), torch.from_numpy(I0[3:H + 3, 2:W + 2].copy()).cuda()
        pairs.append((a, b, 9, stride))
    opts = dgf.TrackOpts(global_motion=True)
    plan = dgf.Batch(pairs, 3, 9, 10, opts)
    sizes = np.diff(plan.offsets)
    assert sizes.min() < 512 and (sizes <= 4096).any() and (sizes > 4096).any()
    pts, flow, status = plan.run()
    for k, (a, b, w, stride) in enumerate(pairs):
        lo, hi = plan.offsets[k], plan.offsets[k + 1]
        f, st = dgf.track(a, b, dgf.detect(a, w, stride), 3, 9, 10, opts=opts)
        assert torch.equal(st, status[lo:hi])
        assert torch.equal(torch.nan_to_num(f, nan=-1e9), torch.nan_to_num(flow[lo:hi], nan=-1e9)), k
