"""The adjoint of float32 pairs with point gradients at every compiled support, where the robust norm's
bands are all in use: residuals that are exactly zero (an unchanged background, flat and saturated
regions), residuals beyond the outer threshold, and with the plain model those between the two.

The frames hold whole grey levels, the positions are whole or half pixels and the flow is zero, so every
residual is exact in FP32 and takes the same band as in FP64.  The illumination model's outliers are all
beyond the outer threshold, at whole positions: the point is then a fixed point of the model at gain 1 and
offset 0.  (Not at support 5: of the few pixels left some points' four unknowns are not determined in FP32.)
Bar: relative L2 <= 1e-4 on dI0, dI1 and dp, the bar of every adjoint test."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf
from paper_1901_09971_amd import synth

pytestmark = pytest.mark.gpu
SUPPORTS = [5, 7, 9, 11, 15, 21]


@pytest.mark.parametrize("support,illum", [(s, False) for s in SUPPORTS] + [(s, True) for s in SUPPORTS[1:]])
def test_exact_matches_and_outliers(support, illum):
    rng = np.random.default_rng(1000 * illum + support)
    W, H = 117, 83
    I0 = np.rint(synth.smoothed_noise(rng, W, H, 2.0))
    I0 = np.clip(np.rint((I0 - I0.mean()) * 2 + 128), 0, 255)
    out = rng.uniform(size=I0.shape) < 0.15
    I1 = np.where(out, np.where(I0 < 128, I0 + 100, I0 - 100), I0)
    if not illum:  # and some in every band
        I1 = np.where(rng.uniform(size=I0.shape) < 0.3, I0 + rng.integers(-40, 41, I0.shape), I1)
    ys, xs = np.mgrid[4:H - 4:5, 4:W - 4:5]
    P = np.stack([xs.ravel(), ys.ravel()], 1).astype(np.float64)
    if not illum:
        P += 0.5 * rng.integers(0, 2, P.shape) * (rng.uniform(size=(len(P), 1)) < 0.5)
    st = (rng.uniform(size=len(P)) < 0.1).astype(np.uint8)
    u, df = np.zeros_like(P), rng.normal(size=P.shape).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).float().cuda()
    t0, t1, tp = t(I0), t(I1), t(P)
    dI0, dI1, dp = torch.zeros_like(t0), torch.zeros_like(t1), torch.full_like(tp, np.nan)
    dgf.track_backward(t0, t1, tp, support, t(u), torch.from_numpy(st).cuda(), t(df), dI0, dI1,
                       opts=dgf.TrackOpts(illum=illum), dpoints=dp, illum=t(u) if illum else None)
    torch.cuda.synchronize()
    if illum:
        ref = oracle.track_grad_illum(I0, I1, P, support, u, u, st, df.astype(np.float64), return_dpoints=True)
    else:
        ref = oracle.track_grad(I0, I1, P, support, u, st, df.astype(np.float64), return_dpoints=True)
    for name, g, o in zip(("dI0", "dI1", "dp"), (dI0, dI1, dp), ref):
        rel = np.linalg.norm(g.cpu().numpy() - o) / np.linalg.norm(o)
        print(f"s{support} {'IM ' if illum else ''}{name} rel {rel:.1e}", flush=True)
        assert rel <= 1e-4, name
    assert torch.all(dp[torch.from_numpy(st != 0).cuda()] == 0)
