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


def _threshold_residuals(count):
    """(residual a, outer threshold s2, weight) of pixels whose weight psi(a) / a = (s2 - a) / a, in FP32
    and the inner threshold s2 / 2, is the least float whose square exceeds 1e-6f, or the one below it."""
    f32, unit = np.float32, np.float32(2.0 ** -20)
    w = f32(1e-3)
    while w * w > f32(1e-6):
        w = np.nextafter(w, f32(0))
    pair = (w, np.nextafter(w, f32(1)))
    assert not pair[0] * pair[0] > f32(1e-6) and pair[1] * pair[1] > f32(1e-6)
    out = []
    for k in range(8400, 16700):  # s2 - a and a in units of 2^-20, so that a, s2 and the difference are exact
        for m in range(int(k / float(pair[1])) - 1, int(k / float(pair[0])) + 3):
            a, s2 = f32(m) * unit, f32(m + k) * unit
            assert a + f32(k) * unit == s2 and m + k <= 1 << 24
            q = (s2 - a) / a
            if q in pair:
                out.append((a, s2, q))
    return out[:: max(1, len(out) // count)][:count]


@pytest.mark.parametrize("support", [5, 9, 21])
def test_fallback_threshold_takes_the_rounded_quotient(support):
    """Four pixels around a spike carry all the gradient and share one weight w, every other quantity is
    exact, and the point falls back to least squares exactly where fl(w w) <= 1e-6f: the decision then
    tells whether w is the correctly rounded psi / r.  Least squares shows in dI0, whose terms in psi are
    then of the residuals' size (about 16) instead of a thousandth of it."""
    N = 41
    c = N // 2
    t = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")
    I0 = torch.zeros((N, N), device="cuda")
    I0[c, c] = 2.0
    P, u, df = t([[c, c]]), t([[0.0, 0.0]]), t([[1.0, 0.5]])
    st = torch.zeros(1, dtype=torch.uint8, device="cuda")
    cases = _threshold_residuals(300)
    assert len(cases) >= 200 and 20 < sum(q * q > np.float32(1e-6) for _, _, q in cases) < len(cases) - 20
    grads = []
    for a, s2, _ in cases:
        I1 = torch.full((N, N), float(a), device="cuda")
        I1[c, c] = float(a) - 0.5
        d0, d1 = torch.zeros_like(I0), torch.zeros_like(I0)
        dgf.track_backward(I0, I1, P, support, u, st, df, d0, d1, opts=dgf.TrackOpts(sigma1=float(s2) / 2, sigma2=float(s2)),
                           dpoints=torch.empty_like(P))
        grads.append(d0.abs().max())
    least_squares = (torch.stack(grads) > 4.0).cpu().numpy()
    want = np.array([not q * q > np.float32(1e-6) for _, _, q in cases])
    print(f"s{support}: {len(cases)} points, {want.sum()} by least squares, {(least_squares != want).sum()} wrong", flush=True)
    assert np.array_equal(least_squares, want)
