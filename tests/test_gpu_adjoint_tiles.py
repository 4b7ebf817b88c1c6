"""The tiled adjoint of batch plans (points of a grid tile combined in LDS) against the FP64 oracle,
at every compiled support and at strides from tiles of 128 points to no tile at all.  Two pairs of
uneven odd size.  The frames repeat every 32 columns, so a point matches at its own place and any
number of repeats away: most points get flow zero, some two repeats, whose dI1 patches lie further
off than a tile reaches and go to device memory one by one; patches hang over the frame's edges.

The illumination model's gradient is that of its fixed point, so its frames match exactly there (gain
1, offset 0, every residual zero); the plain model's have noise and flows a little off.  Bar: relative
L2 <= 1e-4 on dI0 and on dI1 of every pair, the bar of every adjoint test."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf
from paper_1901_09971_amd import synth

pytestmark = pytest.mark.gpu
REPEAT = 32


@pytest.mark.parametrize("support", [5, 7, 9, 11, 15, 21])
@pytest.mark.parametrize("stride,illum", [(1, False), (2, True), (3, False), (5, False), (8, True)])
def test_tiles_against_oracle(support, stride, illum):
    rng = np.random.default_rng(support + 100 * stride)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    f64 = lambda a: np.nan_to_num(np.asarray(a, np.float64))
    made = []
    for W, H in [(151, 61), (197, 43)] if stride > 1 else [(163, 29), (171, 23)]:
        I0 = np.rint(np.tile(synth.smoothed_noise(rng, REPEAT, H, 2.0), (1, W // REPEAT + 1))[:, :W])
        I1 = np.rint(np.clip(I0 + (0.0 if illum else 0.5) * rng.normal(size=I0.shape), 0, 255))
        P = oracle.detect(I0.astype(np.uint8), 9, stride)[0].astype(np.float32)
        r = support // 2 + 2
        dx = np.where(rng.uniform(size=len(P)) < 0.2, 2 * REPEAT, 0) * np.where(P[:, 0] < W / 2, 1, -1)
        moved = P[:, 0] + dx
        ok = (dx == 0) | ((moved >= r) & (moved < W - r) & (P[:, 0] >= r) & (P[:, 0] < W - r))
        st = np.where(ok & (rng.uniform(size=len(P)) < 0.8), 0, 1).astype(np.uint8)
        u = np.stack([dx, 0 * dx], 1) + (0.0 if illum else 0.05) * rng.normal(size=P.shape)
        u = np.where((st == 0)[:, None], u, np.nan).astype(np.float32)
        made.append((I0, I1, P, u, st, rng.normal(size=P.shape).astype(np.float32)))
    plan = dgf.Batch([(dev(m[0].astype(np.uint8)), dev(m[1].astype(np.uint8)), 9, stride) for m in made], 1, support, 1,
                     opts=dgf.TrackOpts(illum=illum))
    cat = lambda k: dev(np.concatenate([m[k] for m in made]))
    _, views = plan.backward(cat(5), points=cat(2), flow=cat(3), status=cat(4),
                             illum=torch.zeros_like(cat(3)) if illum else None)
    torch.cuda.synchronize()
    for (I0, I1, P, u, st, df), got in zip(made, views):
        assert (st == 0).sum() > 30 and (np.abs(f64(u)[:, 0]) > REPEAT).sum() > 3
        if illum:
            ref = oracle.track_grad_illum(f64(I0), f64(I1), f64(P), support, f64(u), f64(0 * u), st, f64(df))
        else:
            ref = oracle.track_grad(f64(I0), f64(I1), f64(P), support, f64(u), st, f64(df))
        for g, o in zip(got, ref):
            rel = np.linalg.norm(g.cpu().numpy() - o) / np.linalg.norm(o)
            print(f"\ns{support} stride {stride} {'IM ' if illum else ''}points {len(P)} rel {rel:.1e}", flush=True)
            assert rel <= 1e-4
    plan.close()
