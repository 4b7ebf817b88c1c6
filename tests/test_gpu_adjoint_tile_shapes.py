"""The adjoint of batch plans in every shape of tile that the plan's size can choose, at every compiled
support, with and without the illumination model, against the FP64 oracle.  Which shape a plan takes is
asked of the library, so that a change of the rule cannot leave a shape untested unnoticed.

Blocks of neighbouring points converge, so that tiles are full and their wavefronts contend for the LDS
tiles; others are empty.  The frames repeat every 32 columns, so a point matches at its own place and any
number of repeats away: most points get flow zero, some two repeats, whose dI1 patches lie further off
than a tile reaches; patches hang over the frame's edges.  The illumination model's frames match exactly
(gain 1, offset 0, every residual zero: its fixed point) and have fine texture, as its four unknowns need;
the plain model's have noise and flows a little off, and residuals within the inner threshold (a pixel on
a threshold takes either band, and tiles have nothing to do with bands).  Bar: relative L2 <= 1e-4 on dI0 and on dI1 of every pair, the bar of every adjoint test."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf
from paper_1901_09971_amd import _lib, synth

pytestmark = pytest.mark.gpu
REPEAT = 32


class AdjPair(ctypes.Structure):  # the library's AdjPair
    _fields_ = ([(n, ctypes.c_int64) for n in ("I0", "I1", "pitch0", "pitch1", "g0", "g1", "gpitch0", "gpitch1")]
                + [(n, ctypes.c_int32) for n in ("W", "H")] + [("tile_first", ctypes.c_int64)]
                + [(n, ctypes.c_int32) for n in ("nx", "ny", "tx", "ty", "w0", "h0", "w1", "h1")])


def _tile_shape(nx, ny, support, window, stride, n):
    """(tx, ty) of a pair of nx x ny points in a plan of n, None where it takes no tiles."""
    f = getattr(_lib.lib(), "_ZN3dgf18adjoint_tile_shapeERNS_7AdjPairEiiiiil")
    f.argtypes, f.restype = [ctypes.POINTER(AdjPair)] + 5 * [ctypes.c_int32] + [ctypes.c_int64], None
    p = AdjPair()
    f(p, nx, ny, support, window, stride, n)
    return (p.tx, p.ty) if p.w0 else None


@pytest.mark.parametrize("illum", [False, True])
@pytest.mark.parametrize("support,window,stride,points,shape", [
    (5, 3, 1, 32768, (8, 4)), (5, 9, 1, 262144, (16, 8)), (7, 9, 1, 65536, (8, 8)), (7, 3, 2, 262144, (16, 8)),
    (9, 3, 1, 16384, (4, 4)), (9, 9, 2, 65536, (8, 8)), (9, 9, 3, 262144, (16, 8)), (11, 3, 2, 16384, (4, 4)),
    (11, 9, 1, 262144, (16, 8)), (15, 9, 1, 16384, (4, 4)), (15, 9, 3, 32768, (8, 4)), (15, 9, 2, 262144, (16, 8)),
    (21, 9, 3, 16384, (4, 4)), (21, 9, 2, 32768, (8, 4)), (21, 9, 4, 65536, (8, 8)), (21, 9, 2, 262144, (16, 8)),
])
def test_tile_shape_against_oracle(support, window, stride, points, shape, illum):
    rng = np.random.default_rng(support + 100 * stride + window + 1000 * illum)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    f64 = lambda a: np.nan_to_num(np.asarray(a, np.float64))
    # two pairs of uneven size, about two thirds and one third of the points and a few more
    grids = [(int((points * 0.9) ** 0.5) + 1, int(points * 0.67 / (points * 0.9) ** 0.5) + 3),
             (int(points * 0.34 / (points * 0.2) ** 0.5) + 2, int((points * 0.2) ** 0.5) + 2)]
    made = []
    for nx, ny in grids:
        W, H = (nx - 1) * stride + window + stride // 2, (ny - 1) * stride + window
        I0 = np.rint(np.tile(synth.smoothed_noise(rng, REPEAT, H, 1.0 if illum else 2.0), (1, W // REPEAT + 1))[:, :W])
        I1 = np.rint(np.clip(I0 + (0.0 if illum else 0.5) * rng.normal(size=I0.shape), 0, 255))
        P = oracle.detect(I0.astype(np.uint8), window, stride)[0].astype(np.float32)
        assert len(P) == nx * ny
        blocks = rng.uniform(size=(ny // 20 + 1, nx // 24 + 1)) < 0.25
        blocks[0, 0] = True
        on = np.kron(blocks, np.ones((20, 24), bool))[:ny, :nx].ravel()
        r = support // 2 + 2
        dx = np.where(rng.uniform(size=len(P)) < 0.2, 2 * REPEAT, 0) * np.where(P[:, 0] < W / 2, 1, -1)
        moved = P[:, 0] + dx
        ok = (dx == 0) | ((moved >= r) & (moved < W - r) & (P[:, 0] >= r) & (P[:, 0] < W - r))
        st = np.where(on & ok & (rng.uniform(size=len(P)) < 0.95), 0, 1).astype(np.uint8)
        u = np.stack([dx, 0 * dx], 1) + (0.0 if illum else 0.02) * rng.normal(size=P.shape)
        u = np.where((st == 0)[:, None], u, np.nan).astype(np.float32)
        made.append((I0, I1, P, u, st, rng.normal(size=P.shape).astype(np.float32)))
    n = sum(nx * ny for nx, ny in grids)
    assert [_tile_shape(nx, ny, support, window, stride, n) for nx, ny in grids] == [shape, shape]
    plan = dgf.Batch([(dev(m[0].astype(np.uint8)), dev(m[1].astype(np.uint8)), window, stride) for m in made], 1,
                     support, 1, opts=dgf.TrackOpts(illum=illum))
    assert plan.num_points == n
    cat = lambda k: dev(np.concatenate([m[k] for m in made]))
    _, views = plan.backward(cat(5), points=cat(2), flow=cat(3), status=cat(4),
                             illum=torch.zeros_like(cat(3)) if illum else None)
    torch.cuda.synchronize()
    for (I0, I1, P, u, st, df), got in zip(made, views):
        conv = st == 0
        assert conv.sum() > 300 and (np.abs(f64(u)[:, 0]) > REPEAT).sum() > 20
        args = [f64(I0), f64(I1), f64(P)[conv], support, f64(u)[conv]]
        if illum:
            ref = oracle.track_grad_illum(*args, f64(0 * u)[conv], st[conv], f64(df)[conv])
        else:
            ref = oracle.track_grad(*args, st[conv], f64(df)[conv])
        for g, o in zip(got, ref):
            rel = np.linalg.norm(g.cpu().numpy() - o) / np.linalg.norm(o)
            print(f"\ns{support} w{window} stride {stride} {'IM ' if illum else ''}tiles {shape} converged {conv.sum()} "
                  f"of {len(P)} rel {rel:.1e}", flush=True)
            assert rel <= 1e-4
    plan.close()


@pytest.mark.parametrize("illum", [False, True])
@pytest.mark.parametrize("support", [5, 9, 21])
def test_few_points_of_a_tile(support, illum):
    """One to a dozen converged points in a tile, around the number from which on the LDS tiles are used."""
    rng = np.random.default_rng(support + illum)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    W, H, window, stride = 301, 259, 3, 1
    I0 = np.rint(synth.smoothed_noise(rng, W, H, 1.0 if illum else 2.0))
    I1 = I0 if illum else np.rint(np.clip(I0 + 0.5 * rng.normal(size=I0.shape), 0, 255))
    P = oracle.detect(I0.astype(np.uint8), window, stride)[0].astype(np.float32)
    nx, ny = W - window + 1, H - window + 1
    tx, ty = _tile_shape(nx, ny, support, window, stride, nx * ny)
    ky, kx = np.divmod(np.arange(nx * ny), nx)
    tile = (ky // ty) * 1000 + kx // tx
    share = (tile * 7 % 13) / (tx * ty)  # 0 to 12 points of every tile
    st = np.where(rng.uniform(size=len(P)) < share, 0, 2).astype(np.uint8)
    per_tile = np.unique(tile[st == 0], return_counts=True)[1]
    assert per_tile.min() == 1 and per_tile.max() > 10 and all((per_tile == k).sum() > 3 for k in range(4, 9))
    u = (0.0 if illum else 0.02) * rng.normal(size=P.shape).astype(np.float32)
    df = rng.normal(size=P.shape).astype(np.float32)
    plan = dgf.Batch([(dev(I0.astype(np.uint8)), dev(I1.astype(np.uint8)), window, stride)], 1, support, 1,
                     opts=dgf.TrackOpts(illum=illum))
    _, views = plan.backward(dev(df), points=dev(P), flow=dev(u), status=dev(st),
                             illum=torch.zeros((len(P), 2), device="cuda") if illum else None)
    torch.cuda.synchronize()
    c, f64 = st == 0, lambda a: np.asarray(a, np.float64)
    args = [f64(I0), f64(I1), f64(P)[c], support, f64(u)[c]]
    ref = oracle.track_grad_illum(*args, f64(0 * u)[c], st[c], f64(df)[c]) if illum else oracle.track_grad(*args, st[c], f64(df)[c])
    for g, o in zip(views[0], ref):
        rel = np.linalg.norm(g.cpu().numpy() - o) / np.linalg.norm(o)
        print(f"s{support} {'IM ' if illum else ''}tiles {(tx, ty)} converged {c.sum()} rel {rel:.1e}", flush=True)
        assert rel <= 1e-4
    plan.close()
