"""The geodesic partition of the dense interpolation where its tiles (62 x 32 pixels, four wavefronts of
eight rows) and its two key forms can go wrong: one pixel around a tile's size, single rows and
columns, few seeds (paths across many tiles), distances beyond the fast form's range (large kappa on a
large frame), and a frame with more tiles than the chip holds at once.  Cells and distances are exact
integers and compared bit for bit with the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,n,kappa,run", [
    (62, 32, 3, 8, "epic"), (63, 33, 3, 8, "epic"), (61, 31, 2, 8, "epic"), (124, 64, 1, 8, "epic"),
    (1, 300, 2, 8, "epic"), (300, 1, 2, 8, "epic"), (1, 1, 1, 8, "epic"), (187, 97, 5, 1, "epic"),
    (311, 129, 40, 8, "async"), (700, 520, 6, 1 << 20, "epic"), (1242, 375, 300, 1 << 20, "async"),
    (2500, 1100, 4000, 8, "epic"), (2500, 1100, 4000, 8, "async"),
])
def test_cells_and_distances(W, H, n, kappa, run):
    rng = np.random.default_rng(W * 7 + H + n)
    I0 = rng.integers(0, 256, (H, W)).astype(np.uint8)
    I0[rng.uniform(size=I0.shape) < 0.6] = 90  # flat stretches between textured pixels: many equal distances
    P = np.stack([rng.uniform(0, W - 1, n), rng.uniform(0, H - 1, n)], 1).astype(np.float32)
    F = rng.normal(size=(n, 2)).astype(np.float32)
    st = (rng.uniform(size=n) < 0.1).astype(np.uint8)
    st[0] = 0
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    opts = dgf.EpicOpts(k=4, kappa=kappa)
    call = dgf.epic if run == "epic" else dgf.epic_async
    out = call(t(I0), t(P), t(F), t(st), opts=opts, return_aux=True)
    torch.cuda.synchronize()
    if run == "async":
        assert int(out[1].item()) == 0
    g = {k: v.cpu().numpy() for k, v in out[-1].items()}
    _, o = oracle.epic(I0, P.astype(np.float64), F.astype(np.float64), st, k=4, kappa=kappa, h=64, full=True)
    assert np.array_equal(g["labels"], o["L"])
    assert np.array_equal(g["dist"].view(np.uint32).astype(np.int64), np.where(o["D"] < 0, 0xFFFFFFFF, o["D"]))


@pytest.mark.parametrize("W,H,step", [(64, 32, 1), (65, 33, 1), (130, 70, 1), (131, 67, 2), (63, 100, 3)])
def test_graph_of_dense_seeds(W, H, step):
    """A seed on every pixel (every second, every third): more touching cells in a 64 x 32 graph tile
    than its table of 1,024 holds, so part of them goes to the rows directly; neighbour lists and
    graph distances bit for bit."""
    rng = np.random.default_rng(W + H + step)
    I0 = rng.integers(0, 256, (H, W)).astype(np.uint8)
    y, x = np.mgrid[0:H:step, 0:W:step]
    P = np.stack([x.ravel(), y.ravel()], 1).astype(np.float32)
    F = rng.normal(size=P.shape).astype(np.float32)
    st = np.zeros(len(P), np.uint8)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    _, aux = dgf.epic(t(I0), t(P), t(F), t(st), opts=dgf.EpicOpts(k=16), return_aux=True)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in aux.items()}
    _, o = oracle.epic(I0, P.astype(np.float64), F.astype(np.float64), st, k=16, full=True)
    assert np.array_equal(g["labels"], o["L"])
    assert np.array_equal(g["nbr"], o["nb"])
    assert np.array_equal(g["nbr_dist"].view(np.uint32).astype(np.int64), np.where(o["nd"] < 0, 0xFFFFFFFF, o["nd"]))
