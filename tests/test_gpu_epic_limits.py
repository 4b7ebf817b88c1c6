"""The dense interpolation at the limits of its parameters and surroundings: no seed at all with both key
forms of the relaxation (distances beyond the fast form's range come with a large kappa on a large
frame); calls side by side on several streams, whose grids are not resident at once; a frame of more
tiles than the chip holds whose distances cross all its rows of tiles; long paths through a resident
grid, whose tiles wait for them; half-distances and step costs
far from the defaults, whose neighbour searches take no longer than the defaults'; seeds denser than the seed
graph's tables hold, at every height of its tiles."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf
from paper_1901_09971_amd import synth
from test_gpu_epic import _run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("run", ["epic", "async"])
@pytest.mark.parametrize("W,H,kappa", [(700, 520, 8), (700, 520, 1 << 20), (2100, 1900, 1 << 20), (65, 33, 1 << 20)])
def test_no_seed(W, H, kappa, run):
    rng = np.random.default_rng(W + H)
    n = 7
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    I0 = t(rng.integers(0, 256, (H, W)).astype(np.uint8))
    P = t(np.stack([rng.uniform(0, W - 1, n), rng.uniform(0, H - 1, n)], 1).astype(np.float32))
    F, st = torch.ones_like(P), torch.ones(n, dtype=torch.uint8, device="cuda")
    call = dgf.epic if run == "epic" else dgf.epic_async
    out = call(I0, P, F, st, opts=dgf.EpicOpts(k=4, kappa=kappa), return_aux=True)
    torch.cuda.synchronize()
    if run == "async":
        assert int(out[1].item()) == 0
    g = out[-1]
    assert torch.all(g["labels"] == -1) and torch.all(g["dist"] == -1)  # (uint32 0xFFFFFFFF)
    assert torch.all(torch.isnan(out[0])) and torch.all(torch.isnan(g["model"]))
    assert torch.all(g["nbr"] == -1) and torch.all(g["nbr_dist"] == -1)


@pytest.mark.parametrize("W,H", [(1400, 700), (1600, 900), (2048, 1024)])
def test_async_calls_side_by_side(W, H):
    """One seed in a corner, so that its distances cross every tile, on four streams at a time: the
    relaxation grids keep each other from being resident, and tiles leave to make room for those that
    have not started.  Every call settles within the default number of launches all the same."""
    rng = np.random.default_rng(W)
    I0 = torch.from_numpy(rng.integers(0, 256, (H, W)).astype(np.uint8)).cuda()
    P = torch.tensor([[W - 3.0, H - 3.0]], device="cuda")
    F, st = torch.tensor([[0.5, -1.0]], device="cuda"), torch.zeros(1, dtype=torch.uint8, device="cuda")
    ref, want = dgf.epic(I0, P, F, st, return_aux=True)
    streams, calls = [torch.cuda.Stream() for _ in range(4)], 8
    torch.cuda.synchronize()
    out = []
    for _ in range(calls):
        for s in streams:
            with torch.cuda.stream(s):
                out.append(dgf.epic_async(I0, P, F, st, return_aux=True))
    torch.cuda.synchronize()
    statuses = [int(status.item()) for _, status, _ in out]
    print(f"{W}x{H}: {sum(s != 0 for s in statuses)} of {len(statuses)} unsettled", flush=True)
    assert not any(statuses)
    for dense, _, aux in out:
        assert torch.equal(dense, ref) and torch.equal(aux["dist"], want["dist"])


@pytest.mark.parametrize("edge", ["lower", "upper"])
def test_async_default_launches_cross_a_wide_frame(edge):
    W, H = 8192, 740
    rng = np.random.default_rng(5)
    I0 = torch.from_numpy(rng.integers(0, 256, (H, W)).astype(np.uint8)).cuda()
    x = torch.arange(4.0, W - 4, 40, device="cuda")
    P = torch.stack([x, torch.full_like(x, H - 3.0 if edge == "lower" else 2.0)], 1).contiguous()
    F, st = torch.ones_like(P), torch.zeros(len(x), dtype=torch.uint8, device="cuda")
    _, want = dgf.epic(I0, P, F, st, return_aux=True)
    _, status, aux = dgf.epic_async(I0, P, F, st, return_aux=True)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert torch.equal(aux["labels"], want["labels"]) and torch.equal(aux["dist"], want["dist"])


@pytest.mark.parametrize("k,kappa,h,n", [(128, 8, 1 << 20, 900), (64, 1, 1 << 24, 900), (32, 1 << 14, 1 << 20, 400),
                                         (16, 1 << 20, 1 << 24, 60), (40, 7, 1 << 12, 12), (128, 65535, 1 << 18, 900)])
def test_large_half_distances(k, kappa, h, n):
    # few seeds: edges beyond the range that bounds the batches; many: ordinary ones
    rng = np.random.default_rng(k + n)
    W, H = 190, 120
    I0 = (rng.integers(0, 40, (H, W)) + np.where(np.arange(W)[None, :] > 90, 100, 0)).astype(np.uint8)
    P = np.stack([rng.uniform(0, W - 1, n), rng.uniform(0, H - 1, n)], 1)
    st = (rng.uniform(size=n) < 0.1).astype(np.uint8)
    _run_both(I0, P, rng.normal(size=(n, 2)), st, dgf.EpicOpts(k=k, kappa=kappa, half_dist=h))


def test_large_half_distance_takes_no_longer():
    """The neighbours and the size of the searches are about those of the default half-distance, so the
    time is too (0.97 to 1.05 of it over all half-distances; searches that settle one node a batch took 2.9
    times as long)."""
    rng = np.random.default_rng(3)
    I0 = torch.from_numpy(np.clip(np.rint(synth.smoothed_noise(rng, 640, 480, 2.0)), 0, 255).astype(np.uint8)).cuda()
    P = dgf.detect(I0, 9, 5)
    F, st = torch.ones_like(P), torch.zeros(len(P), dtype=torch.uint8, device="cuda")

    def ms(h):
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                dgf.epic_async(I0, P, F, st, opts=dgf.EpicOpts(half_dist=h))
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    ms(64)
    base, far = ms(64), ms(1 << 20)
    print(f"half-distance 2^20 takes {far / base:.2f} of 64", flush=True)
    assert far < 1.7 * base


@pytest.mark.parametrize("W,H,kappa", [(2048, 1024, 8), (1242, 375, 1 << 20), (8000, 4, 8), (4, 8000, 8)])
def test_long_paths_settle_in_one_launch(W, H, kappa):
    """One seed in a corner of a frame that fits the chip: the far tiles wait for the front through the
    whole of the first launch, and the second finds nothing to change."""
    rng = np.random.default_rng(W)
    I0 = torch.from_numpy(rng.integers(0, 256, (H, W)).astype(np.uint8)).cuda()
    P = torch.tensor([[W - 2.0, H - 2.0]], device="cuda")
    F, st, opts = torch.ones_like(P), torch.zeros(1, dtype=torch.uint8, device="cuda"), dgf.EpicOpts(kappa=kappa)
    _, want = dgf.epic(I0, P, F, st, opts=opts, return_aux=True)
    _, status, aux = dgf.epic_async(I0, P, F, st, opts=opts, max_relax=2, return_aux=True)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and torch.equal(aux["dist"], want["dist"])


@pytest.mark.parametrize("W,H,step", [(255, 256, 6), (256, 256, 6), (301, 227, 2), (760, 700, 7), (1025, 513, 7)])
def test_graph_tiles(W, H, step):
    """Frames around the sizes at which the graph's tiles change height; a seed on every pixel of two
    rectangles, so that the tables of the tiles there run over, and every few pixels elsewhere."""
    rng = np.random.default_rng(W + step)
    I0 = rng.integers(0, 256, (H, W)).astype(np.uint8)
    on = np.zeros((H, W), bool)
    on[::step, ::step] = True
    on[40:110, 60:190] = True
    on[H - 20:, W - 70:] = True
    y, x = np.nonzero(on)
    P = np.stack([x, y], 1).astype(np.float32)
    F, st = rng.normal(size=P.shape).astype(np.float32), np.zeros(len(P), np.uint8)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    _, aux = dgf.epic(t(I0), t(P), t(F), t(st), opts=dgf.EpicOpts(k=8), return_aux=True)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in aux.items()}
    _, o = oracle.epic(I0, P.astype(np.float64), F.astype(np.float64), st, k=8, full=True)
    assert np.array_equal(g["labels"], o["L"])
    assert np.array_equal(g["nbr"], o["nb"])
    assert np.array_equal(g["nbr_dist"].view(np.uint32).astype(np.int64), np.where(o["nd"] < 0, 0xFFFFFFFF, o["nd"]))
