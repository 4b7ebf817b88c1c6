"""The dense interpolation at the limits of its parameters and surroundings: no seed at all with both key
forms of the relaxation (distances beyond the fast form's range come with a large kappa on a large
frame); calls side by side on several streams, whose grids are not resident at once; a frame of more
tiles than the chip holds whose distances cross all its rows of tiles."""
import numpy as np
import pytest
import torch

import paper_1901_09971_amd as dgf

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
