"""The dense interpolation at the limits of its parameters: no seed at all with both key forms of the
relaxation (distances beyond the fast form's range come with a large kappa on a large frame)."""
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
