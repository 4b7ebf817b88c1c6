"""The float path's tiles: pyramid levels built several per launch equal the same levels built one at a
time, bit for bit, at sizes around the tiles' edges; and tracking float frames whose rows are pitched
views at every 4-byte offset (four-texel loads at any alignment, rows at the image's edges by the
clamped form) equals tracking contiguous copies, bit for bit, at every compiled lane layout."""
import numpy as np
import pytest
import torch

import paper_1901_09971_amd as dgf
from paper_1901_09971_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(1, 1), (2, 3), (1, 40), (65, 1), (63, 64), (64, 65), (129, 127), (640, 480), (333, 77)])
def test_levels_at_once_equal_one_at_a_time(W, H):
    rng = np.random.default_rng(W * 1000 + H)
    img = torch.from_numpy(rng.uniform(-300, 300, (H, W)).astype(np.float32)).cuda()
    at_once = dgf.pyramid(img, 7)
    level = img
    for l in range(1, 7):
        level = dgf.pyramid(level, 2)[1]
        assert torch.equal(at_once[l], level), (l, tuple(level.shape))


@pytest.mark.parametrize("support,lanes", [(5, 16), (7, 16), (9, 16), (9, 32), (11, 16), (15, 16), (15, 32), (21, 16),
                                           (21, 32), (21, 64)])
def test_pitched_float_frames(support, lanes):
    W, H = 117, 83
    I0, I1, _ = synth.noise_translation_pair(W, H, seed=support + lanes, dtype="f32")
    rng = np.random.default_rng(support)
    edge = np.array([(0, 0), (W - 1, 0), (0, H - 1), (W - 1, H - 1), (W - 1, 40), (W - 2.5, 7), (50, H - 1.25), (3, 3)])
    pts = np.concatenate([edge, rng.uniform(0, 1, (150, 2)) * (W - 1, H - 1)]).astype(np.float32)
    P = torch.from_numpy(pts).cuda()
    a, b = torch.from_numpy(I0).cuda(), torch.from_numpy(I1).cuda()
    try:
        dgf.set_tuning(support, 1, lanes, 1, 2)
        ref = dgf.track(a, b, P, 3, support, 8)
        for off in range(4):
            pa, pb = (torch.full((H, W + 9), 1e6, device="cuda")[:, off:off + W] for _ in range(2))
            pa.copy_(a)
            pb.copy_(b)
            got = dgf.track(pa, pb, P, 3, support, 8)
            for x, y in zip(ref, got):
                assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), off
    finally:
        default = 64 if support == 21 else 32 if support in (9, 15) else 16
        dgf.set_tuning(support, 1, default, 1, 2)
