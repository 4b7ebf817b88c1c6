"""Float frames of more than 2^20 pixels, whose first level has tiles of its own (32 output pixels): a tile
exactly and one or two source pixels more or less, and frames of a few rows or columns.  Tolerance: see
test_gpu_pyramid_tiles (at most eight roundings of a weighted mean, a level)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(1088, 1024), (1089, 1025), (1087, 1023), (1090, 1022), (17000, 65), (63, 17001)])
@pytest.mark.parametrize("levels", [2, 3])
def test_first_level(W, H, levels):
    f = np.random.default_rng(W + H).uniform(0, 255, size=(H, W + 3)).astype(np.float32)
    ref = oracle.pyramid(np.ascontiguousarray(f[:, 1:1 + W]).astype(np.float64), levels)
    got = dgf.pyramid(torch.from_numpy(f).cuda()[:, 1:1 + W], levels)
    for l in range(1, levels):
        assert got[l].shape == ref[l].shape
        assert np.abs(got[l].cpu().numpy() - ref[l]).max() <= 8 * l * 2.0**-24 * 255, l
