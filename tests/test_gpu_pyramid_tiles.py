"""Pyramids where their launches change: one to four levels per launch (each with tiles of its own
size), frames of a tile exactly and one pixel more or less, ranges that reach past one, two or all
four borders, rows that start at every byte, and float frames whose first level goes by itself.

uint8 levels are whole numbers, bit for bit the oracle's.  A float level's pixel is a sum of 25
products of positive weights whose sum is 1, with at most eight roundings on its way, at most four
levels deep: 32 x 2^-24 x 255 < 5e-4."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf
from paper_1901_09971_amd import _lib

pytestmark = pytest.mark.gpu

SIZES = [(32, 32), (33, 31), (31, 65), (64, 64), (65, 63), (129, 95), (3, 70), (70, 3), (4, 4), (200, 1), (163, 131)]


def _check(img, levels):
    rng = np.random.default_rng(levels)
    for x in range(4):
        big = rng.integers(0, 256, size=(img[1], img[0] + 8), dtype=np.uint8)
        a = np.ascontiguousarray(big[:, x:x + img[0]])
        ref = oracle.pyramid(a, levels)
        got = dgf.pyramid(torch.from_numpy(big).cuda()[:, x:x + img[0]], levels)
        for l in range(1, levels):
            assert np.array_equal(got[l].cpu().numpy(), ref[l]), (img, levels, x, l)
    f = rng.uniform(0, 255, size=(img[1], img[0])).astype(np.float32)
    ref = oracle.pyramid(f.astype(np.float64), levels)
    got = dgf.pyramid(torch.from_numpy(f).cuda(), levels)
    for l in range(1, levels):
        assert np.abs(got[l].cpu().numpy() - ref[l]).max() <= 32 * 2.0**-24 * 255, (img, levels, l)


@pytest.mark.parametrize("levels", [2, 3, 4, 5, 6])
def test_tiles_and_borders(levels):
    for size in SIZES:
        _check(size, levels)


@pytest.mark.parametrize("W,H", [(1024, 1024), (1025, 1024), (2050, 1100)])
def test_first_level_by_itself(W, H):
    _check((W, H), 4)


@pytest.mark.parametrize("dtype,shift", [(_lib.DGF_U8, 1), (_lib.DGF_U8, 3), (_lib.DGF_F32, 4)])
def test_destination_at_any_alignment(dtype, shift):
    rng = np.random.default_rng(shift)
    img = rng.integers(0, 256, size=(71, 133), dtype=np.uint8)
    t = torch.from_numpy(img).cuda()
    t = t.float() if dtype == _lib.DGF_F32 else t
    e = t.element_size()
    L = _lib.lib()
    im = _lib.DgfImage(t.data_ptr(), 133, 71, 133 * e, dtype)
    need = L.dgf_pyramid_layout(133, 71, 5, dtype, None, None)
    out = []
    for at in (0, shift):
        buf = torch.zeros(need + 64, dtype=torch.uint8, device="cuda")
        assert L.dgf_pyramid(ctypes.byref(im), 5, ctypes.c_void_p(buf.data_ptr() + at), need, None) == 0
        torch.cuda.synchronize()
        out.append(buf[at:at + need].cpu().numpy())
    assert np.array_equal(out[0], out[1])
