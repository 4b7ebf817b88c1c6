"""Detection where its forms change: windows around each count of dwords per row, strides on both
sides of the row sums, grids on both sides of a filled chip, tiles of 8 and of 16 windows, and rows
that start at every byte of a dword.

The sums are whole numbers, so the selection is exact.  A coordinate is x0 + M / S in FP32 with M
and S rounded once: four roundings of 2^-24, each of at most the image's side."""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_09971_amd as dgf

pytestmark = pytest.mark.gpu


def _check(pts, sel, img, window, stride):
    want, osel, _ = oracle.detect(img, window, stride)
    err = np.abs(pts.cpu().numpy().astype(np.float64) - want).max()
    print(f"{img.shape[1]}x{img.shape[0]} window={window} stride={stride} n={len(want)} err={err:.1e}", flush=True)
    assert err <= 4 * 2.0**-24 * max(img.shape)
    if sel is not None:
        assert np.array_equal(sel.cpu().numpy(), osel)


def _frame(W, H, seed):
    rng = np.random.default_rng(seed)
    img = rng.integers(0, 256, size=(H, W), dtype=np.uint8)
    img[: H // 4] = 0  # a negative centroid over an empty sum
    img[-(H // 4):] = 255
    return img


@pytest.mark.parametrize("window", [1, 2, 3, 4, 5, 7, 8, 9, 10, 12, 13, 16, 31, 100])
def test_windows_and_strides(window):
    for stride in (1, 2, 3, 4, 5, 8, 11):
        W, H = window + 17 * stride + window % 3, window + 33 * stride + 1
        _check(*dgf.detect(torch.from_numpy(_frame(W, H, window)).cuda(), window, stride, return_sel=True),
               _frame(W, H, window), window, stride)
    img = _frame(window, window, 7)  # a single window
    _check(*dgf.detect(torch.from_numpy(img).cuda(), window, 1, return_sel=True), img, window, 1)


@pytest.mark.parametrize("window,stride", [(3, 1), (5, 2), (4, 3)])
def test_grids_that_fill_the_chip(window, stride):
    # 256 tiles of 16 x 32 (16 x 16 at stride 3) windows, and one row of them less
    high = 32 if stride < 3 else 16
    for ny in (16 * high, 15 * high):
        W, H = window + stride * 255, window + stride * (ny - 1)
        img = _frame(W, H, ny)
        _check(*dgf.detect(torch.from_numpy(img).cuda(), window, stride, return_sel=True), img, window, stride)


@pytest.mark.parametrize("x", range(4))
def test_rows_at_every_byte(x):
    big = _frame(301, 90, x)
    img = torch.from_numpy(big).cuda()[3:83, x:x + 150]
    for window, stride in ((9, 2), (9, 5), (7, 8)):
        _check(*dgf.detect(img, window, stride, return_sel=True), np.ascontiguousarray(big[3:83, x:x + 150]), window, stride)


def test_plan_and_fused_front_end():
    sizes = [(3, 1), (3, 2), (5, 2), (9, 1), (9, 3), (9, 8), (12, 3), (13, 2), (21, 8), (16, 4)]
    frames = [(torch.from_numpy(_frame(130 + 7 * k, 90 + 5 * k, k)).cuda(),
               torch.from_numpy(_frame(130 + 7 * k, 90 + 5 * k, 50 + k)).cuda()) for k in range(len(sizes))]
    b = dgf.Batch([(a, c, w, s) for (a, c), (w, s) in zip(frames, sizes)], 3, 9, 4)
    pts = b.front()
    for k, ((a, c), (w, s)) in enumerate(zip(frames, sizes)):
        _check(pts[b.offsets[k]:b.offsets[k + 1]], None, a.cpu().numpy(), w, s)
        ws = torch.empty(dgf.track_workspace_bytes(a.shape[1], a.shape[0], 3, 0), dtype=torch.uint8, device="cuda")
        fused = torch.empty((dgf.detect_count(a.shape[1], a.shape[0], w, s), 2), device="cuda")
        dgf.detect_pyramids(a, c, w, s, 3, ws, fused)
        one = dgf.detect(a, w, s)
        assert torch.equal(one, pts[b.offsets[k]:b.offsets[k + 1]]) and torch.equal(one, fused)
