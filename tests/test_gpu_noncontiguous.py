"""Non-contiguous points, flows and statuses give what their contiguous copies give (the binding makes the
copies itself, and they have to outlive one another until the call is made)."""
import numpy as np
import pytest
import torch

import paper_1901_09971_amd as dgf
from paper_1901_09971_amd import synth

pytestmark = pytest.mark.gpu


def _inputs():
    I0, I1, _ = synth.noise_translation_pair(256, 160, seed=4, dtype="f32")
    t0, t1 = torch.from_numpy(I0).cuda(), torch.from_numpy(I1).cuda()
    u8 = t0.round().clamp(0, 255).to(torch.uint8)
    P, sel = dgf.detect(u8, 9, 4, return_sel=True)
    flow, st = dgf.track(t0, t1, P, 3, 9, 20)
    return t0, t1, u8, P, sel, flow, st


def _apart(t):
    """The same values at every second row of a larger tensor."""
    big = torch.full((2 * t.shape[0], *t.shape[1:]), 7, dtype=t.dtype, device=t.device)
    big[::2] = t
    assert not big[::2].is_contiguous()
    return big[::2]


@pytest.mark.parametrize("run", ["epic", "async"])
def test_interpolation(run):
    _, _, u8, P, _, flow, st = _inputs()
    call = dgf.epic if run == "epic" else dgf.epic_async
    want = call(u8, P, flow, st, return_aux=True)[-1]
    got = call(u8, _apart(P), _apart(flow), _apart(st), return_aux=True)[-1]
    torch.cuda.synchronize()
    for k in want:
        assert torch.equal(got[k].view(torch.int32), want[k].view(torch.int32)), k


def test_gradients():
    t0, t1, u8, P, sel, flow, st = _inputs()
    df = torch.randn(flow.shape, generator=torch.Generator().manual_seed(1)).cuda()
    out = []
    for f in (lambda t: t, _apart):
        d0, d1, dp, dd = torch.zeros_like(t0), torch.zeros_like(t1), torch.empty_like(P), torch.zeros_like(t0)
        dgf.track_backward(t0, t1, f(P), 9, f(flow), f(st), f(df), d0, d1, dpoints=dp)
        dgf.detect_backward(u8, 9, 4, f(sel), f(df), dd)
        out.append((d0, d1, dp, dd))
    torch.cuda.synchronize()
    for a, b in zip(*out):  # (sums of atomics in any order)
        assert torch.allclose(a, b, rtol=1e-5, atol=1e-5 * float(a.abs().max()))
