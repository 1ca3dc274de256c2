"""Weight-gradient calls that overlap in time.

dLoss/dw is accumulated into the caller's buffer, so calls on several streams (and
DEM handles) may add to one gradient.  One iteration, so that a call's shots
contribute known numbers: every call's own result is computed alone first, and the
sum of N calls in any order is within N half ulps of the sum of the magnitudes
(N = 32: 32 * 2^-24 = 1.9e-6, so 2e-6).
"""
import pytest

from workloads import TELEPORT, bb

pytestmark = pytest.mark.gpu

SPEC = bb("bb144", TELEPORT, 4, 3, 1e-3, 1e-2)


def _setup(t, handles, n, T=1):
    import torch
    c = t.Circuit(SPEC)
    det, obs = c.alloc_outputs(n)
    c.sample(5, 0, 0, n, det, obs)
    dems = [t.DEM(c) for _ in range(handles)]
    dem = dems[0]
    gen = torch.Generator(device="cuda").manual_seed(3)
    w = torch.rand((T, dem.edges), generator=gen, device="cuda") + 0.5
    llr = torch.empty((T, n, dem.cols), device="cuda")
    ws = torch.empty(dem.wbp_workspace_size(T, n), dtype=torch.uint8, device="cuda")
    dem.wbp_forward(w, T, det, n, llr, ws)
    return dems, det, w, ws, gen


def test_handles_add_to_one_gradient(gpu_lib):
    """Few shots (one row of blocks sums them) of two handles on two streams."""
    import torch
    n, calls = 8, 32
    dems, det, w, ws, gen = _setup(gpu_lib, 2, n)
    gs = [torch.randn((1, n, dems[0].cols), generator=gen, device="cuda") for _ in range(2)]
    alone = []
    for dem, g in zip(dems, gs):
        gw = torch.zeros_like(w)
        dem.wbp_backward(w, 1, det, n, g, gw, ws)
        alone.append(gw.double())
    total = torch.zeros_like(w)
    streams = [torch.cuda.Stream() for _ in dems]
    torch.cuda.synchronize()
    for _ in range(calls // 2):
        for dem, g, s in zip(dems, gs, streams):
            dem.wbp_backward(w, 1, det, n, g, total, ws, stream=s.cuda_stream)
    torch.cuda.synchronize()
    want = sum(alone) * (calls // 2)
    size = sum(a.abs() for a in alone) * (calls // 2)
    assert int((want != 0).sum()) > 0
    assert bool(((total.double() - want).abs() <= 2e-6 * size).all())
