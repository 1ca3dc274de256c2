"""Weight gradients of more shots than the backward pass holds rows for.

One iteration, every shot the same: the per-shot gradients are identical, so
the call's result is the shot count times that of one shot.  FP32 sums of equal
terms: at most 3 + 280 + 16 additions meet one result (runs of 8 shots, the runs
of a thread, the threads of an edge and the rounds), each off by half an ulp:
300 * 2^-24 = 1.8e-5, so 2e-5 relative.
"""
import pytest

from workloads import TELEPORT, bb, sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spec,shots", [(bb("bb144", TELEPORT, 4, 3, 1e-3, 1e-2), 26000), (sc(3, rb=3), 1), (sc(3, rb=3), 4097)],
                         ids=["two-rounds", "one-shot", "small-graph"])
def test_rows_of_equal_shots_sum_up(gpu_lib, spec, shots):
    import torch
    t = gpu_lib
    c = t.Circuit(spec)
    dem = t.DEM(c)
    det, obs = c.alloc_outputs(64)
    c.sample(5, 0, 0, 64, det, obs)
    one = -(det & 1)                                 # shot 0 in every bit
    g = torch.randn(dem.cols, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    w = torch.rand((1, dem.edges), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda") + 0.5

    def grad(n):
        d = one[:, :1].expand(-1, (n + 63) // 64).contiguous()
        ws = torch.empty(dem.wbp_workspace_size(1, n), dtype=torch.uint8, device="cuda")
        llr = torch.empty((1, n, dem.cols), device="cuda")
        gw = torch.zeros_like(w)
        dem.wbp_forward(w, 1, d, n, llr, ws)
        assert torch.equal(llr, llr[:, :1].expand(-1, n, -1))
        dem.wbp_backward(w, 1, d, n, g.expand(1, n, -1).contiguous(), gw, ws)
        return gw

    ref = grad(1).double() * shots
    assert int((ref != 0).sum()) > 0
    assert bool(((grad(shots).double() - ref).abs() <= 2e-5 * ref.abs()).all())
