"""Weights of more iterations than a grid has rows of blocks (65535).

All weights are 0 but the last iteration's, so that BP moves at the last one only:
decoding and the training forward pass read those weights, or the posteriors stay
the priors.  Bit for bit against the device-memory kernel, which reads the weights
as they are given.
"""
import pytest

from workloads import MEMORY, sc

pytestmark = pytest.mark.gpu


def _dem(t, shots):
    c = t.Circuit(sc(3, MEMORY, 1, 0, 2e-2))
    dem = t.DEM(c)
    det, obs = c.alloc_outputs(shots)
    c.sample(5, 0, 0, shots, det, obs)
    return dem, det, obs


def test_decoder_weights(gpu_lib):
    import torch
    t, shots, T = gpu_lib, 64, 65537
    dem, det, obs = _dem(t, shots)
    w = torch.zeros((T, dem.edges), device="cuda")
    w[-1] = 0.75

    def run(**kw):
        o = dict(llr=torch.zeros((shots, dem.cols), dtype=torch.float32, device="cuda"),
                 iters=torch.zeros(shots, dtype=torch.int32, device="cuda"))
        dem.decode(det, shots, torch.zeros_like(obs), max_iter=T, weights=w, use_osd=False, **o, **kw)
        torch.cuda.synchronize()
        return o

    ref, got = run(bp_global_state=1), run()
    last = ref["iters"] == T
    assert bool(last.any()) and bool((ref["llr"][last] != ref["llr"][~last][:1]).any())
    assert torch.equal(ref["iters"], got["iters"]) and torch.equal(ref["llr"], got["llr"])


def test_training_weights(gpu_lib):
    import torch
    t, shots, T = gpu_lib, 3, 65537
    dem, det, obs = _dem(t, 64)
    w = torch.zeros((T, dem.edges), device="cuda")
    w[-1] = 0.75
    llr = torch.empty((T, shots, dem.cols), device="cuda")
    ws = torch.empty(dem.wbp_workspace_size(T, shots), dtype=torch.uint8, device="cuda")
    dem.wbp_forward(w, T, det, shots, llr, ws)
    one, ws1 = torch.empty((1, shots, dem.cols), device="cuda"), torch.empty(dem.wbp_workspace_size(1, shots),
                                                                          dtype=torch.uint8, device="cuda")
    dem.wbp_forward(w[-1:].contiguous(), 1, det, shots, one, ws1)          # from the priors, as the last iteration
    assert bool((llr[:-1] == llr[:1]).all()) and bool((llr[-1] != llr[0]).any())
    assert torch.equal(llr[-1:], one)
