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


def test_calls_on_one_handle_keep_their_gradients(gpu_lib):
    """Backward passes of one handle on three streams, each with its own gradient
    (8 shots: each call adds one number per weight, so the sums have one order)."""
    import torch
    n = 8
    (dem,), det, w, ws, gen = _setup(gpu_lib, 1, n)
    gs = [torch.randn((1, n, dem.cols), generator=gen, device="cuda") for _ in range(3)]

    def grads(streams):
        out = [torch.zeros_like(w) for _ in gs]
        torch.cuda.synchronize()
        for _ in range(8):
            for g, gw, s in zip(gs, out, streams):
                dem.wbp_backward(w, 1, det, n, g, gw, ws, stream=s.cuda_stream)
        torch.cuda.synchronize()
        return out

    one = torch.cuda.current_stream()
    for a, b in zip(grads([one] * 3), grads([torch.cuda.Stream() for _ in gs])):
        assert int((a != 0).sum()) > 0 and torch.equal(a, b)


def test_forward_calls_on_one_handle_keep_their_weights(gpu_lib):
    import torch
    n, T = 200, 3
    (dem,), det, w, _, gen = _setup(gpu_lib, 1, n, T)
    ws = [w * f for f in (1.0, 0.5, 0.25)]

    def outs(streams):
        o = [(torch.empty((T, n, dem.cols), device="cuda"),
              torch.empty(dem.wbp_workspace_size(T, n), dtype=torch.uint8, device="cuda")) for _ in ws]
        torch.cuda.synchronize()
        for x, (llr, space), s in zip(ws, o, streams):
            dem.wbp_forward(x, T, det, n, llr, space, stream=s.cuda_stream)
        torch.cuda.synchronize()
        return [llr for llr, _ in o]

    one = torch.cuda.current_stream()
    for a, b in zip(outs([one] * 3), outs([torch.cuda.Stream() for _ in ws])):
        assert torch.equal(a, b)


@pytest.mark.parametrize("in_device_memory", [False, True], ids=["lds", "device-memory"])
def test_captured_pass_beside_eager_calls(gpu_lib, in_device_memory):
    """A captured forward and backward pass gives the eager call's numbers at every
    replay, with other weights' eager calls of the same handle between the replays.
    Its gradient adds up the same numbers in another order: n terms, so n * 2^-24 of
    the sum of their magnitudes, which n equal shots make n times one shot's (2e-5
    for n = 300, as 300 * 2^-24 = 1.8e-5)."""
    import torch
    t, n = gpu_lib, 300
    (dem,), det, w, ws, gen = _setup(t, 1, n)
    det.copy_(-(det[:, :1] & 1).expand_as(det))              # shot 0 in every bit
    g = torch.randn((1, 1, dem.cols), generator=gen, device="cuda").expand(1, n, -1).contiguous()
    llr, gw = torch.empty((1, n, dem.cols), device="cuda"), torch.zeros_like(w)
    t.wbp_global_state(in_device_memory)
    try:
        def both(x, out, grad):
            dem.wbp_forward(x, 1, det, n, out, ws)
            dem.wbp_backward(x, 1, det, n, g, grad, ws)

        w2, llr2, gw2 = 0.5 * w, torch.empty_like(llr), torch.zeros_like(w)
        want_llr, want = torch.empty_like(llr), torch.zeros_like(w)
        both(w2, llr2, gw2)
        both(w, want_llr, want)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            both(w, llr, gw)
        for _ in range(3):
            gw.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(llr, want_llr)
            assert int((want != 0).sum()) > 0
            assert bool(((gw.double() - want.double()).abs() <= 2 * 2e-5 * want.double().abs()).all())
            both(w2, llr2, gw2.zero_())
            torch.cuda.synchronize()
    finally:
        t.wbp_global_state(False)
