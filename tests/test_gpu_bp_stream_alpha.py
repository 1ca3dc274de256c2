"""BP that streams its state through LDS, with scalings other than 1.

alpha multiplies both minima of every check and iteration; the iterations it can be
run for without reaching infinity decide the kernel (few for a large alpha).  All
outputs equal the two-pass device-memory kernel's bit for bit.
"""
import pytest

from workloads import NLCNOT, sc

pytestmark = pytest.mark.gpu

# (scaling, iterations, kernel): |q| grows by at most 1 + (dv + 1) alpha an iteration
CASES = [(0.625, 20, "k_bp_stream"), (0.9, 30, "k_bp_stream"), (1e-6, 20, "k_bp_stream"), (50.0, 8, "k_bp_stream"),
         (50.0, 60, "k_bp_dev"), (1.0, 70, "k_bp_dev")]


@pytest.mark.parametrize("alpha,T,kernel", CASES, ids=["%g-%d" % c[:2] for c in CASES])
def test_streamed_state_scalings(gpu_lib, alpha, T, kernel):
    import torch
    t, shots = gpu_lib, 130
    c = t.Circuit(sc(15, NLCNOT, 15, 15, 1e-3, 1e-2))
    dem = t.DEM(c)
    det, obs = c.alloc_outputs(shots)
    c.sample(5, 0, 0, shots, det, obs)

    def run(name, **kw):
        o = dict(ehat=torch.zeros((shots, dem.cols), dtype=torch.uint8, device="cuda"),
                 llr=torch.zeros((shots, dem.cols), dtype=torch.float32, device="cuda"),
                 iters=torch.zeros(shots, dtype=torch.int32, device="cuda"),
                 flags=torch.zeros(shots, dtype=torch.uint8, device="cuda"), stats=t.new_stats())
        pred = torch.zeros_like(obs)
        t.timing_reset()
        t.timing_enable(True)
        dem.decode(det, shots, pred, max_iter=T, alpha=alpha, use_osd=False, **o, **kw)
        torch.cuda.synchronize()
        t.timing_enable(False)
        assert name in t.timing_report()
        return dict(o, pred=pred)

    ref, got = run("k_bp_dev", bp_global_state=1), run(kernel)
    for k in ref:
        assert torch.equal(got[k], ref[k]), (alpha, T, k)
