"""What the autotuner's choice is cached for."""
import pytest

from workloads import NLCNOT, sc

pytestmark = pytest.mark.gpu


def _launches(t, dem, det, n, **kw):
    """Kernel launches of one tmcs_autotune call, by kernel."""
    import torch
    t.timing_reset()
    t.timing_enable(True)
    cfg = t.autotune(dem, det, n, t.make_cfg(max_iter=7, use_osd=False, **kw))
    torch.cuda.synchronize()
    t.timing_enable(False)
    return {k: v[0] for k, v in t.timing_report().items()}, cfg


def test_choice_depends_on_shots_and_scaling(gpu_lib):
    t = gpu_lib
    c = t.Circuit(sc(3, NLCNOT, 2, 2, 4e-3, 2e-2))
    dem = t.DEM(c)
    n = 300 * 256
    det, obs = c.alloc_outputs(n)
    c.sample(1, 0, 0, n, det, obs)
    few, _ = c.alloc_outputs(64)
    few.copy_(det[:, :1])
    assert _launches(t, dem, few, 64)[0]
    assert _launches(t, dem, few, 64)[0] == {}
    # (the team size follows from the shots per compute unit, the kernel from alpha)
    assert _launches(t, dem, det, n)[0]
    assert _launches(t, dem, det, n - 64)[0] == {} == _launches(t, dem, det, n)[0]
    assert _launches(t, dem, few, 64, alpha=0.75)[0]

