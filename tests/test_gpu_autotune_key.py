"""What the autotuner's choice is cached for, and that no candidate is timed twice."""
import pytest

from workloads import MEMORY, NLCNOT, sc

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


@pytest.mark.parametrize("state,kernel,trials", [(0, "k_bp", 30), (1, "k_bp_dev", 60)], ids=["lds", "device-memory"])
def test_schedules_are_timed_where_they_differ(gpu_lib, state, kernel, trials):
    """5 team sizes, 2 teams per compute unit, 3 OSD shapes; 2 lane schedules only
    where the state is in device memory.  A warm-up and a timed run of each."""
    t = gpu_lib
    c = t.Circuit(sc(3, MEMORY, 2 + state, 0, 4e-3))
    dem = t.DEM(c)
    det, obs = c.alloc_outputs(128)
    c.sample(1, 0, 0, 128, det, obs)
    got, cfg = _launches(t, dem, det, 128, bp_global_state=state)
    assert got[kernel] == 2 * trials
    assert cfg.bp_sched in (1, 2)
