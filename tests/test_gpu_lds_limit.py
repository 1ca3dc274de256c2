"""DEMs whose BP state only just fits, or just exceeds, a compute unit's LDS.

A team's run tables take LDS too, more of it the more waves the team has, so these
DEMs may fit for a few waves and not for sixteen.  Whatever is chosen, decoding
succeeds with the default shape and with any team size asked for, alone and in a
plan, and gives the device-memory kernel's outputs bit for bit.
"""
import pytest

from workloads import NLCNOT, TELEPORT, bb, sc

pytestmark = pytest.mark.gpu

CASES = [("bb36-nlcnot-34", bb("bb36", NLCNOT, 34, 34, 1e-3, 1e-2)),
         ("sc9-nlcnot-30", sc(9, NLCNOT, 30, 30, 1e-3, 1e-2)),
         ("sc9-teleport-29", sc(9, TELEPORT, 29, 29, 1e-3, 1e-2))]


@pytest.mark.parametrize("name,spec", CASES, ids=[c[0] for c in CASES])
def test_state_at_the_lds_limit(gpu_lib, name, spec):
    import torch
    t = gpu_lib
    shots, T = 100, 6
    c = t.Circuit(spec)
    dem = t.DEM(c)
    det, obs = c.alloc_outputs(shots)
    c.sample(5, 0, 0, shots, det, obs)

    def run(**kw):
        o = dict(llr=torch.zeros((shots, dem.cols), dtype=torch.float32, device="cuda"),
                 iters=torch.zeros(shots, dtype=torch.int32, device="cuda"),
                 flags=torch.zeros(shots, dtype=torch.uint8, device="cuda"))
        pred = torch.zeros_like(obs)
        dem.decode(det, shots, pred, max_iter=T, use_osd=False, **o, **kw)
        torch.cuda.synchronize()
        return dict(o, pred=pred)

    ref = run(bp_global_state=1)
    w = torch.ones((T, dem.edges), device="cuda")
    for kw in (dict(), dict(bp_threads=1024), dict(bp_threads=512), dict(bp_threads=64), dict(weights=w)):
        got = run(**kw)
        for k in ref:
            assert torch.equal(got[k], ref[k]), (name, kw, k)


def test_plan_at_the_lds_limit(gpu_lib):
    """Beside a smaller DEM, whose team takes the size of the larger one's."""
    import torch
    t = gpu_lib
    specs = [CASES[0][1], sc(5, NLCNOT, 5, 5, 1e-3, 1e-2)]
    B, T = 4096, 6
    circuits = [t.Circuit(s) for s in specs]
    dems = [t.DEM(c) for c in circuits]
    plan = t.Plan([(c, d, t.make_cfg(max_iter=T, use_osd=False), 7, i) for i, (c, d) in enumerate(zip(circuits, dems))],
                  B, use_graph=True)
    plan.run(1)
    for i, (c, d) in enumerate(zip(circuits, dems)):
        det, obs = c.alloc_outputs(B)
        c.sample(7, i, 0, B, det, obs)
        pred = torch.zeros_like(obs)
        d.decode(det, B, pred, max_iter=T, use_osd=False, bp_global_state=1)
        ne, _, _ = t.logical_error_rate(pred, obs, c.num_observables, B)
        r = plan.result(i)
        assert r["shots"] == B and r["errors"] == ne
