"""tmcs_decode captured in the caller's own graph after a warm-up of another kind.

A warm-up makes the handle's scratch; a capture of fewer shots may still want a
schedule for another team size or another BP kernel, and one with weights room for
their layout.  Every replay gives the eager call's predictions.
"""
import pytest

from workloads import MEMORY, NLCNOT, bb, sc

pytestmark = pytest.mark.gpu

# (circuit, shots of the warm-up, shots of the capture, settings of the capture)
CASES = [("fewer-shots", sc(5, NLCNOT, 5, 5, 2e-3, 1e-2), 70000, 640, {}),
         ("streamed-then-chunks", sc(11, NLCNOT, 11, 11, 1e-3, 1e-2), 2112, 130, {}),
         ("weights", sc(5, NLCNOT, 5, 5, 2e-3, 1e-2), 70000, 640, dict(weights=0.9)),
         ("weights-beyond-lds", sc(15, NLCNOT, 15, 15, 1e-3, 1e-2), 256, 64, dict(weights=0.9)),
         ("device-memory", sc(15, NLCNOT, 15, 15, 1e-3, 1e-2), 256, 64, dict(bp_global_state=1)),
         ("sweep", bb("bb144", MEMORY, 12, 0, 2e-3), 2112, 640, dict(osd_order=7))]


@pytest.mark.parametrize("name,spec,warm,shots,kw", CASES, ids=[c[0] for c in CASES])
def test_capture_after_a_warm_up_of_another_kind(gpu_lib, name, spec, warm, shots, kw):
    import torch
    t = gpu_lib
    T = 8
    c = t.Circuit(spec)
    dem, other = t.DEM(c), t.DEM(c)
    if "weights" in kw:
        kw = dict(weights=torch.full((T, dem.edges), kw["weights"], device="cuda"))
    det, obs = c.alloc_outputs(warm)
    c.sample(3, 0, 0, warm, det, obs)
    dem.decode(det, warm, torch.zeros_like(obs), max_iter=T)
    det, obs = c.alloc_outputs(shots)
    pred = torch.zeros_like(obs)
    batches = []
    for k in range(3):
        c.sample(3, 1 + k, 0, shots, det, obs)
        other.decode(det, shots, pred, max_iter=T, **kw)
        torch.cuda.synchronize()
        batches.append((det.clone(), pred.clone()))
    assert any(bool((p != 0).any()) for _, p in batches)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dem.decode(det, shots, pred, max_iter=T, **kw)
    for d, p in batches + batches[:1]:
        det.copy_(d)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(pred, p), name
        dem.decode(det, shots, pred.fill_(-1), max_iter=T, **kw)      # eager work between the replays
        assert torch.equal(pred, p)
