"""BP that streams its state through LDS, at the edges of its schedules.

Teams of one to sixteen waves (so tiles of 64 to 1024 checks, a last tile that
is nearly empty, rings of 2 h + 2 tiles with h = 1 and more), more lambda values
than its table holds (ebits of many ages: their columns go through memory),
columns of three and four checks, one iteration, all-zero syndromes.  The
reference is the two-pass device-memory kernel, which the oracle tests pin; all
outputs are equal bit for bit (every sum has one order, nothing is contracted).
"""
import pytest

from workloads import NLCNOT, pstring, sc, with_decoherence

pytestmark = pytest.mark.gpu

CASES = [("sc15-nlcnot", sc(15, NLCNOT, 15, 15, 1e-3, 1e-2), 66, 6, (64, 192, 512, 0)),
         ("sc15-quiet", sc(15, NLCNOT, 15, 15, 2e-5, 1e-4), 300, 20, (0,)),
         ("sc13-ebit-ages", with_decoherence(sc(13, NLCNOT, 13, 13, 5e-4, 5e-3), 1e-3, False), 2049, 3, (0,)),
         ("sc11-one-iteration", sc(11, NLCNOT, 11, 11, 1e-3, 1e-2), 2048, 1, (0, 320)),
         ("sc9-pstring6", pstring(sc(9, p=1e-3), 6, rounds=9), 2050, 5, (0, 448))]


@pytest.mark.parametrize("name,spec,shots,T,threads", CASES, ids=[c[0] for c in CASES])
def test_streamed_state_equals_device_state(gpu_lib, name, spec, shots, T, threads):
    import torch
    t = gpu_lib
    c = t.Circuit(spec)
    dem = t.DEM(c)
    det, obs = c.alloc_outputs(shots)
    c.sample(5, 0, 0, shots, det, obs)

    def run(kernel, **kw):
        o = dict(ehat=torch.zeros((shots, dem.cols), dtype=torch.uint8, device="cuda"),
                 llr=torch.zeros((shots, dem.cols), dtype=torch.float32, device="cuda"),
                 iters=torch.zeros(shots, dtype=torch.int32, device="cuda"),
                 flags=torch.zeros(shots, dtype=torch.uint8, device="cuda"), stats=t.new_stats())
        pred, pred2 = torch.zeros_like(obs), torch.zeros_like(obs)
        t.timing_reset()
        t.timing_enable(True)
        dem.decode(det, shots, pred, max_iter=T, use_osd=False, **o, **kw)
        dem.decode(det, shots, pred2, max_iter=T, use_osd=False, **kw)      # the compacted path
        torch.cuda.synchronize()
        t.timing_enable(False)
        assert kernel in t.timing_report()
        return dict(o, pred=pred, pred2=pred2)

    ref = run("k_bp_dev", bp_global_state=1)
    assert torch.equal(ref["pred"], ref["pred2"])
    for th in threads:
        got = run("k_bp_stream", bp_threads=th)
        for k in ref:
            assert torch.equal(got[k], ref[k]), (name, th, k)
