"""BP with its state in LDS (bp_global_state = 0) at the edges of its schedules.

Checks of more edges than a part holds (bb144 teleport: up to 161, cut into
eight parts), more columns than a 16-bit address reaches (d = 13), one to
sixteen waves, and scalings that take the comparison variant (values that
could overflow).  The reference is a device-memory kernel, which the oracle
tests pin, and for finite scalings the FP32 oracle too.  Everything is bit for
bit: every sum has one order and nothing is contracted.
"""
import numpy as np
import pytest

from oracle.circuits import build_circuit
from oracle.dem import build_dem
from oracle.frame import pack_bits, sample as oracle_sample
from oracle.osd import Decoder
from workloads import MEMORY, NLCNOT, TELEPORT, bb, sc

pytestmark = pytest.mark.gpu


def _decode(tmcs, dem, det, shots, T, **kw):
    import torch
    o = dict(pred=torch.zeros((max(dem.info["obs"], 1), (shots + 63) // 64), dtype=torch.int64, device="cuda"),
             ehat=torch.zeros((shots, dem.cols), dtype=torch.uint8, device="cuda"),
             llr=torch.zeros((shots, dem.cols), dtype=torch.float32, device="cuda"),
             iters=torch.zeros(shots, dtype=torch.int32, device="cuda"),
             flags=torch.zeros(shots, dtype=torch.uint8, device="cuda"), stats=tmcs.new_stats())
    pred = o.pop("pred")
    dem.decode(det, shots, pred, max_iter=T, **o, **kw)
    torch.cuda.synchronize()
    return dict(o, pred=pred)


SHAPES = [("bb144-teleport", bb("bb144", TELEPORT, 4, 3, 1e-3, 1e-2), 130, 12),
          ("bb54-nlcnot", bb("bb54", NLCNOT, 2, 2, 2e-3, 1e-2), 257, 20),
          ("sc13-nlcnot", sc(13, NLCNOT, 13, 13, 1e-3, 1e-2), 65, 8),
          ("sc5-nlcnot", sc(5, NLCNOT, 5, 5, 3e-3, 2e-2), 1000, 30)]


@pytest.mark.parametrize("weighted", [False, True], ids=["plain", "weighted"])
@pytest.mark.parametrize("name,spec,shots,T", SHAPES, ids=[s[0] for s in SHAPES])
def test_lds_state_equals_device_state(gpu_lib, name, spec, shots, T, weighted):
    import torch
    t = gpu_lib
    c = t.Circuit(spec)
    dem = t.DEM(c)
    det, obs = c.alloc_outputs(shots)
    c.sample(5, 0, 0, shots, det, obs)
    w = None
    if weighted:                                    # zeros and negative weights among them
        g = torch.Generator(device="cuda").manual_seed(1)
        w = torch.randn((T, dem.edges), generator=g, device="cuda").round(decimals=1)
    ref = _decode(t, dem, det, shots, T, weights=w, use_osd=False, bp_global_state=1)
    assert int(ref["iters"].max()) == T or int((ref["flags"] & 1).sum()) == shots
    for threads in (0, 64, 192, 1024):
        got = _decode(t, dem, det, shots, T, weights=w, use_osd=False, bp_threads=threads)
        for k in ref:
            assert torch.equal(got[k], ref[k]), (name, threads, k)


@pytest.mark.parametrize("T", [1, 12, 70])
@pytest.mark.parametrize("alpha", [1e-3, 0.75, 30.0, 2e6, 3e38], ids=str)
def test_lds_state_scalings(gpu_lib, alpha, T):
    import torch
    t = gpu_lib
    spec, shots = sc(3, MEMORY, 3, 0, 2e-2), 300
    oc = build_circuit(spec)
    d, _ = oracle_sample(oc, 3, 0, 0, shots)
    det = torch.from_numpy(pack_bits(d).view(np.int64)).cuda()
    dem = t.DEM(t.Circuit(spec))
    got = _decode(t, dem, det, shots, T, alpha=alpha, use_osd=False)
    # (the one-pass kernel: it pads nothing, so infinities meet only what the definition has them meet)
    ref = _decode(t, dem, det, shots, T, alpha=alpha, use_osd=False, bp_global_state=3)
    for k in ref:
        assert np.array_equal(got[k].cpu().numpy(), ref[k].cpu().numpy(), equal_nan=k == "llr"), (alpha, T, k)
    llr = got["llr"].cpu().numpy()
    if np.isfinite(llr).all() and T <= 12:          # (the oracle's minimum lets a NaN through, the library's does not)
        od = build_dem(oc)
        o = Decoder(od.H(), od.priors(), od.L(), max_iter=T, alpha=alpha, dtype=np.float32, use_osd=False).decode(d.T)
        assert (got["iters"].cpu().numpy() == o["iters"]).all()
        assert (llr == o["llr"].astype(np.float32)).all()
