"""OSD-CS with its order in device memory (DEMs beyond the LDS basis: 720
detectors here) against the oracle's, correction by correction, in one pass and
in several."""
import numpy as np
import pytest

from oracle.circuits import build_circuit
from oracle.dem import build_dem
from oracle.frame import pack_bits, sample as oracle_sample
from oracle.osd import Decoder
from workloads import NLCNOT, sc

pytestmark = pytest.mark.gpu


def test_dense_osd_cs_matches_oracle(gpu_lib):
    import torch
    t = gpu_lib
    spec, shots, T = sc(7, NLCNOT, 7, 7, 5e-3, 2e-2), 24, 20
    oc = build_circuit(spec)
    od = build_dem(oc)
    assert od.H().shape[0] > 512
    d, _ = oracle_sample(oc, 3, 0, 0, shots)
    want = Decoder(od.H(), od.priors(), od.L(), max_iter=T, dtype=np.float32, osd_order=7).decode(d.T, chunk=64)
    assert int(want["osd"].sum()) > 8
    dem = t.DEM(t.Circuit(spec))
    # (128 copies of the shots: more jobs than one round of resident workgroups of a few compute units)
    det = torch.from_numpy(pack_bits(np.tile(d, (1, 128))).view(np.int64)).cuda()
    n = shots * 128
    for kw in ({}, {"decode_chunk": 1024}, {"osd_per_cu": 1}):
        pred = torch.zeros((max(dem.info["obs"], 1), (n + 63) // 64), dtype=torch.int64, device="cuda")
        ehat = torch.zeros((n, dem.cols), dtype=torch.uint8, device="cuda")
        dem.decode(det, n, pred, max_iter=T, ehat=ehat, osd_order=7, **kw)
        torch.cuda.synchronize()
        got = ehat.cpu().numpy().astype(bool)
        assert (got == np.tile(want["e_hat"].astype(bool), (128, 1))).all(), kw
