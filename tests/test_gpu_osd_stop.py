"""OSD-0's stop at the column that completes the span of s.

Syndromes of 1 to several hundred random columns, and random events, put that
column anywhere: inside the first wave's candidates, at and past its 63rd, in
later waves and passes, and past the prefix (the full sort decides those).  The correction is unique
given the posteriors, so it is compared bit for bit with an elimination over
Python integers on the decoder's own posteriors.
"""
import numpy as np
import pytest

from oracle.circuits import build_circuit
from oracle.dem import build_dem
from oracle.frame import pack_bits
from oracle.osd import column_ints
from workloads import NLCNOT, TELEPORT, bb, sc

pytestmark = pytest.mark.gpu


def _osd0(cols, s, L):
    """(columns of the correction, place of the last column looked at)."""
    order = np.argsort(np.where(L == 0, 0, L), kind="stable")
    basis = {}                                      # lowest bit -> (vector, places)
    rest, taken = s, 0
    for place, v in enumerate(order):
        if not rest:
            return [int(order[k]) for k in range(len(order)) if taken >> k & 1], place - 1
        x, c = cols[v], 1 << place
        while x and (x & -x) in basis:
            y, d = basis[x & -x]
            x, c = x ^ y, c ^ d
        if not x:
            continue
        basis[x & -x] = (x, c)
        t, left, bit = rest, 0, 0
        while t:                                    # reduce what is left of s as far as the basis goes
            bit = t & -t
            if bit in basis:
                y, d = basis[bit]
                t, taken = t ^ y, taken ^ d
            else:
                left |= bit
                t ^= bit
        rest = left
    return ([int(order[k]) for k in range(len(order)) if taken >> k & 1], len(order)) if not rest else (None, len(order))


@pytest.mark.parametrize("name,spec,kw", [
    ("one-wave", sc(5, NLCNOT, 5, 5, 3e-3, 2e-2), {}),
    ("prefix", bb("bb144", TELEPORT, 4, 3, 1e-3, 1e-2), {}),
    ("window", bb("bb54", NLCNOT, 2, 2, 2e-3, 1e-2), {"osd_window": 2048}),
], ids=["one-wave", "prefix", "window"])
def test_stop_at_any_column(gpu_lib, name, spec, kw):
    import torch
    t = gpu_lib
    oc = build_circuit(spec)
    od = build_dem(oc)
    H = od.H()
    m = H.shape[0]
    rng = np.random.default_rng(11)
    weights = [1, 2, 3, 4, 6, 8, 12, 16, 20, 24, 28, 32, 40, 48, 64, 80, 100, 130, 200, 300]
    det = np.zeros((m, len(weights) + 4), dtype=np.uint8)
    for k, w in enumerate(weights):
        det[:, k] = H[:, rng.choice(H.shape[1], w, replace=False)].sum(axis=1) & 1
    for k, w in enumerate([1, 20, m // 2, m]):      # (few of these are in the span)
        det[rng.choice(m, w, replace=False), len(weights) + k] = 1
    dem = t.DEM(t.Circuit(spec))
    shots = det.shape[1]
    pred = torch.zeros((max(dem.info["obs"], 1), 1), dtype=torch.int64, device="cuda")
    ehat = torch.zeros((shots, dem.cols), dtype=torch.uint8, device="cuda")
    llr = torch.zeros((shots, dem.cols), dtype=torch.float32, device="cuda")
    flags = torch.zeros(shots, dtype=torch.uint8, device="cuda")
    dem.decode(torch.from_numpy(pack_bits(det).view(np.int64)).cuda(), shots, pred, max_iter=3, ehat=ehat, llr=llr,
               flags=flags, **kw)
    torch.cuda.synchronize()
    e, L, f = ehat.cpu().numpy(), llr.cpu().numpy(), flags.cpu().numpy()
    cols = column_ints(H)
    seen = []
    for k in range(shots):
        if not f[k] & 2 or f[k] & 8:
            continue
        s = sum(1 << int(r) for r in np.nonzero(det[:, k])[0])
        want, stop = _osd0(cols, s, L[k])
        seen.append(stop)
        assert (want is None) == bool(f[k] & 4), (name, k)
        if want is not None:
            assert np.nonzero(e[k])[0].tolist() == sorted(want), (name, k, stop)
    assert len(seen) >= shots // 2 and min(seen) < 63 and max(seen) >= 252, seen
