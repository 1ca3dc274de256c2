"""The windowed OSD-0's chain of windows: 512, then 1024, then 2048 rows.

With the default window every shot starts with 512 rows; what that leaves open
goes on to 1024 and then to 2048.  Syndromes sampled at higher noise than the DEM's
give shots that are decided in each.  Which window decides a shot follows from its
posteriors alone: the first whose rows hold those touched by the sorted columns up
to the one that completes the span of the syndrome (an XOR basis over Python
integers, as in the oracle's OSD-0, which also gives the one solution there is).
"""
import numpy as np
import pytest

from workloads import NLCNOT, sc

pytestmark = pytest.mark.gpu


def _solve(cols, synd, llr):
    """(rows touched up to the column that completes the span, the solution's columns)."""
    y, e = synd, 0                        # what is left of the syndrome, and the kept columns taken into it
    basis, kept, touched = {}, [], 0
    for v in np.lexsort((np.arange(len(cols)), np.asarray(llr))):
        touched |= cols[v]
        x, comb = cols[v], 0
        while x and (x.bit_length() - 1) in basis:
            b, bc = basis[x.bit_length() - 1]
            x, comb = x ^ b, comb ^ bc
        if not x:
            continue
        basis[x.bit_length() - 1] = (x, comb | (1 << len(kept)))
        kept.append(int(v))
        while y and (y.bit_length() - 1) in basis:
            b, bc = basis[y.bit_length() - 1]
            y, e = y ^ b, e ^ bc
        if not y:
            return bin(touched).count("1"), sorted(k for i, k in enumerate(kept) if (e >> i) & 1)
    return None, None


def test_each_window_decides_shots(gpu_lib):
    import torch
    t, T, n = gpu_lib, 6, 128
    ps = (1e-3, 4e-3, 6e-3, 7e-3, 8e-3, 1e-2)
    dem = t.DEM(t.Circuit(sc(17, NLCNOT, 17, 17, 1e-3, 1e-2)))
    parts = []
    for p in ps:
        c = t.Circuit(sc(17, NLCNOT, 17, 17, p, 1e-2))
        det, _ = c.alloc_outputs(n)
        c.sample(3, 0, 0, n, det, c.alloc_outputs(n)[1])
        parts.append(det)
    det = torch.cat(parts, 1).contiguous()
    shots = n * len(ps)
    assert dem.rows > 2048 and det.shape[0] == dem.rows

    def run(window):
        o = dict(ehat=torch.zeros((shots, dem.cols), dtype=torch.uint8, device="cuda"),
                 llr=torch.zeros((shots, dem.cols), dtype=torch.float32, device="cuda"),
                 flags=torch.zeros(shots, dtype=torch.uint8, device="cuda"))
        stats = t.new_stats()
        pred = torch.zeros((dem.info["obs"], shots // 64), dtype=torch.int64, device="cuda")
        dem.decode(det, shots, pred, max_iter=T, osd_window=window, stats=stats, **o)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in o.items()}, t.read_stats(stats)

    got, stats = run(0)
    osd = (got["flags"] & 2) != 0
    open_at = {w: (run(w)[0]["flags"] & 8) != 0 for w in (512, 1024)}
    open_at[2048] = (got["flags"] & 8) != 0
    decided = {512: osd & ~open_at[512], 1024: open_at[512] & ~open_at[1024], 2048: open_at[1024] & ~open_at[2048]}
    print({w: int(d.sum()) for w, d in decided.items()}, int(open_at[2048].sum()), stats, flush=True)
    assert all(d.sum() >= 3 for d in decided.values())
    # the later windows' jobs, each counted where it ends
    assert stats["osd_prefix_retry"] == int(open_at[512].sum()) and stats["osd_incomplete"] == int(open_at[2048].sum())
    h = dem.export()
    cols = [0] * dem.cols
    for v in range(dem.cols):
        for r in h.row_idx[h.col_ptr[v]:h.col_ptr[v + 1]]:
            cols[v] |= 1 << int(r)
    words = det.cpu().numpy().view(np.uint64)
    for w, d in decided.items():
        for i in np.nonzero(d)[0][:3]:
            bits = (words[:, i // 64] >> np.uint64(i % 64)) & np.uint64(1)
            rows, cor = _solve(cols, sum(1 << int(r) for r in np.nonzero(bits)[0]), got["llr"][i])
            assert w // 2 * (w > 512) < rows <= w, (w, i, rows)
            assert list(np.nonzero(got["ehat"][i])[0]) == cor, (w, i)
