"""The frame kernel's launch shapes: words per workgroup and its threads follow
from the shots of a call, the bits do not.

A large call (many words per workgroup, several workgroups per compute unit) is
compared with the same shots drawn in pieces, down to one word of one shot block
(one word per workgroup, the other thread counts); the small sizes themselves
are pinned to the oracle by the sampler tests.  Bit for bit: every shot's noise
is a function of its number alone.
"""
import pytest

from workloads import MEMORY, NLCNOT, TELEPORT, bb, sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spec,shots", [
    (sc(3, MEMORY, 3, 0, 5e-3), (1 << 20) + 77),
    (sc(5, NLCNOT, 5, 5, 1e-3, 1e-2), (1 << 18) + 65),
    (sc(9, NLCNOT, 2, 2, 1e-3, 1e-2), 1 << 18),
    (bb("bb144", MEMORY, 2, 0, 1e-3, 1e-3), (1 << 18) + 1),
    (bb("bb144", TELEPORT, 1, 1, 1e-3, 1e-2), 1 << 16),
], ids=["sc3", "sc5", "sc9", "bb144-memory", "bb144-teleport"])
def test_pieces_equal_the_whole(gpu_lib, spec, shots):
    import torch
    c = gpu_lib.Circuit(spec)
    det, obs = c.alloc_outputs(shots)
    c.sample(9, 1, 0, shots, det, obs)
    assert bool(det.any()) and bool(obs.any())
    for begin, n in ((0, 64), (4096 - 64, 128), (64, 9999), (8192, 16384), (4096 * 3, 40000), (shots // 64 * 64 - 64, 64 + shots % 64)):
        n = min(n, shots - begin)
        d, o = c.alloc_outputs(n)
        c.sample(9, 1, begin, n, d, o)
        w = begin // 64
        k = (n + 63) // 64
        mask = torch.full((k,), -1, dtype=torch.int64, device="cuda")
        if n % 64:                                   # shots past the piece's end stay zero
            mask[-1] = (1 << (n % 64)) - 1
        assert torch.equal(d, det[:, w : w + k] & mask), (begin, n)
        assert torch.equal(o, obs[:, w : w + k] & mask), (begin, n)
