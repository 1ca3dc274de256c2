"""The rule that puts a shot's BP state into LDS, around its limit (host code only)."""
import os
import shutil
import subprocess
from collections import defaultdict

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2504_05611_amd")
LIMIT, STATIC = 160 * 1024, 1024            # a compute unit's LDS; what a team has beside the dynamic part


def test_a_team_fits_exactly_where_its_bytes_do(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    if not os.path.exists(os.path.join(PKG, "libtmcs.so")):
        from paper_2504_05611_amd.build import build
        build(verbose=False)
    exe = str(tmp_path / "chunk_fit")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "native", "chunk_fit.cpp"), os.path.join(PKG, "libtmcs.so"),
                    "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined", "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    fits, size = defaultdict(dict), defaultdict(dict)
    for line in out:
        name, rows, cols, P, ok, lds, usual = line.split()
        fits[name][int(P)] = ok == "1"
        if ok == "1":
            size[name][int(P)] = int(lds)
            assert int(lds) + STATIC <= LIMIT
            # a message's part and a column's L are 12 and 4 bytes, checks and columns in chunks of 64
            assert int(lds) >= 12 * int(rows) + 4 * int(cols) + 32 * (int(P) // 64)
            assert int(usual) - int(lds) in range(-64 * 32, 64 * 32)
    kinds = {name: (all(f.values()), any(f.values())) for name, f in fits.items()}
    assert (True, True) in kinds.values() and (False, False) in kinds.values()
    # the largest circuits that still fit leave less room than a team of 16 waves was once promised
    assert max(max(s.values()) for s in size.values()) + STATIC > LIMIT - 2 * 224 * 16
    for name, f in fits.items():
        for P in (1024, 512, 256, 128):     # a smaller team never needs more
            assert not f[P] or f[P // 2], (name, P)
