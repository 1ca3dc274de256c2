"""Scratch that shrinks instead of failing (host/scratch.h), with a fake allocator."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_alloc_most_halves_until_it_fits(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "scratch_check")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2504_05611_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "scratch_check.cpp"), "-o", exe], check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    rows = [tuple(int(x) for x in line.split()) for line in out]
    assert len(rows) == 10
    for want, least, room, got, calls in rows:
        steps = []
        n = want
        while n >= least and n > 0:
            steps.append(n)
            n //= 2
        fitting = [s for s in steps if s <= room]
        assert got == (fitting[0] if fitting else 0), (want, least, room)
        assert calls == (steps.index(got) + 1 if got else len(steps))
