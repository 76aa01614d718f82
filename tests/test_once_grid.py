"""How the kernel with a workgroup for every tile cuts up a payload: every element of every flow
belongs to one workgroup, tiles are no larger than a workgroup's columns, and as small as they can be
without a workgroup more on any compute unit.  No GPU: what host and kernel share is compiled here
with the host compiler."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("once") / "once_grid_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1910_04940_amd", "csrc"), os.path.join(ROOT, "tests", "c", "once_grid_check.cpp"),
                    "-o", exe], check=True)

    def run(flows, most, shift, cus):
        out = subprocess.run([exe, str(most), str(shift), str(cus)] + [str(v) for f in flows for v in f],
                             check=True, capture_output=True, text=True).stdout
        head, *rest = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
        return head, rest
    return run


def _covers(flows, pieces):
    for f, (off, n) in enumerate(flows):
        seen = np.zeros(n, np.int32)
        for g, lo, ln in pieces:
            if g == f:
                assert off <= lo and lo + ln <= off + n
                seen[lo - off:lo - off + ln] += 1
        assert (seen == 1).all(), (f, off, n)


# shares of a payload (the last one with a ragged end), pieces at odd offsets, flows of a few elements
@pytest.mark.parametrize("flows", [
    [(0, 16_411)], [(0, 4_100), (4_100, 4_100), (8_200, 4_100), (12_300, 4_111)], [(0, 100_000), (100_000, 4), (100_004, 3)],
    [(j * 7_001, 7_001) for j in range(16)], [(0, 1)], [(5, 1)], [(2, 9)], [(1, 2), (3, 3), (6, 4), (10, 5)],
], ids=str)
@pytest.mark.parametrize("shift", [0, 4, 128, 252])
@pytest.mark.parametrize("most,cus", [(1024, 256), (6144, 256), (2048, 7), (1024, 1)])
def test_every_element_belongs_to_one_workgroup(check, flows, shift, most, cus):
    (tile, busy, whole), pieces = check(flows, most, shift, cus)
    assert 0 < tile <= most and tile % 64 == 0
    _covers(flows, pieces)
    rounds = -(-whole // cus)
    assert -(-busy // cus) == rounds
    if tile > 64:       # one step smaller and some compute unit would get another
        smaller = sum(-(-((off + shift) % 256 + n) // (tile - 64)) for off, n in flows)
        assert smaller > rounds * cus


def test_random_flows(check):
    rng = np.random.default_rng(8)
    for _ in range(60):
        flows, at = [], 0
        for _ in range(int(rng.integers(1, 17))):
            at += int(rng.integers(0, 9))
            n = int(rng.integers(1, 30_000))
            flows.append((at, n))
            at += n
        most = 1024 * int(rng.integers(1, 9))
        _, pieces = check(flows, most, 4 * int(rng.integers(0, 64)), int(rng.choice([1, 13, 256])))
        _covers(flows, pieces)
