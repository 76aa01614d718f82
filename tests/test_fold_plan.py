"""The tables and the ticket mapping of the kernel that runs schedules without
dependencies (whole-tree programs): whatever the flows' ranges, the tile size, the
distance of the rank buffers from a 1 KiB boundary and the order, every element of
every flow is handed out exactly once, tiles start on 1 KiB boundaries in memory,
and the orders are what they claim to be.  No GPU: the mapping host and kernel
share is compiled here with the host compiler."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TURN_PAYLOAD = 0xFFFFFFFF


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("fold") / "fold_plan_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1910_04940_amd", "csrc"), os.path.join(ROOT, "tests", "c", "fold_plan_check.cpp"),
                    "-o", exe], check=True)

    def run(flows, tile, shift, every, turn):
        out = subprocess.run([exe, str(tile), str(shift), str(int(every)), str(turn)] + [str(v) for f in flows for v in f],
                             check=True, capture_output=True, text=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


FLOWS = {
    "one": [(0, 10_007)],
    "shorter than a tile": [(0, 3), (4, 1), (8, 250)],
    "equal": [(i * 65_536, 65_536) for i in range(4)],
    "equal, off the tile grid": [(i * 25_604, 25_604) for i in range(4)],
    "unequal": [(0, 100_000), (100_000, 3), (100_004, 50_021), (150_028, 50_021), (200_052, 1_000)],
    "pieces at odd offsets": [(j * 7_001 + b, n) for j in range(16) for b, n in ((0, 3_500), (3_500, 3_501))],
}


@pytest.mark.parametrize("name", FLOWS)
@pytest.mark.parametrize("tile", [256, 1024, 3072, 8192])
@pytest.mark.parametrize("turn", [1, 3, 32, TURN_PAYLOAD])
def test_every_element_is_handed_out_once(check, name, tile, turn):
    flows = FLOWS[name]
    for shift in (0, 4, 128, 252):
        for every in (False, True):
            got = check(flows, tile, shift, every, turn)
            empty = 0
            for f, (off, ln) in enumerate(flows):
                mine = sorted((lo, n) for g, lo, n in got if g == f and n)
                assert mine[0][0] == off and sum(n for _, n in mine) == ln
                assert all(a + n == b for (a, n), (b, _) in zip(mine, mine[1:]))
                assert all((lo + shift) % 256 == 0 for lo, _ in mine[1:])        # 1 KiB of 4-byte elements
                assert all(n == tile for _, n in mine[1:-1])
            empty = sum(1 for _, _, n in got if n == 0)
            # a ticket without elements: only where one table serves every shift, or
            # where a shorter flow touches one tile more than a longer one
            assert empty <= len(flows)
            if not every and len(flows) == 1:
                assert empty == 0


def test_the_orders(check):
    flows = FLOWS["equal"]
    tile, tiles = 1024, 64
    assert [f for f, _, _ in check(flows, tile, 0, False, 1)] == [0, 1, 2, 3] * tiles
    by_chunk = check(flows, tile, 0, False, 24)              # 24, 24 and a last turn of 16 tiles
    assert [f for f, _, _ in by_chunk] == [f for g in (24, 24, 16) for f in range(4) for _ in range(g)]
    front = check(flows, tile, 0, False, TURN_PAYLOAD)
    assert [lo for _, lo, _ in front] == list(range(0, 4 * 65_536, tile))


def test_unequal_shares_leave_no_ticket_empty(check):
    """Flows of 40, 20, 20 and 1 tiles: 81 tickets, in turns while a flow has tiles left."""
    tile = 256
    flows = [(0, 40 * tile), (40 * tile, tile), (41 * tile, 20 * tile), (61 * tile, 20 * tile)]
    got = check(flows, tile, 0, False, 1)
    assert len(got) == 81 and all(n for _, _, n in got)
    assert [f for f, _, _ in got] == [0, 2, 3, 1] + [0, 2, 3] * 19 + [0] * 20


def test_random_flows(check):
    rng = np.random.default_rng(5)
    for _ in range(40):
        flows, at = [], 0
        for _ in range(int(rng.integers(1, 20))):
            at += int(rng.integers(0, 9))
            ln = int(rng.integers(1, 5_000))
            flows.append((at, ln))
            at += ln
        tile, shift = 256 * int(rng.integers(1, 12)), 4 * int(rng.integers(0, 64))
        got = check(flows, tile, shift, bool(rng.integers(2)), int(rng.choice([1, 2, 7, TURN_PAYLOAD])))
        seen = np.zeros(at, np.int32)
        for f, lo, n in got:
            assert n == 0 or (flows[f][0] <= lo and lo + n <= sum(flows[f]))
            seen[lo:lo + n] += 1
        want = np.zeros(at, np.int32)
        for off, ln in flows:
            want[off:off + ln] = 1
        assert np.array_equal(seen, want)
