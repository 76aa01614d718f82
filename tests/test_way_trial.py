"""The timed choice among the ways to serve a whole-tree schedule: only like calls are
compared.  No GPU: the rule is compiled here with the host
compiler."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def play(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("trial") / "way_trial_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1910_04940_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "way_trial_check.cpp"), "-o", exe], check=True)

    def run(front, turns, classes):
        out = subprocess.run([exe, str(int(front)), str(int(turns))] + [str(c) for c in classes], check=True,
                             capture_output=True, text=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("front,turns", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("order", ["one", "alternating", "a stray first", "mixed"])
def test_every_kind_of_call_is_compared_with_its_like(play, front, turns, order):
    ways = [1] + [2] * front + [3] * turns
    n = 4 * len(ways)
    classes = {"one": [0] * 40, "alternating": [0, 1] * 40, "a stray first": [1] + [0] * 40,
               "mixed": random.Random(3).choices(range(3), k=120)}[order]
    calls = play(front, turns, classes)
    timed = [c for c in calls if c[2]]
    for cls in set(classes):
        mine = [way for c, way, _ in timed if c == cls]
        assert mine == (ways * 4)[:len(mine)]               # goes round the ways, whoever calls in between
    first_untimed = next(i for i, c in enumerate(calls) if not c[2])
    decider = calls[first_untimed][0]
    assert sum(1 for c in timed if c[0] == decider) == n    # one kind is complete: it decides
    assert first_untimed <= 4 * n and not any(c[2] for c in calls[first_untimed:])
    assert {c[1] for c in calls[first_untimed:]} == {max(ways)}       # the fastest here
