"""The rules by which the launcher of the fold kernel chooses workgroups and counters.  No GPU:
they are compiled here with the host compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("rules") / "fold_rules_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1910_04940_amd", "csrc"), os.path.join(ROOT, "tests", "c", "fold_rules_check.cpp"),
                    "-o", exe], check=True)

    def ask(*args):
        out = subprocess.run([exe] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout
        return tuple(int(v) for v in out.split())
    return ask


@pytest.mark.parametrize("cus", [32, 64, 128, 256])
@pytest.mark.parametrize("eighths", [6, 7, 8])
def test_counters_cost_no_workgroup(rule, cus, eighths):
    """Drawn tickets: every workgroup that the launcher wants runs, on parts of a card too; small tickets draw from two
    counters where the workgroups are more than one counter keeps up with."""
    most = cus * eighths // 8
    for ticket_bytes in (57_344, 131_072):
        grid, dealt, two = rule("grid", most, 100_000, 0, ticket_bytes)
        assert (grid, dealt) == (most, 0)
        assert two == (cus == 256 and ticket_bytes < 131_072)


@pytest.mark.parametrize("most", [1, 15, 17, 159, 168, 1000])
def test_grids_that_two_counters_do_not_divide(rule, most):
    """By request of the caller a grid can have any size; the two counters need a multiple of sixteen."""
    assert rule("grid", most, 100_000, 0, 57_344) == (most, 0, 0)


def test_a_workgroup_for_every_ticket_draws_none(rule):
    assert rule("grid", 5_000, 5_000, 1, 57_344) == (5_000, 1, 0)     # a small payload
    assert rule("grid", 256, 1_000, 1, 57_344) == (256, 1, 0)         # the same on fewer, by request
    assert rule("grid", 256, 200, 0, 57_344) == (200, 1, 0)
    assert rule("grid", 256, 256, 0, 57_344) == (256, 1, 0)
    assert rule("grid", 256, 257, 0, 57_344) == (256, 0, 1)
