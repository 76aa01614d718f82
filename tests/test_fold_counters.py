"""How the fold kernel's workgroups take their tickets, from one counter or two, whatever order they
draw in: every ticket once, as many draws as the host counts on.  No GPU: the mapping host and kernel share
is compiled here with the host compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("counters") / "fold_counters_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1910_04940_amd", "csrc"), os.path.join(ROOT, "tests", "c", "fold_counters_check.cpp"),
                    "-o", exe], check=True)
    return lambda *args: subprocess.run([exe] + [a if isinstance(a, str) else str(int(a)) for a in args]).returncode


@pytest.mark.parametrize("two,grid", [(False, 1), (False, 7), (False, 224), (True, 16), (True, 48), (True, 256)])
@pytest.mark.parametrize("more", [0, 1, 2, 15, 16, 999, 12_345])
def test_every_ticket_is_taken_once(check, two, grid, more):
    for seed in range(3):
        assert check(grid + more, grid, two, seed) == 0


@pytest.mark.parametrize("start", [0, (1 << 32) - 5, (1 << 32) - 2_000, (1 << 32) - 30_000, (7 << 32) - 1, (1 << 40) + 3])
def test_calls_on_one_schedule_wherever_its_counters_stand(check, start):
    """Forty calls, with one counter and with two, on grids of several sizes.  The counters have 32 bits, which a schedule
    that streams without a pause goes through in a minute or two; the host counts on in 64."""
    for seed in range(4):
        assert check("calls", start, seed) == 0
