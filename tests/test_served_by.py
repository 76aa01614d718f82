"""Which of the two kernels serves a schedule, and that one whose sums the waiting kernel would
add in another order than its trees prescribe is refused instead of sent there.  No GPU: the
rule is compiled here with the host compiler and shown schedules no program makes."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WANT = {
    "tree": "fold",
    "tree, asked to wait": "fold",               # no stage waits for another
    "tree, unlike stages": "not",
    "node": "fold",
    "node, asked to wait": "hand over",
    "node, unlike stages": "hand over",          # one fan-in at a time: load_rank is the order of the sum
    "edge, fills the cache": "fold",
    "edge, asked to wait": "hand over",
    "edge, larger": "hand over",
    "edge without dependencies": "fold",
}


def test_which_kernel_serves_a_schedule(tmp_path):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path / "served_by_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1910_04940_amd", "csrc"), os.path.join(ROOT, "tests", "c", "served_by_check.cpp"),
                    "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    assert dict(line.split(": ") for line in out.splitlines()) == WANT
