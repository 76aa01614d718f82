"""Compile the HIP library in-tree: csrc/* -> libblink.so (gfx950 only), and the Python
module that calls it (_blinkcall, without which calls go through ctypes).

The objects are linked WITHOUT a dependency on a particular libamdhip64: a
process must hold exactly one HIP runtime, and a PyTorch wheel brings its own.
The HIP entry points are therefore left undefined and bind, at load time, to
the runtime the process has already loaded (binding.py sees to that; a C or
C++ program simply links its own libamdhip64)."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libblink.so")
# call.c: a Python module, host code only.  Its name carries the interpreter it is for: another one does not load it.
CALL = os.path.join(HERE, "_blinkcall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ["kernel_f32.hip", "kernel_i32.hip",
           "fold_f32_sum.hip", "fold_i32_sum.hip", "fold_f32_other.hip", "fold_i32_other.hip",
           "fold_once_f32_sum.hip", "fold_once_i32_sum.hip", "fold_once_f32_other.hip", "fold_once_i32_other.hip",
           "fold_once_f32_mid.hip", "fold_once_i32_mid.hip", "fold_once_copy.hip",
           "fold_f32_mid.hip", "fold_i32_mid.hip", "fold_copy.hip", "exec.hip",
           "api.cpp", "pack.cpp", "schedule.cpp", "miad.cpp"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-c",
    "-fno-gpu-flush-denormals-to-zero",      # fp32 subnormals are ordinary addends
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # A ticket is drawn for one lane: by lane 0 alone where stages wait for one another, in the
    # one-pass kernel by a buffer atomic whose window holds lane 0's word at most.  The compiler's
    # wave-level rewriting of atomics (one lane adds for all, the others derive their values) gains
    # nothing there and reads the counter's answer, hence waits for it, right
    # after the atomic; without it the answer travels while other work goes on.
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    "-Wall", "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    def compile_one(src: str) -> str:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc] + FLAGS + [os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True, stderr=None if verbose else subprocess.DEVNULL)
        return obj

    # the kernel instantiation units take about half a minute each: side by side
    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
        objs = list(pool.map(compile_one, SOURCES))
    link = [os.environ.get("CXX", "g++"), "-shared", "-o", LIB] + objs
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.run(link, check=True)
    build_call(CALL, verbose)
    return LIB


def build_call(to: str, verbose: bool = False) -> bool:
    """The module of call.c.  It saves a call a microsecond of host time and nothing depends on it: where there is no C
    compiler or no Python headers none is left behind, and the caller is told."""
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-std=c11", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "call.c"), "-o", to]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        subprocess.run(cmd, check=True)
        return True
    except (OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(to):
            os.remove(to)
        print(f"{os.path.basename(to)} was not built, calls go through ctypes: {e}", file=sys.stderr, flush=True)
        return False


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
