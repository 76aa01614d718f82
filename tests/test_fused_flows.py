"""What the one-pass kernel writes on the way through a tree: the sums that the per-edge program's
REDUCE steps write, each to the same rank, in the same order and with the same value, and of
them the per-node program's last one per node.  No GPU: the scheduler is compiled here with
the host compiler, and both programs are run on small integers."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_1910_04940_amd as bl
from test_random_schedules import random_case

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1910_04940_amd", "csrc")


@pytest.fixture(scope="module")
def fused(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("fused") / "fused_flow_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "c", "fused_flow_check.cpp"), os.path.join(CSRC, "schedule.cpp"),
                    os.path.join(CSRC, "pack.cpp"), "-o", exe], check=True)

    def run(op, fusion, n, chunk, k, roots, parents, w):
        args = [op, fusion, n, chunk, k, len(roots)]
        for r, p, weight in zip(roots, parents, w):
            args += [r, repr(weight)] + list(p)
        out = subprocess.run([exe] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout
        flows = []
        for line in out.splitlines():
            lo, hi, stores, seq, sums = line.split(" ")
            flows.append((int(lo), int(hi), [int(v) for v in stores.split(",")],
                          [tuple(int(v) for v in e.split(":")) for e in seq.split(",")],
                          [tuple(int(v) for v in e.split(":")) for e in sums.split(",")]))
        return flows
    return run


def _one_pass(seq, sums, x):
    """(rank, value) of every sum written on the way, and the result."""
    stack, writes, nth = [], [], 0

    def add(v):
        nonlocal nth
        stack[-1] += v
        rank, written = sums[nth]
        if written:
            writes.append((rank, stack[-1]))
        nth += 1
    for i, (rank, push, folds) in enumerate(seq):
        if i == 0 or push:
            stack.append(x[rank])
        else:
            add(x[rank])
        for _ in range(folds):
            top = stack.pop()
            add(top)
    assert len(stack) == 1 and nth == len(sums)
    return writes, stack[0]


@pytest.mark.parametrize("op", [bl.BLINK_OP_ALLREDUCE, bl.BLINK_OP_REDUCE])
@pytest.mark.parametrize("seed", range(40))
def test_sums_written_on_the_way_are_those_of_the_step_list(fused, seed, op):
    k, roots, parents, w, _, _ = random_case(5_000 + seed, same_root=False)
    n, chunk = 5_003, 1 << 20            # one chunk per tree
    trees = bl.blink_trees_from_arrays(k, roots, parents, w)
    steps = bl.blink_make_schedule(trees, op, n, chunk, bl.BLINK_FUSE_EDGE).steps()
    x = [int(v) for v in np.random.default_rng([83, seed]).integers(1, 1 << 40, k)]
    bounds = [b for b in zip(*[trees_bounds(trees, op, n, chunk)[i:] for i in (0, 1)]) if b[0] != b[1]]
    per_edge = fused(op, bl.BLINK_FUSE_EDGE, n, chunk, k, roots, parents, w)
    per_node = fused(op, bl.BLINK_FUSE_NODE, n, chunk, k, roots, parents, w)
    whole = fused(op, bl.BLINK_FUSE_TREE, n, chunk, k, roots, parents, w)
    assert [(lo, hi) for lo, hi, *_ in per_edge] == bounds
    for (lo, hi, stores, seq, sums), node, tree in zip(per_edge, per_node, whole):
        t = next(i for i, s in enumerate(steps) if int(s["off"]) == lo and int(s["len"]) == hi - lo)
        tree_no = int(steps[t]["tree"])
        held, writes = list(x), []
        for s in steps:                  # the reduce phase of this tree, as the step list has it
            if int(s["tree"]) == tree_no and int(s["kind"]) == bl.BLINK_STEP_REDUCE:
                held[int(s["dst"])] += held[int(s["src"])]
                writes.append((int(s["dst"]), held[int(s["dst"])]))
        root = roots[tree_no]
        got, result = _one_pass(seq, sums, x)
        assert result == sum(x) == held[root]
        assert stores == ([root] if op == bl.BLINK_OP_REDUCE else list(range(k)))
        # every write but the root's last, which the result is; per rank in the step list's order
        for r in range(k):
            mine = [v for rank, v in writes if rank == r]
            assert [v for rank, v in got if rank == r] == (mine[:-1] if r == root else mine), r
        # per node: the last of each inner node but the root
        got, result = _one_pass(node[3], node[4], x)
        last = dict(writes)
        last.pop(root)
        assert len(got) == len(last) and dict(got) == last and result == held[root]
        # a whole-tree program writes none
        assert _one_pass(tree[3], tree[4], x) == ([], held[root])


def trees_bounds(trees, op, n, chunk):
    return bl.blink_make_schedule(trees, op, n, chunk, bl.BLINK_FUSE_TREE).bounds()
