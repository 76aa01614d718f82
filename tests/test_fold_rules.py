"""The rules by which the launcher of the fold kernel chooses workgroups, counters, a copy's columns and how results are written.
No GPU: they are compiled here with the host compiler."""
import os
import shutil
import subprocess

import pytest

import paper_1910_04940_amd as bl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1910_04940_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "no host compiler"
    exe = str(tmp_path_factory.mktemp("rules") / "fold_rules_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "c", "fold_rules_check.cpp"), os.path.join(CSRC, "schedule.cpp"),
                    os.path.join(CSRC, "pack.cpp"), "-o", exe], check=True)

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


MIB = 1 << 20
KEEP, STREAM, SPREAD = 0, 1, 2


def _policy(rule, k, mib, op, way=1, deps=0, alternates=1):
    """Sums of k ranks of mib MiB that all get the result, or a gather of them."""
    n_load, n_store = (k, k) if op == "sum" else (1, 1)
    kernel = 2 * k * mib * MIB if op == "sum" else 2 * (mib * MIB - mib * MIB // k)
    return rule("policy", n_load, n_store, k * mib * MIB, kernel, deps, way, alternates)[0]


@pytest.mark.parametrize("way", [1, 3])
def test_results_of_sums_stream_from_twelve_caches(rule, way):
    for k, mib in ((8, 384), (16, 192), (4, 800)):
        assert _policy(rule, k, mib, "sum", way) == STREAM
        assert _policy(rule, k, mib // 2, "sum", way) == KEEP


@pytest.mark.parametrize("k,mib", [(8, 80), (8, 400), (8, 4000), (4, 800), (2, 1600), (3, 1100)])
def test_what_a_gather_wrote_stays_for_the_next_call(rule, k, mib):
    """It writes one rank: of 8 x 400 MiB 350 MiB, not twelve times the cache."""
    assert _policy(rule, k, mib, "gather", 1) == KEEP
    assert _policy(rule, k, mib, "gather", 3) == KEEP


def test_one_front_streams_what_does_not_fit(rule):
    assert _policy(rule, 8, 64, "sum", 2) == STREAM and _policy(rule, 8, 63, "sum", 2) == KEEP
    # a gather of 8 x 128 MiB reads 112 and writes 112: all of it fits the cache, though 1 GiB is set aside
    assert _policy(rule, 8, 128, "gather", 2) == KEEP
    assert _policy(rule, 4, 140, "gather", 2) == KEEP
    assert _policy(rule, 2, 200, "gather", 2) == KEEP
    assert _policy(rule, 8, 200, "gather", 2) == STREAM
    assert _policy(rule, 4, 200, "gather", 2) == STREAM


def test_calls_that_do_not_alternate_stream_past_a_cache_that_is_too_small(rule):
    assert _policy(rule, 8, 32, "sum", alternates=0) == KEEP
    assert _policy(rule, 8, 33, "sum", alternates=0) == STREAM
    assert _policy(rule, 8, 33, "sum", deps=1) == STREAM
    assert _policy(rule, 8, 146, "gather", alternates=0) == KEEP       # 255 MiB moved
    assert _policy(rule, 8, 147, "gather", alternates=0) == STREAM     # 257
    assert _policy(rule, 8, 147, "gather", deps=1) == STREAM
    assert rule("policy", 1, 7, 64 * MIB, 64 * MIB, 0, 1, 1) == (SPREAD,)


@pytest.mark.parametrize("k", [3, 4, 5])
def test_a_copy_has_the_columns_of_what_it_moves(rule, k):
    """Down a chain the stages of per-edge and per-node programs read what other stages wrote; the kernel that carries a tile
    through all of them does not, so all three programs are the same copy."""
    chain = list(range(-1, k - 1))
    line = 512 if k == 5 else 160     # MiB in all rank buffers, each read or written once
    for mib, columns in ((0.75 * line, 4), (0.98 * line, 4), (1.02 * line, 8)):
        for fusion in (bl.BLINK_FUSE_EDGE, bl.BLINK_FUSE_NODE, bl.BLINK_FUSE_TREE):
            n = int(mib * MIB) // 4 // k
            assert rule("columns", bl.BLINK_OP_BROADCAST, fusion, n, 1 << 16, *chain) == (columns,), (mib, fusion)


def test_a_copys_columns_by_ranks_written(rule):
    def star(k, mib, op=bl.BLINK_OP_BROADCAST):
        return rule("columns", op, bl.BLINK_FUSE_TREE, mib * MIB // 4 // k, 1 << 16, *([-1] + [0] * (k - 1)))[0]
    assert [star(k, 1000) for k in (2, 3, 5, 6, 7, 8, 9, 10, 16)] == [16, 8, 8, 4, 4, 3, 3, 2, 2]
    assert [star(k, 100) for k in (2, 3, 5, 6, 7, 8, 9, 10, 16)] == [4, 4, 4, 4, 4, 3, 3, 2, 2]


# Up to how many MiB read and written on 256 compute units a whole-tree payload has a workgroup per tile: (ranks, collective,
# MiB).  tests/test_gpu_once.py runs both sides of them.
ONCE_LINES = [(2, "allreduce", 160), (3, "allreduce", 160), (8, "allreduce", 160), (16, "allreduce", 160),
              (3, "reduce", 160), (4, "reduce", 320), (8, "reduce", 320), (9, "reduce", 192),
              (2, "gather", 160), (3, "gather", 256), (4, "gather", 384), (8, "gather", 384),
              (2, "broadcast", 160), (4, "broadcast", 160), (8, "broadcast", 160),
              (2, "allgather", 256), (4, "allgather", 192), (8, "allgather", 192), (10, "allgather", 208)]
# The same for programs that write sums on the way: k - 2 of them per edge in a chain, of 4 bytes, where they count.
ONCE_SUMS = [(3, "allreduce", 160, 1), (7, "allreduce", 160, 5), (8, "allreduce", 160, 0), (16, "allreduce", 160, 0),
             (3, "reduce", 160, 0), (4, "reduce", 320, 2), (8, "reduce", 320, 6), (9, "reduce", 192, 0), (16, "reduce", 192, 0)]
# bytes that a collective reads and writes per element of k ranks' payload
MOVED = {"allreduce": lambda k: 8 * k, "reduce": lambda k: 4 * (k + 1), "gather": lambda k: 8 * (k - 1) / k,
         "broadcast": lambda k: 4 * k, "allgather": lambda k: 4 * k}
OPS = {"allreduce": bl.BLINK_OP_ALLREDUCE, "reduce": bl.BLINK_OP_REDUCE, "gather": bl.BLINK_OP_GATHER,
       "broadcast": bl.BLINK_OP_BROADCAST, "allgather": bl.BLINK_OP_ALLGATHER}


@pytest.mark.parametrize("k,op,mib", ONCE_LINES)
def test_how_far_a_payload_has_a_workgroup_per_tile(rule, k, op, mib):
    """Whichever rank is the root: the piece that a Gather's root keeps is not one that is copied."""
    for root in {0, k // 2, k - 1}:
        star = [-1 if v == root else root for v in range(k)]
        for n, served in ((int(mib * MIB / MOVED[op](k)) - 4_099, 1), (int(mib * MIB / MOVED[op](k)) + 4_099, 0)):
            assert rule("once", OPS[op], bl.BLINK_FUSE_TREE, n - n % k, 1 << 16, *star) == (served,), (root, n)


# Shares of a payload, flows of the kernel with a workgroup per tile (0: it cannot run them).  tests/test_gpu_once.py runs them.
ONCE_SHARES = [([1.0], 1), ([1.0, 2.0, 3.0], 3), ([1.0] * 4, 4), ([1.0] * 5, 5), ([1.0 + t for t in range(16)], 16), ([1.0] * 17, 0),
               ([1.0, 1.0, 1.0, 40.0], 0)]


@pytest.mark.parametrize("weights,flows", ONCE_SHARES)
def test_which_shares_have_a_workgroup_per_tile(rule, weights, flows):
    assert rule("shares", OPS["allreduce"], 1_000_003, *weights) == (flows, int(flows > 0))
    # what goes from one rank to the same others is one flow, whatever trees it was split among
    assert rule("shares", OPS["broadcast"], 1_000_003, *weights) == (1, 1)
    assert rule("shares", OPS["gather"], 1_000_000, *weights) == (3, 1)
    assert rule("shares", OPS["allgather"], 1_000_000, *weights) == (4, 1)


@pytest.mark.parametrize("k,op,mib,sums", ONCE_SUMS)
def test_how_far_programs_with_sums_on_the_way_have_one(rule, k, op, mib, sums):
    chain = list(range(-1, k - 1))
    line = int(mib * MIB / (MOVED[op](k) + 4 * sums))
    for fusion in (bl.BLINK_FUSE_EDGE, bl.BLINK_FUSE_NODE):
        for n, served in ((line - 4_099, 1), (line + 4_099, 0)):
            assert rule("once", OPS[op], fusion, n, 1 << 16, *chain) == (served,), (fusion, n)


@pytest.mark.parametrize("k", [2, 3, 5, 8])
def test_the_piece_that_a_gathers_root_keeps(rule, k):
    """No workgroups for it, unless it lies between pieces that move."""
    for m in (1, 5_003):
        for root in range(k):
            star = [-1 if v == root else root for v in range(k)]
            got = rule("flows", OPS["gather"], bl.BLINK_FUSE_TREE, k * m, 1 << 16, *star)
            want = [(v * m, m, int(v != root)) for v in range(k)]
            want = want[1:] if root == 0 else want[:-1] if root == k - 1 else want
            assert got == tuple(x for w in want for x in w), (m, root)


def test_what_a_caller_asks_for_comes_from_the_kernel_that_has_it(rule):
    """Beyond a few tiles per compute unit a way, a sweep that does not alternate and a grid are the drawing kernel's."""
    for small in (0, 1):
        for deps in (0, 1):
            assert rule("call", small, deps, 0, 0, 1) == (1,)
            for wg in (1, 4):
                assert rule("call", small, deps, wg, 0, 1) == (0,)
            for kernel, alternates in ((1, 1), (2, 1), (3, 1), (0, 0), (2, 0)):
                assert rule("call", small, deps, 0, kernel, alternates) == (int(small or deps),)


@pytest.mark.parametrize("n,chunk,own,shared", [(3_000_000, 1 << 16, 1, 1), (3_000_000, 1 << 17, 2, 2), (3_000_000, 1 << 20, 16, 16),
                                                (20_000_000, 1 << 17, 2, 1), (20_000_000, 1 << 22, 64, 1)])
def test_only_stages_that_hand_over_have_counters_for_pieces(rule, n, chunk, own, shared):
    """The kernels that carry a tile through all stages count none of them, so their blocks have no room for pieces; in the
    shared block chunks have one counter each where those of pieces do not fit (the last two)."""
    chain = list(range(-1, 15))
    in_cache = 16 * 4 * n <= 256 * MIB
    for fusion in (bl.BLINK_FUSE_EDGE, bl.BLINK_FUSE_NODE, bl.BLINK_FUSE_TREE):
        waits = [own, shared] if fusion != bl.BLINK_FUSE_TREE else [1, 1]
        as_served = waits if fusion == bl.BLINK_FUSE_EDGE and not in_cache else [1, 1]
        assert rule("counters", OPS["allreduce"], fusion, n, chunk, *chain) == tuple(as_served + waits), fusion


def test_sums_written_on_the_way(rule):
    """Of k ranks in a chain: per edge and per node all but the last, which is the result.  Two ranks have none."""
    for k in (2, 3, 8):
        chain = list(range(-1, k - 1))
        for op in ("allreduce", "reduce"):
            for fusion, sums in ((bl.BLINK_FUSE_EDGE, k - 2), (bl.BLINK_FUSE_NODE, k - 2), (bl.BLINK_FUSE_TREE, 0)):
                assert rule("sums", OPS[op], fusion, 1_003, 1 << 16, *chain) == (sums,), (k, op, fusion)
