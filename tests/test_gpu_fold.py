"""The kernel that carries a tile along its whole tree in one pass, at the sizes where
its tables, tiles and variants change: the edges of a tile and of a flow, one tile and
several per compute unit, tickets dealt out and drawn, every number of ranks, tables in
the kernel's arguments, in a wave's lanes and in memory, and the per-edge and
per-node programs, whose intermediate writes must be those of the step list.  Bit for
bit against the oracle."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import execute as ox
from oracle import schedule as osch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1910_04940_amd as bl  # noqa: E402

FUSIONS = {"edge": bl.BLINK_FUSE_EDGE, "node": bl.BLINK_FUSE_NODE, "tree": bl.BLINK_FUSE_TREE}
REDOPS = {"sum": (bl.BLINK_SUM, ox.SUM), "prod": (bl.BLINK_PROD, ox.PROD), "min": (bl.BLINK_MIN, ox.MIN),
          "max": (bl.BLINK_MAX, ox.MAX)}


def _stream():
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch.cuda.current_stream().cuda_stream


def _tree(k, seed):
    """A random tree on k ranks: its root and parents."""
    rng = np.random.default_rng([7, k, seed])
    order = [int(v) for v in rng.permutation(k)]
    parent = [-1] * k
    for i in range(1, k):
        parent[order[i]] = order[int(rng.integers(max(0, i - 3), i))]
    return order[0], parent


def _slab(x, guard=64):
    """Rank buffers inside one allocation, guard elements between them, and a check
    that nothing but the buffers was written."""
    n = len(x[0])
    step = (n + guard + 255) // 256 * 256
    slab = torch.zeros(len(x) * step, dtype=torch.int32, device="cuda")
    bufs = [slab[r * step:r * step + n] for r in range(len(x))]
    for b, a in zip(bufs, x):
        b.copy_(torch.from_numpy(a.view(np.int32)))

    def untouched():
        return all(int(torch.count_nonzero(slab[r * step + n:(r + 1) * step])) == 0 for r in range(len(x)))
    return bufs, untouched


@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("k", range(2, 17))
def test_every_number_of_ranks_at_the_edges_of_a_tile(k, fusion):
    """One random tree; payloads of a few elements, one element around a tile of
    4 * U KiB for U = 1, 2, 3, 4, 6 and 8, and three tiles and a ragged end."""
    stream = _stream()
    root, parent = _tree(k, 0)
    trees = bl.blink_trees_from_arrays(k, [root], [parent], [1.0])
    for n in (1, 3, 4, 5, 255, 1023, 1024, 1025, 2047, 2049, 3073, 4097, 6145, 8191, 8193, 25_003):
        x = [si.hash_payload(11, r, 0, n, "fp32") for r in range(k)]
        want = ox.tree_order_allreduce(x, [root], [parent], [1.0])
        bufs, untouched = _slab(x)
        sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1000, FUSIONS[fusion])
        bl.blink_allreduce(bufs, n, bl.BLINK_FP32, sched, stream)
        torch.cuda.synchronize()
        for r, b in enumerate(bufs):
            assert b.cpu().numpy().tobytes() == want.tobytes(), (k, fusion, n, r)
        assert untouched()


# elements per rank: half tiles, whole tiles, a workgroup per tile, drawn tickets, larger than the memory-side cache
@pytest.mark.parametrize("n", [70_001, 1_100_003, 2_000_006, 3_000_001, 9_000_002])
@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("op,dtype", [("sum", "int32"), ("max", "int32"), ("min", "fp32"), ("prod", "int32")])
def test_sizes_where_the_launch_changes(n, fusion, op, dtype):
    """8 ranks, 4 packed trees; two calls in place (a whole-tree call's second goes backwards)."""
    stream = _stream()
    top = si.hybrid_cube_mesh()
    trees = bl.blink_pack_trees(top.k, top.src, top.dst, top.cap, 0)
    roots, parents, w = trees.as_lists()
    code, oracle_op = REDOPS[op]
    x = [si.hash_payload(13, r, 0, n, dtype) for r in range(top.k)]
    bufs, untouched = _slab(x)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 16, FUSIONS[fusion])
    for call in range(2):
        want = ox.tree_order_allreduce(x, roots, parents, w, oracle_op)
        x = [want] * top.k
        bl.blink_allreduce_op(bufs, n, bl.BLINK_INT32 if dtype == "int32" else bl.BLINK_FP32, code, sched, stream)
        torch.cuda.synchronize()
        for r in (0, 3, 7):
            assert bufs[r].cpu().numpy().tobytes() == want.tobytes(), (call, r)
    assert untouched()
    assert sched.status()[0] == bl.BLINK_OK


# a copy's columns per wave follow the ranks written and the traffic: two (a workgroup per tile, or more
# than eight ranks written), three (more than six), four, eight and sixteen (by what the copy moves)
@pytest.mark.parametrize("k,sizes", [(2, (41_000_002, 43_000_002)), (3, (2_000_003, 12_000_001, 20_000_003, 23_000_003)),
                                     (8, (1_500_003, 6_000_001)), (10, (600_003, 4_500_003))])
def test_copies_of_every_width(k, sizes):
    """Broadcast from, and Gather to, the middle of a star; two calls, the second goes backwards."""
    stream = _stream()
    trees = bl.blink_trees_from_arrays(k, [1], [[-1 if r == 1 else 1 for r in range(k)]], [1.0])
    rng = torch.Generator(device="cuda")
    rng.manual_seed(k)
    for n in sizes:
        m = n - n % k
        slab = torch.zeros(k, n + 64 - n % 64 + 64, dtype=torch.int32, device="cuda")
        bufs = [slab[r, :n] for r in range(k)]
        bcast = bl.blink_make_schedule(trees, bl.BLINK_OP_BROADCAST, n, 1 << 18)
        gather = bl.blink_make_schedule(trees, bl.BLINK_OP_GATHER, m, 1 << 18)
        for _ in range(2):
            for b in bufs:
                b.random_(generator=rng)
            want = bufs[1].clone()
            bl.blink_broadcast(bufs, n, bl.BLINK_INT32, bcast, stream)
            assert all(torch.equal(b, want) for b in bufs), n
            for b in bufs:
                b.random_(generator=rng)
            others = [b.clone() for b in bufs]
            want = torch.cat([others[r][r * (m // k):(r + 1) * (m // k)] for r in range(k)] + [others[1][m:]])
            bl.blink_gather(bufs, m, bl.BLINK_INT32, gather, stream)
            assert torch.equal(bufs[1], want), n
            assert all(torch.equal(bufs[r], others[r]) for r in range(k) if r != 1), n
        assert int(torch.count_nonzero(slab[:, n:])) == 0


@pytest.mark.parametrize("fusion", ["edge", "node"])
@pytest.mark.parametrize("k", [3, 5, 8, 13, 16])
@pytest.mark.parametrize("n", [4_099, 300_002])
def test_a_reduce_leaves_what_the_program_writes_on_the_way(k, n, fusion):
    """The reduce phase alone: every rank's buffer, not only the root's, holds what
    the step list leaves there.  The per-edge program writes a vertex's running sum
    after every child and the per-node program once, so both leave the vertex's sum."""
    stream = _stream()
    forest = [_tree(k, s) for s in range(3)]
    roots, parents, w = [r for r, _ in forest], [p for _, p in forest], [1.0, 2.0, 1.5]
    trees = bl.blink_trees_from_arrays(k, roots, parents, w)
    x = [si.payload(17, r, n, "uniform", "fp32") for r in range(k)]
    want = [a.copy() for a in x]
    ox.run_steps(want, osch.make_steps(roots, parents, w, osch.REDUCE_TO_ROOT, n, 5_000))
    bufs, untouched = _slab(x)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_REDUCE, n, 5_000, FUSIONS[fusion])
    bl.blink_reduce(bufs, n, bl.BLINK_FP32, bl.BLINK_SUM, sched, stream)
    torch.cuda.synchronize()
    for r, b in enumerate(bufs):
        assert b.cpu().numpy().tobytes() == want[r].tobytes(), r
    assert untouched()


@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("op", ["broadcast", "reduce", "allreduce"])
@pytest.mark.parametrize("n", [5_003, 400_001])
def test_a_star_has_several_stages_that_wait_for_nothing(op, fusion, n):
    """Two stars round one centre: the per-edge broadcast is five copies per chunk and tree
    without a dependency among them."""
    stream = _stream()
    k, root = 6, 2
    parent = [root] * k
    parent[root] = -1
    trees = bl.blink_trees_from_arrays(k, [root, root], [parent, parent], [1.0, 1.0])
    x = [si.hash_payload(19, r, 0, n, "int32") for r in range(k)]
    bufs, untouched = _slab(x)
    which = {"broadcast": bl.BLINK_OP_BROADCAST, "reduce": bl.BLINK_OP_REDUCE, "allreduce": bl.BLINK_OP_ALLREDUCE}[op]
    sched = bl.blink_make_schedule(trees, which, n, 1_000, FUSIONS[fusion])
    if op == "broadcast":
        bl.blink_broadcast(bufs, n, bl.BLINK_INT32, sched, stream)
        want = [x[root]] * k
    elif op == "reduce":
        bl.blink_reduce(bufs, n, bl.BLINK_INT32, bl.BLINK_SUM, sched, stream)
        want = list(x)
        want[root] = ox.allreduce_int32_definition(x)
    else:
        bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
        want = [ox.allreduce_int32_definition(x)] * k
    torch.cuda.synchronize()
    for r, b in enumerate(bufs):
        assert np.array_equal(b.cpu().numpy(), want[r]), r
    assert untouched()


@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("k,n_trees", [(4, 1), (5, 3), (8, 8), (16, 16)])
@pytest.mark.parametrize("m", [5, 1_237, 70_001])
def test_allgather_with_few_and_many_flows(k, n_trees, m, fusion):
    """4, 15, 64 and 256 flows: tables in the arguments, in a wave's lanes and in memory."""
    stream = _stream()
    n = k * m
    forest = [_tree(k, s) for s in range(n_trees)]
    trees = bl.blink_trees_from_arrays(k, [r for r, _ in forest], [p for _, p in forest], [1.0] * n_trees)
    x = [si.hash_payload(23, r, 0, n, "int32") for r in range(k)]
    want = ox.allgather_definition(x)
    bufs, untouched = _slab(x)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLGATHER, n, 4_096, FUSIONS[fusion])
    for _ in range(2):
        bl.blink_allgather(bufs, n, bl.BLINK_INT32, sched, stream)
    torch.cuda.synchronize()
    for r, b in enumerate(bufs):
        assert np.array_equal(b.cpu().numpy(), want), r
    assert untouched()


@pytest.mark.parametrize("fusion", ["node", "tree"])
@pytest.mark.parametrize("wg,tile", [(1, 256), (2, 1024), (0, 16_384), (4, 65_536)])
def test_launch_overrides(fusion, wg, tile):
    """Tiles smaller and larger than the kernel's own, few and many workgroups, then automatic again."""
    stream = _stream()
    top = si.hybrid_cube_mesh()
    trees = bl.blink_pack_trees(top.k, top.src, top.dst, top.cap, 0)
    n = 1_000_003
    x = [si.hash_payload(29, r, 0, n, "int32") for r in range(top.k)]
    want = ox.allreduce_int32_definition(x).view(np.uint32).astype(np.uint64)
    bufs, untouched = _slab(x)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 16, FUSIONS[fusion])
    for call, launch in enumerate([(0, 0), (wg, tile), (wg, tile), (0, 0)]):
        sched.set_launch(*launch)
        bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
        torch.cuda.synchronize()
        expect = ((want * np.uint64(pow(8, call, 1 << 32))) & np.uint64(0xFFFFFFFF)).astype(np.uint32)
        for r in (0, 5):
            assert np.array_equal(bufs[r].cpu().numpy().view(np.uint32), expect), (call, r)
    assert untouched()


@pytest.mark.parametrize("before,after", [(65_536, 256), (256, 65_536), (256, 1024), (0, 256)])
def test_tile_sizes_of_calls_that_allocate_nothing(before, after):
    """Six shares of different lengths: one stretch of tile positions with large tiles, which
    travels with the launch, six with small ones, which lie in the block that such calls share."""
    stream = _stream()
    k, n = 4, 100_003
    forest = [_tree(k, seed) for seed in range(6)]
    trees = bl.blink_trees_from_arrays(k, [r for r, _ in forest], [p for _, p in forest], [1.0, 2.0, 3.0, 4.0, 5.0, 6.0])
    x = [si.hash_payload(37, r, 0, n, "int32") for r in range(k)]
    want = ox.allreduce_int32_definition(x)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 20, bl.BLINK_FUSE_TREE)
    for tile in (before, after, before):
        sched.set_launch(0, tile)
        bufs, untouched = _slab(x)
        bl.blink_allreduce_noalloc(bufs, n, bl.BLINK_INT32, sched, stream)
        torch.cuda.synchronize()
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs), tile
        assert untouched()


def test_waiting_stages_after_calls_that_did_not_wait():
    """A per-node schedule that has run on this kernel hands chunks over once a call has been
    skipped, and is itself again after a reset."""
    stream = _stream()
    top = si.hybrid_cube_mesh()
    trees = bl.blink_pack_trees(top.k, top.src, top.dst, top.cap, 0)
    n = 3_000_001       # drawn tickets: the block's counters have moved
    x = [si.hash_payload(31, r, 0, n, "int32") for r in range(top.k)]
    want = ox.allreduce_int32_definition(x)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 16, bl.BLINK_FUSE_NODE)

    def call():
        bufs, untouched = _slab(x)
        bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
        torch.cuda.synchronize()
        return bufs, untouched
    for _ in range(2):
        bufs, untouched = call()
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs) and untouched()
    sched.set_wait_limit(2000)
    sched.test_skip_call()
    call()
    st, rec = sched.status()
    assert st == bl.BLINK_ESTUCK and rec["call"] == 4 and rec["seen"] < rec["wanted"]
    sched.reset()
    sched.set_wait_limit(0)
    for _ in range(2):
        bufs, untouched = call()
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs) and untouched()
    assert sched.status()[0] == bl.BLINK_OK


def test_the_timed_choice_compares_like_with_like():
    """A job that alternates sums and maxima on one schedule: either kind of call goes round the
    ways by itself.  Another sweep mode has a choice of its own, and calls that allocate nothing
    use the pick."""
    stream = _stream()
    k, n = 7, 4_000_001
    root, parent = _tree(k, 1)
    trees = bl.blink_trees_from_arrays(k, [root], [parent], [1.0])
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 18, bl.BLINK_FUSE_TREE)
    bufs = [torch.ones(n, dtype=torch.int32, device="cuda") for _ in range(k)]
    seen = {bl.BLINK_SUM: [], bl.BLINK_MAX: []}
    value = 1

    def call(op):
        nonlocal value
        bl.blink_allreduce_op(bufs, n, bl.BLINK_INT32, op, sched, stream)
        value = (value * k) % (1 << 32) if op == bl.BLINK_SUM else value
        return sched.last_kernel

    for i in range(22):
        op = (bl.BLINK_SUM, bl.BLINK_MAX)[i % 2]
        seen[op].append(call(op))
    picked = seen[bl.BLINK_SUM][-1]
    for ways in seen.values():
        assert ways[:8] == [1, 2] * 4 and set(ways[8:]) == {picked}
    bl.blink_allreduce_noalloc(bufs, n, bl.BLINK_INT32, sched, stream)
    value = (value * k) % (1 << 32)
    assert sched.last_kernel == picked
    sched.set_sweep(False)
    assert [call(bl.BLINK_MAX) for _ in range(8)] == [1, 2] * 4
    torch.cuda.synchronize()
    for b in bufs:
        assert int(b.min()) == int(b.max()) and int(b.min()) % (1 << 32) == value


@pytest.mark.parametrize("n_trees", [1, 6])
@pytest.mark.parametrize("k,n", [(4, 9_000_005), (6, 5_000_003), (8, 6_000_002)])
def test_sums_and_other_operators_by_turns(k, n, n_trees):
    """Drawn tickets, from two counters where a ticket is small (four and six ranks) and from one: calls of all operators on
    one schedule, with its tables in the arguments (one tree) and on the device (six)."""
    stream = _stream()
    forest = [_tree(k, s) for s in range(n_trees)]
    roots, parents, w = [r for r, _ in forest], [p for _, p in forest], [1.0 + s for s in range(n_trees)]
    trees = bl.blink_trees_from_arrays(k, roots, parents, w)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 16, bl.BLINK_FUSE_TREE)
    x = [si.hash_payload(17, r, 0, n, "int32") for r in range(k)]
    bufs, untouched = _slab(x)
    for op in ("sum", "max", "sum", "prod", "min", "sum"):
        code, oracle_op = REDOPS[op]
        want = ox.tree_order_allreduce(x, roots, parents, w, oracle_op)
        bl.blink_allreduce_op(bufs, n, bl.BLINK_INT32, code, sched, stream)
        torch.cuda.synchronize()
        assert all(b.cpu().numpy().tobytes() == want.tobytes() for b in bufs), op
        x = [si.hash_payload(19, r, len(op), n, "int32") for r in range(k)]
        for b, a in zip(bufs, x):
            b.copy_(torch.from_numpy(a))
    assert untouched()
    assert sched.status()[0] == bl.BLINK_OK


def _drawn_elems(traffic_per_elem):
    """Elements per rank, ragged, of a payload just too large to have a workgroup for every tile."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return int(1.04 * 5 * 128 * 1024 * cus / traffic_per_elem) // 4 * 4 + 3


def _random(k, n, dtype, rng):
    """k rank buffers in one allocation with 64 guard elements behind each."""
    step = (n + 64 + 255) // 256 * 256
    slab = torch.zeros(k * step, dtype=torch.int32, device="cuda")
    bufs = [slab[r * step:r * step + n].view(torch.float32 if dtype == "fp32" else torch.int32) for r in range(k)]
    for b in bufs:
        b.normal_(generator=rng) if dtype == "fp32" else b.random_(-2 ** 31, 2 ** 31, generator=rng)
    return bufs, lambda: int(torch.count_nonzero(slab.view(k, step)[:, n:])) == 0


def _in_tree_order(x, root, parent, op):
    """The oracle's recursion along one tree, on the device, with a stretch of it checked against the oracle."""
    combine = {"sum": torch.add, "max": torch.maximum}[op]

    def total(v):
        acc = x[v]
        for c in range(len(parent)):
            if parent[c] == v:
                acc = combine(acc, total(c))
        return acc
    out = total(root)
    at = out.numel() // 3
    want = ox.tree_order_allreduce([b[at:at + 2000].cpu().numpy() for b in x], [root], [parent], [1.0], REDOPS[op][1])
    assert out[at:at + 2000].cpu().numpy().tobytes() == want.tobytes()
    return out


def _same_bits(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("fusion", ["node", "tree"])
@pytest.mark.parametrize("k", range(2, 17))
def test_drawn_tickets_with_every_number_of_ranks(k, fusion):
    """AllReduce and Reduce, sums and maxima of both types by turns on one schedule, with results that may stay in the
    memory-side cache; sums that stream past it (whole-tree programs of more than a cache, calls all forwards)."""
    stream = _stream()
    rng = torch.Generator(device="cuda")
    rng.manual_seed(k)
    root, parent = _tree(k, 1)
    trees = bl.blink_trees_from_arrays(k, [root], [parent], [1.0])
    cases = [("allreduce", _drawn_elems(8 * k), False), ("reduce", _drawn_elems(4 * (k + 1)), False)]
    if fusion == "tree":
        cases.append(("allreduce", (260 << 20) // (4 * k) + 1, True))
    for which, n, streams in cases:
        sched = bl.blink_make_schedule(trees, bl.BLINK_OP_REDUCE if which == "reduce" else bl.BLINK_OP_ALLREDUCE, n, 1 << 16,
                                       FUSIONS[fusion])
        if streams:
            sched.set_sweep(False)
        for op, dtype in (("sum", "fp32"), ("max", "int32"), ("sum", "int32"), ("max", "fp32")):
            if streams and op == "max":
                continue
            bufs, untouched = _random(k, n, dtype, rng)
            want = _in_tree_order([b.clone() for b in bufs], root, parent, op)
            code = bl.BLINK_FP32 if dtype == "fp32" else bl.BLINK_INT32
            if which == "reduce":
                bl.blink_reduce(bufs, n, code, REDOPS[op][0], sched, stream)
            else:
                bl.blink_allreduce_op(bufs, n, code, REDOPS[op][0], sched, stream)
            for r in [root] if which == "reduce" else range(k):
                assert _same_bits(bufs[r], want), (which, n, op, dtype, r)
            assert untouched()
        assert sched.status()[0] == bl.BLINK_OK


# MiB moved: where a payload ceases to have a workgroup for every tile, where it ceases to fit the memory-side cache and
# at twice that a copy's columns and its way of writing change
@pytest.mark.parametrize("moved", [150, 170, 240, 300, 530])
@pytest.mark.parametrize("k", [2, 4, 5, 6])
def test_copies_on_both_sides_of_their_lines(k, moved):
    """Broadcast from, and Gather to, the middle of a star; forwards only, where results stream, and in way 2."""
    stream = _stream()
    trees = bl.blink_trees_from_arrays(k, [1], [[-1 if r == 1 else 1 for r in range(k)]], [1.0])
    rng = torch.Generator(device="cuda")
    rng.manual_seed(moved)
    n = (moved << 20) // (4 * k) + 3
    m = (moved << 20) // (8 * (k - 1)) * k
    for way in (1, 2):
        for op, size, sweep in ((bl.BLINK_OP_BROADCAST, n, True), (bl.BLINK_OP_GATHER, m, True), (bl.BLINK_OP_GATHER, m, False)):
            sched = bl.blink_make_schedule(trees, op, size, 1 << 18)
            sched.set_kernel(way)
            sched.set_sweep(sweep)
            bufs, untouched = _random(k, size, "int32", rng)
            before = [b.clone() for b in bufs]
            for _ in range(2):
                if op == bl.BLINK_OP_BROADCAST:
                    bl.blink_broadcast(bufs, size, bl.BLINK_INT32, sched, stream)
                    assert all(torch.equal(b, before[1]) for b in bufs)
                else:
                    bl.blink_gather(bufs, size, bl.BLINK_INT32, sched, stream)
                    piece = size // k
                    for r in range(k):
                        assert torch.equal(bufs[1][r * piece:(r + 1) * piece], before[r][r * piece:(r + 1) * piece]), r
                    assert all(torch.equal(bufs[r], before[r]) for r in range(k) if r != 1)
            assert untouched()
            assert sched.status()[0] == bl.BLINK_OK
