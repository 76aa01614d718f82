"""Stages that hand chunks over to one another (one wavefront's result is the next one's input,
through counters and memory), asked for at the sizes where the library would serve the
program in one pass: ragged payloads and ends, chunks that do not start on 16-byte boundaries,
every number of ranks a stage can read, every collective, calls on the shared block, recorded calls.
Every test asserts that chunks were handed over where a stage depends on another.  Bit for bit against the oracle."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import execute as ox
from oracle import multiserver as om
from oracle import schedule as osch

from test_gpu_fold import REDOPS, _slab, _tree
from test_host_multiserver import make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1910_04940_amd as bl  # noqa: E402

FUSIONS = {"edge": bl.BLINK_FUSE_EDGE, "node": bl.BLINK_FUSE_NODE}
CODES = {"fp32": bl.BLINK_FP32, "int32": bl.BLINK_INT32}


def _stream():
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch.cuda.current_stream().cuda_stream


def _forest(k, n_trees):
    forest = [_tree(k, s) for s in range(n_trees)]
    roots, parents, w = [r for r, _ in forest], [p for _, p in forest], [1.0 + t for t in range(n_trees)]
    return bl.blink_trees_from_arrays(k, roots, parents, w), roots, parents, w


def _schedule(trees, op, n, chunk, fusion):
    sched = bl.blink_make_schedule(trees, op, n, chunk, FUSIONS[fusion])
    sched.set_hand_over(True)
    return sched


# chunks of whole and of odd elements; payloads below, at and above a few of them, ragged
@pytest.mark.parametrize("n,chunk", [(13, 5), (4_099, 1_000), (70_003, 4_096), (70_003, 1_001), (300_001, 33_333)])
@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("k", [2, 3, 5, 8, 12, 16])
def test_allreduce(k, fusion, n, chunk):
    stream = _stream()
    trees, roots, parents, w = _forest(k, 3)
    sched = _schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, fusion)
    depends = k > 2 or fusion == "edge"       # two ranks per node: a single stage
    for dtype in CODES:
        x = [si.hash_payload(61, r, 0, n, dtype) for r in range(k)]
        want = ox.tree_order_allreduce(x, roots, parents, w)
        bufs, untouched = _slab(x)
        bl.blink_allreduce(bufs, n, CODES[dtype], sched, stream)
        assert sched.status()[0] == bl.BLINK_OK and sched.handed_over == int(depends)
        for r, b in enumerate(bufs):
            assert b.cpu().numpy().tobytes() == want.tobytes(), (dtype, r)
        assert untouched()


@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("op,dtype", [("max", "int32"), ("min", "fp32"), ("prod", "int32"), ("prod", "fp32")])
def test_other_operators(op, dtype, fusion):
    stream = _stream()
    k, n = 9, 50_003
    trees, roots, parents, w = _forest(k, 2)
    code, oracle_op = REDOPS[op]
    x = [si.hash_payload(67, r, 0, n, dtype) for r in range(k)]
    want = ox.tree_order_allreduce(x, roots, parents, w, oracle_op)
    bufs, untouched = _slab(x)
    sched = _schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 2_047, fusion)
    bl.blink_allreduce_op(bufs, n, CODES[dtype], code, sched, stream)
    assert sched.status()[0] == bl.BLINK_OK and sched.handed_over == 1
    assert all(b.cpu().numpy().tobytes() == want.tobytes() for b in bufs) and untouched()


@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("k", [4, 7, 16])
def test_the_other_collectives(k, fusion):
    stream = _stream()
    n, chunk = k * 5_003, 1_021
    trees, roots, parents, w = _forest(k, 1)      # one root for broadcast and gather
    root = roots[0]
    x = [si.hash_payload(71, r, 0, n, "int32") for r in range(k)]
    gathered = ox.allgather_definition(x)
    for op, call, want in (
            (bl.BLINK_OP_BROADCAST, bl.blink_broadcast, [x[root]] * k),
            (bl.BLINK_OP_ALLGATHER, bl.blink_allgather, [gathered] * k),
            (bl.BLINK_OP_GATHER, bl.blink_gather, {root: gathered})):
        bufs, untouched = _slab(x)
        sched = _schedule(trees, op, n, chunk, fusion)
        depends = any(int(s["n_dep"]) for s in sched.stages())
        call(bufs, n, bl.BLINK_INT32, sched, stream)
        assert sched.status()[0] == bl.BLINK_OK and sched.handed_over == int(depends)
        for r in range(k):
            if not isinstance(want, dict) or r in want:
                assert np.array_equal(bufs[r].cpu().numpy(), want[r]), (op, r)
        assert untouched()
    # a reduce leaves in every rank's buffer what the step list leaves there
    left = [a.copy() for a in x]
    ox.run_steps(left, osch.make_steps(roots, parents, w, osch.REDUCE_TO_ROOT, n, chunk))
    bufs, untouched = _slab(x)
    sched = _schedule(trees, bl.BLINK_OP_REDUCE, n, chunk, fusion)
    bl.blink_reduce(bufs, n, bl.BLINK_INT32, bl.BLINK_SUM, sched, stream)
    assert sched.status()[0] == bl.BLINK_OK and sched.handed_over == 1
    assert all(np.array_equal(b.cpu().numpy(), a) for b, a in zip(bufs, left)) and untouched()


@pytest.mark.parametrize("layout", ["8+8", "3+5 interleaved"])
@pytest.mark.parametrize("fusion", FUSIONS)
def test_three_phases_across_servers(layout, fusion):
    stream = _stream()
    n, chunk = 100_003, 4_099
    sched, servers = make(layout, n, chunk, FUSIONS[fusion])
    sched.set_hand_over(True)
    k = sum(len(s.ranks) for s in servers)
    x = [si.payload(73, r, n, "uniform", "fp32") for r in range(k)]
    want = om.three_phase_allreduce(x, servers)
    bufs, untouched = _slab(x)
    bl.blink_allreduce(bufs, n, bl.BLINK_FP32, sched, stream)
    assert sched.status()[0] == bl.BLINK_OK and sched.handed_over == 1
    assert all(b.cpu().numpy().tobytes() == want.tobytes() for b in bufs) and untouched()


@pytest.mark.parametrize("fusion", FUSIONS)
@pytest.mark.parametrize("n_trees", [2, 6])
def test_the_shared_block_and_recorded_calls(fusion, n_trees):
    """Calls on the block and a recorded one, replayed with the program's own work in between; then
    the same schedule served in one pass on the same block, and back."""
    stream = _stream()
    k, n, chunk = 6, 60_001, 2_500
    trees, _, _, _ = _forest(k, n_trees)
    x = [si.hash_payload(79, r, 0, n, "int32") for r in range(k)]
    want = ox.allreduce_int32_definition(x)
    sched = _schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, fusion)
    src = [torch.from_numpy(a).to("cuda") for a in x]
    bufs = [b.clone() for b in src]

    def check():
        torch.cuda.synchronize()
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs)
        assert sched.status()[0] == bl.BLINK_OK
        for b, s0 in zip(bufs, src):
            b.copy_(s0)
        torch.cuda.synchronize()

    bl.blink_allreduce_noalloc(bufs, n, bl.BLINK_INT32, sched, stream)
    assert sched.handed_over == 1
    check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bl.blink_allreduce_noalloc(bufs, n, bl.BLINK_INT32, sched, torch.cuda.current_stream().cuda_stream)
    for _ in range(4):
        graph.replay()
        check()
        bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)     # on the schedule's own block
        assert sched.handed_over == 1
        check()
    for always in (False, True):
        sched.set_hand_over(always)
        for call in (bl.blink_allreduce_noalloc, bl.blink_allreduce):
            call(bufs, n, bl.BLINK_INT32, sched, stream)
            assert sched.handed_over == int(always)
            check()


def test_what_the_switch_takes():
    top = si.hybrid_cube_mesh()
    trees = bl.blink_pack_trees(top.k, top.src, top.dst, top.cap, 0)
    tree = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, 4_096, 1_024, bl.BLINK_FUSE_TREE)
    assert tree.handed_over == -1
    tree.set_hand_over(True)          # no stage waits for another: nothing to hand over
    bufs = [torch.ones(4_096, dtype=torch.int32, device="cuda") for _ in range(8)]
    bl.blink_allreduce(bufs, 4_096, bl.BLINK_INT32, tree, _stream())
    assert tree.handed_over == 0 and int(bufs[3].min()) == int(bufs[3].max()) == 8
    edge = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, 4_096, 1_024, bl.BLINK_FUSE_EDGE)
    assert edge.kernel_bytes < edge.traffic_bytes
    edge.set_hand_over(True)
    assert edge.kernel_bytes == edge.traffic_bytes


# chunks that are handed on in pieces of 65,536 elements: whole and odd numbers of them, tiles as large as a
# piece and as small as they get
@pytest.mark.parametrize("n,chunk", [(300_007, 131_072), (1_000_003, 200_001), (1_000_003, 1 << 20), (500_001, 131_071)])
@pytest.mark.parametrize("tile", [0, 256, 65_536])
def test_chunks_in_pieces(n, chunk, tile):
    stream = _stream()
    k = 5
    trees, _, _, _ = _forest(k, 2)
    x = [si.hash_payload(107, r, 0, n, "int32") for r in range(k)]
    want = ox.allreduce_int32_definition(x)
    sched = _schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, "edge")
    sched.set_launch(0, tile)
    for call in (bl.blink_allreduce, bl.blink_allreduce, bl.blink_allreduce_noalloc, bl.blink_allreduce):
        bufs, untouched = _slab(x)
        call(bufs, n, bl.BLINK_INT32, sched, stream)
        assert sched.status()[0] == bl.BLINK_OK and sched.handed_over == 1
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs) and untouched()


def _in_place(sched, k, n, calls):
    """Calls on device data, each against torch's sum."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    x = [torch.randint(-2**31, 2**31, (n,), dtype=torch.int32, device="cuda", generator=gen) for _ in range(k)]
    want = x[0].clone()
    for b in x[1:]:
        want += b
    bufs = [torch.empty_like(b) for b in x]
    for call in calls:
        for b, a in zip(bufs, x):
            b.copy_(a)
        call(bufs, n, bl.BLINK_INT32, sched, _stream())
        assert sched.status()[0] == bl.BLINK_OK
        assert all(torch.equal(b, want) for b in bufs)
        yield


def test_more_pieces_than_the_shared_block_has_counters_for():
    """A chunk has one counter there and a counter per piece in the schedule's own block."""
    k, n, chunk = 16, 17_000_003, 131_072
    trees = bl.blink_trees_from_arrays(k, [0], [list(range(-1, k - 1))], [1.0])
    sched = _schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, "edge")
    assert sched.num_stages * (2 * 256 + 56) > 2 << 20      # two counters and the stage itself
    for _ in _in_place(sched, k, n, [bl.blink_allreduce_noalloc, bl.blink_allreduce, bl.blink_allreduce_noalloc, bl.blink_allreduce,
                                     bl.blink_allreduce]):
        assert sched.handed_over == 1


def test_a_block_grows_with_the_pieces():
    """Tickets are drawn from a block without counters of pieces; where waiting stages are asked for later it is made anew."""
    k, n, chunk = 6, 6_000_007, 1 << 20
    trees, _, _, _ = _forest(k, 2)
    sched = _schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, "node")
    served = [0, 0, 1, 1, 1, 0, 1, 1]
    calls = _in_place(sched, k, n, [bl.blink_allreduce] * 4 + [bl.blink_allreduce_noalloc] + [bl.blink_allreduce] * 3)
    for handed_over in served:
        sched.set_hand_over(bool(handed_over))
        next(calls)
        assert sched.handed_over == handed_over


def test_an_abandoned_wait_names_the_chunks_stages():
    """Counters of pieces, reported as those of the stage; a reset clears them all."""
    stream = _stream()
    k, n, chunk = 6, 700_001, 262_144
    trees, _, _, _ = _forest(k, 2)
    x = [si.hash_payload(109, r, 0, n, "int32") for r in range(k)]
    want = ox.allreduce_int32_definition(x)
    sched = _schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, "edge")
    bufs, _ = _slab(x)
    bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
    assert sched.status()[0] == bl.BLINK_OK
    sched.set_wait_limit(2000)
    sched.test_skip_call()
    bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
    st, rec = sched.status()
    stages = sched.stages()
    assert st == bl.BLINK_ESTUCK and rec["call"] == 3
    assert rec["awaited_stage"] in [int(d) for d in stages[rec["stage"]]["deps"][:stages[rec["stage"]]["n_dep"]]]
    assert rec["wanted"] % 3 == 0 and rec["seen"] <= rec["wanted"] // 3 * 2
    sched.reset()
    sched.set_wait_limit(0)
    for _ in range(2):
        bufs, _ = _slab(x)
        bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
        assert sched.status()[0] == bl.BLINK_OK
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs)
