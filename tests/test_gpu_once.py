"""The kernel with a workgroup for every tile: payloads around the lines where its tiles change (half and
whole ones, a few elements, a workgroup more on some compute unit), shares of different length, up to
four flows, up to sixteen and more, buffers off the 1 KiB grid, every operator.  Bit for bit against
the oracle, nothing written beside the buffers."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import execute as ox
from oracle import schedule as osch

from test_fold_rules import MOVED, ONCE_LINES, ONCE_SHARES, ONCE_SUMS, OPS
from test_gpu_fold import REDOPS, _slab, _stream, _tree

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1910_04940_amd as bl  # noqa: E402

CODES = {"fp32": bl.BLINK_FP32, "int32": bl.BLINK_INT32}


def _forest(k, weights):
    forest = [_tree(k, s) for s in range(len(weights))]
    roots, parents = [r for r, _ in forest], [p for _, p in forest]
    return bl.blink_trees_from_arrays(k, roots, parents, weights), roots, parents


# equal and unequal shares in the small and in the large arguments, one flow more than these hold, and
# shares so unequal that the general kernel serves
@pytest.mark.parametrize("weights", [w for w, _ in ONCE_SHARES], ids=lambda w: f"{len(w)} trees, {w[-1]:g}")
@pytest.mark.parametrize("k,op,dtype", [(2, "sum", "fp32"), (3, "max", "fp32"), (4, "sum", "fp32"), (5, "min", "int32"),
                                        (8, "sum", "int32"), (9, "prod", "fp32"), (16, "sum", "fp32")])
def test_shares(k, op, dtype, weights):
    stream = _stream()
    trees, roots, parents = _forest(k, weights)
    code, oracle_op = REDOPS[op]
    # traffic of 96 and 160 MiB is where half tiles, and a workgroup per tile, end on 256 compute units
    half, small = 96 * 2**20 // (8 * k), 160 * 2**20 // (8 * k)
    large = (half - 5, half + 4_099, small - 2_047) if len(weights) in (1, 3, 5) else (half + 4_099,) if len(weights) == 4 else ()
    for n in (7, 1_027, 65_539) + large:
        x = [si.hash_payload(83, r, 0, n, dtype) for r in range(k)]
        want = ox.tree_order_allreduce(x, roots, parents, weights, oracle_op)
        bufs, untouched = _slab(x)
        sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 16, bl.BLINK_FUSE_TREE)
        bl.blink_allreduce_op(bufs, n, CODES[dtype], code, sched, stream)
        torch.cuda.synchronize()
        for r in {0, k // 2, k - 1}:
            assert bufs[r].cpu().numpy().tobytes() == want.tobytes(), (n, r)
        assert untouched()


# sums written on the way, of every addition or of a node's last, and one rank written: where they lie in the arguments
# changes with the number of ranks (4, 8) and of flows
@pytest.mark.parametrize("n_trees", [1, 4, 16])
@pytest.mark.parametrize("k", [3, 4, 5, 8, 9, 16])
def test_sums_on_the_way_and_at_one_rank(k, n_trees):
    stream = _stream()
    trees, roots, parents = _forest(k, [1.0] * n_trees)
    w = [1.0] * n_trees
    for n in (5, 4_099, 16 * 2**20 // (8 * k), 100 * 2**20 // (8 * k) + 3):
        x = [si.hash_payload(103, r, 0, n, "int32") for r in range(k)]
        want = ox.allreduce_int32_definition(x)
        steps = osch.make_steps(roots, parents, w, osch.REDUCE_TO_ROOT, n, 1 << 16)
        left = [a.copy() for a in x]
        ox.run_steps(left, steps)
        for fusion in (bl.BLINK_FUSE_EDGE, bl.BLINK_FUSE_NODE, bl.BLINK_FUSE_TREE):
            bufs, untouched = _slab(x)
            sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 16, fusion)
            bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
            torch.cuda.synchronize()
            assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs) and untouched(), (n, fusion)
            bufs, untouched = _slab(x)
            sched = bl.blink_make_schedule(trees, bl.BLINK_OP_REDUCE, n, 1 << 16, fusion)
            bl.blink_reduce(bufs, n, bl.BLINK_INT32, bl.BLINK_SUM, sched, stream)
            torch.cuda.synchronize()
            b = sched.bounds()
            for r, got in enumerate(bufs):
                got = got.cpu().numpy()
                if fusion == bl.BLINK_FUSE_TREE:        # only the roots are written, each on its share
                    keep = x[r].copy()
                    for t, root in enumerate(roots):
                        if root == r:
                            keep[b[t]:b[t + 1]] = want[b[t]:b[t + 1]]
                    assert np.array_equal(got, keep), (n, r)
                else:                                   # a reduce leaves what the step list leaves
                    assert np.array_equal(got, left[r]), (n, fusion, r)
            assert untouched()


@pytest.mark.parametrize("past", [(16,) * 5, (528,) * 5, (1008,) * 5, (0, 16, 512, 1008, 64)])
def test_buffers_off_the_grid(past):
    """One schedule, called on buffers at different distances from a 1 KiB boundary."""
    stream = _stream()
    k, n = 5, 300_007
    trees, roots, parents = _forest(k, [1.0, 1.0])
    x = [si.hash_payload(89, r, 0, n, "int32") for r in range(k)]
    want = ox.allreduce_int32_definition(x)
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, 1 << 16, bl.BLINK_FUSE_TREE)
    for at in ((0,) * k, past, (0,) * k):
        step = (n + 1024) // 256 * 256 + 256
        whole = torch.zeros(k * step + 512, dtype=torch.int32, device="cuda")
        slab = whole[-whole.data_ptr() // 4 % 256:]
        bufs = [slab[r * step + at[r] // 4:][:n] for r in range(k)]
        for b, a in zip(bufs, x):
            b.copy_(torch.from_numpy(a))
        bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream)
        torch.cuda.synchronize()
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs)
        for b in bufs:
            b.zero_()
        assert int(torch.count_nonzero(whole)) == 0


@pytest.mark.parametrize("fusion", [bl.BLINK_FUSE_TREE, bl.BLINK_FUSE_EDGE])
@pytest.mark.parametrize("k", [2, 3, 5, 8, 9, 16])
def test_copies(k, fusion):
    """One rank read and copied to one, several or all others, to another number of them per piece (a
    per-edge Gather), pieces that begin and end anywhere, a root that keeps its own."""
    stream = _stream()
    trees, roots, _ = _forest(k, [1.0])
    root = roots[0]
    for m in (1, 3, 1_021, 30_011, 20 * 2**20 // (4 * k * k)):
        n = k * m
        x = [si.hash_payload(97, r, 0, n, "int32") for r in range(k)]
        gathered = ox.allgather_definition(x)
        for op, call, want in ((bl.BLINK_OP_BROADCAST, bl.blink_broadcast, [x[root]] * k),
                               (bl.BLINK_OP_ALLGATHER, bl.blink_allgather, [gathered] * k),
                               (bl.BLINK_OP_GATHER, bl.blink_gather, {root: gathered})):
            bufs, untouched = _slab(x)
            sched = bl.blink_make_schedule(trees, op, n, 1 << 12, fusion)
            call(bufs, n, bl.BLINK_INT32, sched, stream)
            torch.cuda.synchronize()
            for r in range(k):
                if not isinstance(want, dict) or r in want:
                    assert np.array_equal(bufs[r].cpu().numpy(), want[r]), (op, n, r)
                elif fusion == bl.BLINK_FUSE_TREE:      # a piece goes to the root alone
                    assert np.array_equal(bufs[r].cpu().numpy(), x[r]), (op, n, r)
            assert untouched()


def test_copies_along_trees_with_different_roots():
    """A Gather whose pieces go to a root per tree, some of which stay where they are."""
    stream = _stream()
    k, n = 3, 3 * 5_003
    trees = bl.blink_trees_from_arrays(k, [0, 1], [[-1, 0, 0], [1, -1, 1]], [1.0, 2.0])
    x = [si.hash_payload(101, r, 0, n, "int32") for r in range(k)]
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_GATHER, n, 1 << 12, bl.BLINK_FUSE_TREE)
    b = sched.bounds()
    bufs, untouched = _slab(x)
    bl.blink_gather(bufs, n, bl.BLINK_INT32, sched, stream)
    torch.cuda.synchronize()
    want = [a.copy() for a in x]
    for t, root in enumerate((0, 1)):
        for j in range(k):
            lo, hi = j * (n // k) + b[t], j * (n // k) + b[t + 1]
            want[root][lo:hi] = x[j][lo:hi]
    assert all(np.array_equal(a.cpu().numpy(), w) for a, w in zip(bufs, want)) and untouched()


# traffic on either side of where drawn tickets take over, on 256 compute units; with sums written on the way along a chain
@pytest.mark.parametrize("k,op,mib,sums", [line + (None,) for line in ONCE_LINES] + ONCE_SUMS)
def test_both_sides_of_the_line(k, op, mib, sums):
    stream = _stream()
    fusion = bl.BLINK_FUSE_TREE if sums is None else bl.BLINK_FUSE_EDGE
    trees, roots, _ = _forest(k, [1.0])
    if sums is not None:
        trees, roots = bl.blink_trees_from_arrays(k, [0], [list(range(-1, k - 1))], [1.0]), [0]
    root = roots[0]
    code, per = OPS[op], MOVED[op](k) + 4 * (sums or 0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    for n in (int(mib * 2**20 / per) - 4_099, int(mib * 2**20 / per) + 4_099):
        n -= n % k
        bufs = [torch.randint(-2**31, 2**31, (n,), dtype=torch.int32, device="cuda", generator=gen) for _ in range(k)]
        m = n // k
        if op in ("allreduce", "reduce"):
            want = bufs[0].clone()
            for b in bufs[1:]:
                want += b
        else:
            want = bufs[root].clone() if op == "broadcast" else torch.cat([b[r * m:(r + 1) * m] for r, b in enumerate(bufs)])
        sched = bl.blink_make_schedule(trees, code, n, 1 << 18, fusion)
        if op == "reduce":
            bl.blink_reduce(bufs, n, bl.BLINK_INT32, bl.BLINK_SUM, sched, stream)
        else:
            getattr(bl, "blink_" + op)(bufs, n, bl.BLINK_INT32, sched, stream)
        torch.cuda.synchronize()
        for r in ([root] if op in ("reduce", "gather") else range(k)):
            assert torch.equal(bufs[r], want), (n, r)


# payloads with a workgroup per tile that are more than a few tiles per compute unit: (ranks, collective, MiB of traffic)
@pytest.mark.parametrize("k,op,mib", [(8, "reduce", 180), (4, "reduce", 310), (8, "reduce", 318), (9, "reduce", 185), (3, "gather", 240),
                                      (4, "gather", 370), (8, "gather", 200), (4, "allgather", 185), (10, "allgather", 200)])
def test_wishes_beyond_a_few_tiles(k, op, mib):
    """A way, a sweep or a grid that a caller asks for is served with it, and right, then the usual call again."""
    stream = _stream()
    trees = bl.blink_trees_from_arrays(k, [0, 0], [[-1] + [0] * (k - 1), list(range(-1, k - 1))], [1.0, 1.0])   # a star and a chain
    n = int(mib * 2**20 / MOVED[op](k))
    n -= n % k
    m = n // k
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    x = [torch.randint(-2**31, 2**31, (n,), dtype=torch.int32, device="cuda", generator=gen) for _ in range(k)]
    if op == "reduce":
        want = x[0].clone()
        for b in x[1:]:
            want += b
    else:
        want = torch.cat([b[r * m:(r + 1) * m] for r, b in enumerate(x)])
    sched = bl.blink_make_schedule(trees, OPS[op], n, 1 << 18, bl.BLINK_FUSE_TREE)

    def call(way):
        bufs = [b.clone() for b in x]
        for _ in range(1 if op == "reduce" else 2):        # (a second gather finds what the first one left)
            if op == "reduce":
                bl.blink_reduce(bufs, n, bl.BLINK_INT32, bl.BLINK_SUM, sched, stream)
            else:
                getattr(bl, "blink_" + op)(bufs, n, bl.BLINK_INT32, sched, stream)
        assert sched.status()[0] == bl.BLINK_OK
        if way:
            assert sched.last_kernel == way
        for r in (range(k) if op == "allgather" else [0]):
            assert torch.equal(bufs[r], want), (way, r)

    call(1)
    for kernel, way in ((2, 2), (3, 1 if op == "reduce" and k > 8 else 3), (1, 1), (0, 1)):
        sched.set_kernel(kernel)
        call(way)
    sched.set_sweep(False)
    call(0)
    sched.set_sweep(True)
    sched.set_launch(2, 0)
    call(0)
    sched.set_launch(0, 0)
    sched.reset()
    call(1)
