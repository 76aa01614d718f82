"""GPU parity at the full sizes of the benchmark configurations, in the launch
configuration bench.py times (defaults).  Small enough cases are compared in
full; the 16 GiB switch case on sampled slices the oracle computes one by one,
plus properties that hold at any size (all ranks identical)."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import execute as ox
from oracle import schedule as osch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1910_04940_amd as bl  # noqa: E402

FUSION = {"edge": bl.BLINK_FUSE_EDGE, "node": bl.BLINK_FUSE_NODE, "tree": bl.BLINK_FUSE_TREE}


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available()
    d = torch.device("cuda:0")
    torch.cuda.set_device(d)
    return d


def stream():
    return torch.cuda.current_stream().cuda_stream


def pack(top, root):
    return bl.blink_pack_trees(top.k, top.src, top.dst, top.cap, root)


def bits(a):
    return a.view(np.uint32)


@pytest.mark.parametrize("fusion", ["tree", "node", "edge"])
@pytest.mark.parametrize("layout", ["separate", "slab"])
def test_headline_8_ranks_cube_mesh_256MiB_fp32(dev, fusion, layout):
    """The benchmark's workload, every element of every rank against the oracle,
    with one allocation per rank buffer and with the benchmark's own placement
    (one allocation, consecutive rank buffers a little further apart than the
    payload); there the gaps between the buffers must come back untouched."""
    import bench
    top = si.hybrid_cube_mesh()
    n, chunk = 1 << 26, 1 << 18
    trees = pack(top, 0)
    roots, parents, w = trees.as_lists()
    assert trees.count == 4 and w == [1.0] * 4
    x = [si.payload(0, r, n, "uniform", "fp32") for r in range(8)]
    if layout == "separate":
        bufs = [torch.from_numpy(a).to(dev) for a in x]
    else:
        stride = n + bench.RANK_PAD_BYTES // 4
        slab = torch.full((8 * stride,), float("nan"), dtype=torch.float32, device=dev)
        bufs = [slab[r * stride: r * stride + n] for r in range(8)]
        for b, a in zip(bufs, x):
            b.copy_(torch.from_numpy(a))
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, FUSION[fusion])
    assert sched.num_steps == 3584
    bl.blink_allreduce(bufs, n, bl.BLINK_FP32, sched, stream())
    ox.run_steps(x, osch.make_steps(roots, parents, w, osch.ALLREDUCE, n, chunk))
    torch.cuda.synchronize()
    for r in range(8):
        got = bufs[r].cpu().numpy()
        rel = np.max(np.abs(got - x[0]) / np.maximum(np.abs(x[0]), np.finfo(np.float32).tiny))
        assert rel <= 1e-6
        assert np.array_equal(bits(got), bits(x[0])), f"rank {r}"
        if layout == "slab":
            assert bool(torch.isnan(slab[r * stride + n:(r + 1) * stride]).all()), f"gap after rank {r}"


@pytest.mark.parametrize("fusion", ["tree", "edge"])
def test_config2_broadcast_64MiB(dev, fusion):
    top = si.hybrid_cube_mesh()
    n, chunk = 1 << 24, 1 << 18
    trees = pack(top, 0)
    src = si.payload(2, 0, n, "normal", "fp32")
    bufs = [torch.from_numpy(src).to(dev)] + \
           [torch.full((n,), float("nan"), dtype=torch.float32, device=dev) for _ in range(7)]
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_BROADCAST, n, chunk, FUSION[fusion])
    assert sched.num_steps == 4 * 16 * 7
    bl.blink_broadcast(bufs, n, bl.BLINK_FP32, sched, stream())
    torch.cuda.synchronize()
    for b in bufs:
        assert b.cpu().numpy().tobytes() == src.tobytes()


@pytest.mark.parametrize("ranks", [(0, 1, 4), (2, 3, 5, 6, 7), (0, 1, 3, 4, 5, 7)])
@pytest.mark.parametrize("fusion", ["tree", "edge"])
def test_config3_fragmented_allocations_25_6M(dev, ranks, fusion):
    top = si.induced(si.hybrid_cube_mesh(doubled=True), ranks)
    n, chunk = 25_600_000, 1 << 18
    trees = pack(top, 0)
    roots, parents, w = trees.as_lists()
    assert trees.rate == {3: 2.0, 5: 2.0, 6: 4.0}[len(ranks)]
    x = [si.payload(3, r, n, "normal", "fp32", 1e-2) for r in range(top.k)]
    bufs = [torch.from_numpy(a).to(dev) for a in x]
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, FUSION[fusion])
    bl.blink_allreduce(bufs, n, bl.BLINK_FP32, sched, stream())
    want = ox.tree_order_allreduce(x, roots, parents, w)
    torch.cuda.synchronize()
    for b in bufs:
        assert np.array_equal(bits(b.cpu().numpy()), bits(want))


@pytest.mark.parametrize("dtype", ["fp32", "int32"])
def test_config4_sixteen_buckets_back_to_back(dev, dtype):
    """138M gradient elements in 16 log-uniform buckets, one call per bucket on
    one stream with no synchronisation in between."""
    top = si.hybrid_cube_mesh()
    sizes = si.bucket_sizes()
    chunk = 1 << 18
    trees = pack(top, 0)
    roots, parents, w = trees.as_lists()
    dist, scale = ("normal", 1e-3) if dtype == "fp32" else ("int", 1.0)
    code = bl.BLINK_FP32 if dtype == "fp32" else bl.BLINK_INT32
    hosts, devs, scheds = [], [], []
    for i, n in enumerate(sizes):
        x = [si.payload(100 + i, r, n, dist, dtype, scale) for r in range(8)]
        hosts.append(x)
        devs.append([torch.from_numpy(a).to(dev) for a in x])
        scheds.append(bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, bl.BLINK_FUSE_TREE))
    torch.cuda.synchronize()
    for n, bufs, sched in zip(sizes, devs, scheds):
        bl.blink_allreduce(bufs, n, code, sched, stream())
    torch.cuda.synchronize()
    for i, (n, x, bufs) in enumerate(zip(sizes, hosts, devs)):
        if dtype == "int32":
            want = ox.allreduce_int32_definition(x)
        else:
            want = ox.tree_order_allreduce(x, roots, parents, w)
        for r in (0, 7):
            assert np.array_equal(bits(bufs[r].cpu().numpy()), bits(want)), f"bucket {i} ({n} elements) rank {r}"
        for r in range(1, 7):
            assert torch.equal(bufs[r], bufs[0])


def test_config5_sixteen_rank_switch_1GiB_per_rank(dev):
    """16 one-hop trees, 256M fp32 per rank (16 GiB on the device), 4 MiB
    chunks.  Inputs are generated where they live; the oracle recomputes sampled
    slices (share boundaries, both ends, random interior) from the same
    counter-based recipe; all ranks must be identical everywhere."""
    top = si.complete_graph(16)
    n, chunk = 1 << 28, 1 << 20
    trees = pack(top, bl.BLINK_ROOT_ANY)
    roots, parents, w = trees.as_lists()
    bufs = [si.hash_payload_torch(9, r, n, "fp32", dev) for r in range(16)]
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, bl.BLINK_FUSE_TREE)
    assert sched.num_steps == 16 * 16 * 30
    bl.blink_allreduce(bufs, n, bl.BLINK_FP32, sched, stream())
    torch.cuda.synchronize()
    for r in range(1, 16):
        assert torch.equal(bufs[r], bufs[0]), f"rank {r} differs from rank 0"
    bounds = osch.split_by_weight(n, w)
    rng = np.random.default_rng(5)
    width = 4096
    starts = {0, n - width}
    for b in bounds[1:-1]:
        starts |= {b - width, b}           # both sides of every share boundary
    starts |= {int(s) for s in rng.integers(0, n - width, 24)}
    for a in sorted(starts):
        t = max(i for i in range(16) if bounds[i] <= a)
        if a + width > bounds[t + 1]:
            continue                        # keep a slice inside one share
        xs = [si.hash_payload(9, r, a, width, "fp32") for r in range(16)]
        want = ox.tree_order_allreduce(xs, [roots[t]], [parents[t]], [1.0])
        got = bufs[3][a:a + width].cpu().numpy()
        assert np.array_equal(bits(got), bits(want)), f"slice at {a} (tree {t})"


# ---- every kernel flavour at streaming size -------------------------------------------
# Large payloads run other kernel instantiations (32 columns per lane, cache
# policy by the schedule's read/write mix) than the small ones the element-by-
# element tests mostly use.  A whole-tree schedule streams from about
# 6144 tickets x 4096 elements = 25 M elements on, hence 2^25 per rank here.
@pytest.mark.parametrize("dtype", ["int32", "fp32"])
@pytest.mark.parametrize("coll", ["reduce", "broadcast", "allgather"])
def test_read_heavy_and_write_heavy_collectives_at_streaming_size(dev, dtype, coll):
    top = si.hybrid_cube_mesh()
    n, chunk, k = 1 << 25, 1 << 18, 8
    trees = pack(top, 0)
    roots, parents, w = trees.as_lists()
    code = bl.BLINK_INT32 if dtype == "int32" else bl.BLINK_FP32
    x = [si.payload(31, r, n, "int" if dtype == "int32" else "uniform", dtype) for r in range(k)]
    bufs = [torch.from_numpy(a).to(dev) for a in x]
    if coll == "reduce":
        sched = bl.blink_make_schedule(trees, bl.BLINK_OP_REDUCE, n, chunk, bl.BLINK_FUSE_TREE)
        bl.blink_reduce(bufs, n, code, bl.BLINK_SUM, sched, stream())
        want = ox.tree_order_allreduce(x, roots, parents, w)
        if dtype == "int32":
            assert np.array_equal(want, ox.allreduce_int32_definition(x))
        torch.cuda.synchronize()
        assert bufs[0].cpu().numpy().tobytes() == want.tobytes()      # every tree is rooted at 0
        for r in range(1, k):                                          # a whole-tree pass writes the root only
            assert bufs[r].cpu().numpy().tobytes() == x[r].tobytes()
    elif coll == "broadcast":
        sched = bl.blink_make_schedule(trees, bl.BLINK_OP_BROADCAST, n, chunk, bl.BLINK_FUSE_TREE)
        bl.blink_broadcast(bufs, n, code, sched, stream())
        want = ox.broadcast_definition(x, roots, w)
        torch.cuda.synchronize()
        for b in bufs:
            assert b.cpu().numpy().tobytes() == want.tobytes()
    else:
        sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLGATHER, n, chunk, bl.BLINK_FUSE_TREE)
        bl.blink_allgather(bufs, n, code, sched, stream())
        want = ox.allgather_definition(x)
        torch.cuda.synchronize()
        for b in bufs:
            assert b.cpu().numpy().tobytes() == want.tobytes()


@pytest.mark.parametrize("fusion", ["edge", "node"])
def test_int32_hand_over_kernels_at_streaming_size(dev, fusion):
    top = si.hybrid_cube_mesh()
    n, chunk = 1 << 24, 1 << 18
    trees = pack(top, 0)
    x = [si.payload(32, r, n, "int", "int32") for r in range(8)]
    bufs = [torch.from_numpy(a).to(dev) for a in x]
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, FUSION[fusion])
    sched.set_hand_over(True)     # per-node programs are served in one pass otherwise
    bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream())
    want = ox.allreduce_int32_definition(x)
    torch.cuda.synchronize()
    assert sched.handed_over == 1 and sched.status()[0] == bl.BLINK_OK
    for b in bufs:
        assert np.array_equal(b.cpu().numpy(), want)


@pytest.mark.parametrize("fusion", ["tree", "edge"])
def test_more_than_2_to_the_32_elements_per_rank(dev, fusion):
    """Offsets beyond 32 bits: 2 ranks of 2^32 + 12,291 int32 each (34 GiB on the
    device), ragged end included.  Inputs are generated where they live; the
    oracle recomputes sampled slices from the same counter-based recipe."""
    n, chunk, k = (1 << 32) + 12_291, 1 << 20, 2
    top = si.complete_graph(2)
    trees = pack(top, 1)
    bufs = [si.hash_payload_torch(13, r, n, "int32", dev) for r in range(k)]
    sched = bl.blink_make_schedule(trees, bl.BLINK_OP_ALLREDUCE, n, chunk, FUSION[fusion])
    assert sched.num_steps == 2 * ((n + chunk - 1) // chunk)
    bl.blink_allreduce(bufs, n, bl.BLINK_INT32, sched, stream())
    torch.cuda.synchronize()
    assert torch.equal(bufs[0], bufs[1])
    width = 8192
    starts = [0, (1 << 31) - width // 2, (1 << 32) - width, (1 << 32) - width // 2, 1 << 32, n - width, n - 5]
    starts += [int(s) for s in np.random.default_rng(6).integers(0, n - width, 16)]
    for a in starts:
        m = min(width, n - a)
        xs = [si.hash_payload(13, r, a, m, "int32") for r in range(k)]
        want = ox.allreduce_int32_definition(xs)
        got = bufs[0][a:a + m].cpu().numpy()
        assert np.array_equal(got, want), f"slice at {a}"
