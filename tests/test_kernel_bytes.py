"""What a call moves, counted from the trees: by the stages of the program, and by the kernel
that serves it, which carries a tile through all of a per-node or small per-edge program
at once.  No GPU."""
import pytest

import paper_1910_04940_amd as bl
import synth_inputs as si

MIB = 1 << 20


def _per_element(k, parent, op, fusion):
    """Reads and writes of one pass along a tree, partial sums included."""
    inner = len({p for p in parent if p >= 0})
    if op == bl.BLINK_OP_BROADCAST:
        return 1 + (k - 1)
    # every addition forms a sum; the root's last one is the result
    on_the_way = {bl.BLINK_FUSE_EDGE: k - 2, bl.BLINK_FUSE_NODE: inner - 1, bl.BLINK_FUSE_TREE: 0}[fusion]
    return k + on_the_way + (k if op == bl.BLINK_OP_ALLREDUCE else 1)


@pytest.mark.parametrize("op", [bl.BLINK_OP_ALLREDUCE, bl.BLINK_OP_BROADCAST, bl.BLINK_OP_REDUCE])
@pytest.mark.parametrize("fusion", [bl.BLINK_FUSE_EDGE, bl.BLINK_FUSE_NODE, bl.BLINK_FUSE_TREE])
@pytest.mark.parametrize("top", [si.hybrid_cube_mesh(), si.star(6, 2), si.chain(5), si.complete_graph(4)], ids=lambda t: t.name)
@pytest.mark.parametrize("n", [5, 100_003, 64 * MIB])
def test_bytes_of_the_kernel_that_serves(top, fusion, op, n):
    k = top.k
    trees = bl.blink_pack_trees(k, top.src, top.dst, top.cap, 0)
    _, parents, _ = trees.as_lists()
    sched = bl.blink_make_schedule(trees, op, n, MIB, fusion)
    b = sched.bounds()
    one_pass = 4 * sum((b[t + 1] - b[t]) * _per_element(k, p, op, fusion) for t, p in enumerate(parents))
    depends = any(int(s["n_dep"]) for s in sched.stages())
    handed_over = fusion == bl.BLINK_FUSE_EDGE and depends and 4 * k * n > 256 * MIB
    assert sched.kernel_bytes == (sched.traffic_bytes if handed_over else one_pass)
    if fusion == bl.BLINK_FUSE_TREE:
        assert sched.kernel_bytes == sched.traffic_bytes
    else:
        assert sched.kernel_bytes <= sched.traffic_bytes
