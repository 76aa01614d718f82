"""The device block that all calls of blink_allreduce_noalloc on a GPU share: a call finds
in it the tables of the kernel that serves it, whichever schedule and whichever of the two
kernels used the block before, and a schedule's status is that of its own calls."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import execute as ox

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1910_04940_amd as bl  # noqa: E402


def _stream():
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    return torch.cuda.current_stream().cuda_stream


def _chain(k, order):
    parent = [-1] * k
    for a, b in zip(order, order[1:]):
        parent[b] = a
    return order[0], parent


def _forest(k, n_trees):
    chains = [_chain(k, [(t + i) % k for i in range(k)]) for t in range(n_trees)]
    return bl.blink_trees_from_arrays(k, [r for r, _ in chains], [p for _, p in chains],
                                      [1.0 + t for t in range(n_trees)])


def _bufs(x):
    return [torch.from_numpy(a).to("cuda") for a in x]


# up to four trees travel with a launch, six lie in the block
@pytest.mark.parametrize("n_trees", [2, 6])
@pytest.mark.parametrize("fusion", [bl.BLINK_FUSE_EDGE, bl.BLINK_FUSE_NODE])
def test_the_block_holds_the_tables_of_the_kernel_that_runs(fusion, n_trees):
    """One schedule's calls on the block change from the one-pass kernel to waiting stages,
    with a reset before the change, and back."""
    stream = _stream()
    k, n = 5, 70_003
    x = [si.hash_payload(43, r, 0, n, "int32") for r in range(k)]
    want = ox.allreduce_int32_definition(x)
    sched = bl.blink_make_schedule(_forest(k, n_trees), bl.BLINK_OP_ALLREDUCE, n, 4_096, fusion)

    def noalloc():
        bufs = _bufs(x)
        bl.blink_allreduce_noalloc(bufs, n, bl.BLINK_INT32, sched, stream)
        torch.cuda.synchronize()
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs)
        assert sched.status()[0] == bl.BLINK_OK

    bl.blink_allreduce(_bufs(x), n, bl.BLINK_INT32, sched, stream)
    noalloc()
    sched.reset()
    sched.test_skip_call()        # from here on its stages wait; calls on the block start from cleared counters
    noalloc()
    noalloc()
    sched.reset()
    noalloc()
    sched.test_skip_call()
    assert sched.status()[0] == bl.BLINK_OK
    noalloc()


def test_a_record_on_the_block_is_not_taken_for_another_schedules():
    """A wait given up on the block leaves a record there.  A schedule whose calls then use the
    block without waits reports on its own, also after a reset."""
    stream = _stream()
    # one tile per stage, fourteen stages one after the other: the last waits for 13 tiles
    k, n = 8, 1 << 16
    slow = bl.blink_make_schedule(_forest(k, 1), bl.BLINK_OP_ALLREDUCE, n, n, bl.BLINK_FUSE_EDGE)
    slow.set_launch(0, 1 << 16)
    big = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(k)]
    bl.blink_allreduce(big, n, bl.BLINK_INT32, slow, stream)
    slow.test_skip_call()
    slow.set_wait_limit(1)
    bl.blink_allreduce_noalloc(big, n, bl.BLINK_INT32, slow, stream)
    assert slow.status()[0] == bl.BLINK_ESTUCK

    m = 4_099
    x = [si.hash_payload(47, r, 0, m, "int32") for r in range(k)]
    quick = bl.blink_make_schedule(_forest(k, 1), bl.BLINK_OP_ALLREDUCE, m, m, bl.BLINK_FUSE_TREE)
    bufs = _bufs(x)
    bl.blink_allreduce_noalloc(bufs, m, bl.BLINK_INT32, quick, stream)
    assert quick.status()[0] == bl.BLINK_OK
    quick.reset()
    assert quick.status()[0] == bl.BLINK_OK
    assert all(np.array_equal(b.cpu().numpy(), ox.allreduce_int32_definition(x)) for b in bufs)

    slow.reset()                  # its own record goes with a reset, on the block too
    bl.blink_allreduce(big, n, bl.BLINK_INT32, slow, stream)
    slow.test_skip_call()
    bl.blink_allreduce_noalloc(big, n, bl.BLINK_INT32, slow, stream)
    assert slow.status()[0] == bl.BLINK_ESTUCK
    slow.reset()
    assert slow.status()[0] == bl.BLINK_OK


@pytest.mark.parametrize("before,after", [(0, 256), (65_536, 1_024), (256, 0), (256, 256)])
def test_a_call_can_be_recorded_after_a_new_tile_size_or_a_reset(before, after):
    """Six shares of different lengths, whose tables lie in the block for every tile size.  The
    recorded call is replayed with the program's own work in between."""
    stream = _stream()
    k, n = 5, 100_003
    x = [si.hash_payload(53, r, 0, n, "int32") for r in range(k)]
    want = ox.allreduce_int32_definition(x)
    sched = bl.blink_make_schedule(_forest(k, 6), bl.BLINK_OP_ALLREDUCE, n, 1 << 20, bl.BLINK_FUSE_TREE)
    sched.set_launch(0, before)
    src = _bufs(x)
    bufs = [b.clone() for b in src]
    bl.blink_allreduce_noalloc(bufs, n, bl.BLINK_INT32, sched, stream)
    torch.cuda.synchronize()
    if before == after:
        sched.reset()
    sched.set_launch(0, after)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bl.blink_allreduce_noalloc(bufs, n, bl.BLINK_INT32, sched, torch.cuda.current_stream().cuda_stream)
    for replay in range(3):
        for b, s0 in zip(bufs, src):
            b.copy_(s0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(b.cpu().numpy(), want) for b in bufs), replay
