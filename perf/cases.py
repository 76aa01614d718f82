"""The collectives whose speed is looked after, each through the public binding.

One case is one kind of call that a data-parallel training job makes, repeated on
buffers that stay in HBM: `prepare` packs the trees, makes the schedule and fills
the rank buffers, `run` enqueues the collective on the current stream, in place,
as the job would after every backward pass.  `exact` is the same collective in 64
bits (int32: modulo 2^32) with plain torch.

Results are compared bit for bit: the trees fix the order in which a sum is
formed, everything else moves or selects values.
"""
import math

import torch

import paper_1910_04940_amd as bl
import synth_inputs as si

MIB = 1 << 20

OPS = {"broadcast": bl.BLINK_OP_BROADCAST, "allreduce": bl.BLINK_OP_ALLREDUCE, "reduce": bl.BLINK_OP_REDUCE,
       "allgather": bl.BLINK_OP_ALLGATHER, "gather": bl.BLINK_OP_GATHER}
FUSIONS = {"edge": bl.BLINK_FUSE_EDGE, "node": bl.BLINK_FUSE_NODE, "tree": bl.BLINK_FUSE_TREE}
REDOPS = {"sum": bl.BLINK_SUM, "prod": bl.BLINK_PROD, "min": bl.BLINK_MIN, "max": bl.BLINK_MAX}
RANKS = {"cube": 8, "k4": 4, "k16": 16, "servers": 16, "frag3": 3, "frag5": 5, "frag6": 6}
FRAGMENTS = {"frag3": (0, 1, 4), "frag5": (2, 3, 5, 6, 7), "frag6": (0, 1, 3, 4, 5, 7)}


def _case(name, op, top, n, fusion="tree", chunk=MIB // 4, dtype="fp32", redop="sum", buckets=False):
    return {"name": name, "op": op, "top": top, "n": n, "fusion": fusion, "chunk": chunk, "dtype": dtype,
            "redop": redop, "buckets": buckets}


def listed():
    return [
        # the smallest gradient bucket of a model (64 KiB and a ragged end): all latency
        _case("small bucket", "allreduce", "cube", 16_411),
        # a 4 MiB bucket on a fully connected group of four
        _case("4 ranks 4 MiB", "allreduce", "k4", MIB, chunk=65_536),
        # sending a model's weights out at the start, or a pipeline stage's activations
        _case("broadcast 64 MiB", "broadcast", "cube", 16 * MIB),
        # a fragmented allocation (6 GPUs of a server), gradients of a 25.6 M parameter model
        _case("fragment of 6", "allreduce", "frag6", 25_600_000),
        # the same model on 5 GPUs, an odd count: the largest value per element (gradient clipping, overflow flags)
        _case("max over 5 int32", "allreduce", "frag5", 25_600_003, dtype="int32", redop="max"),
        # one large fused gradient buffer: the headline size of the benchmark
        _case("8 ranks 256 MiB", "allreduce", "cube", 64 * MIB),
        # a whole backward pass: 138 M gradients in sixteen buckets of 64 KiB to 120 MiB, one call each
        _case("16 buckets", "allreduce", "cube", 138_000_000, buckets=True),
        # sixteen GPUs behind a switch, one-hop trees, the largest payload the benchmark has
        _case("16 ranks 1 GiB", "allreduce", "k16", 256 * MIB, chunk=MIB),
        # two servers of eight, the three-phase protocol
        _case("two servers", "allreduce", "servers", 16 * MIB),
        # the paper's own program, one transfer per tree edge and chunk, as tuned by the chunk size search
        _case("per edge 64 MiB", "allreduce", "cube", 16 * MIB, fusion="edge", dtype="int32"),
        # the program one GPU of a real server would run, fan-ins and fan-outs, on a ragged mid-size bucket
        _case("per node 20 MB", "allreduce", "cube", 5_000_011, fusion="node"),
        # collecting sharded parameters before a forward pass
        _case("allgather 64 MiB", "allgather", "cube", 16 * MIB),
    ]


def draw(rng):
    op = rng.choice(["allreduce"] * 6 + ["broadcast", "reduce", "allgather", "gather"])
    # reduce and gather are read at their one root; what else a reduce leaves in the
    # other ranks' buffers is only fixed where the tree is fused
    top = rng.choice(["cube", "cube", "k4", "frag3", "frag5", "frag6"] + (["k16", "servers"] if op == "allreduce" else []))
    fusion = "tree" if op == "reduce" else rng.choice(["tree", "tree", "tree", "edge", "node"])
    k = RANKS[top]
    n = int(math.exp(rng.uniform(math.log(4096), math.log(2 ** 29 // k))))   # up to 2 GiB over all ranks
    if op in ("allgather", "gather"):
        n -= n % k
    dtype = rng.choice(["fp32", "fp32", "int32"])
    redop = rng.choice(["sum", "sum", "sum", "min", "max"]) if op in ("allreduce", "reduce") else "sum"
    chunk = rng.choice([16_384, 65_536, 262_144, 262_144, 1_048_576])
    return {"op": op, "top": top, "n": n, "fusion": fusion, "chunk": chunk, "dtype": dtype, "redop": redop,
            "buckets": False}


def _trees(top):
    if top in FRAGMENTS:
        t = si.induced(si.hybrid_cube_mesh(True), FRAGMENTS[top])
    else:
        t = {"cube": si.hybrid_cube_mesh, "servers": si.hybrid_cube_mesh, "k4": lambda: si.complete_graph(4),
             "k16": lambda: si.complete_graph(16)}[top]()
    return bl.blink_pack_trees(t.k, t.src, t.dst, t.cap, bl.BLINK_ROOT_ANY if top == "k16" else 0)


def _schedule(case, trees, n):
    if case["top"] == "servers":
        return bl.blink_make_schedule_servers([trees, trees], [range(8), range(8, 16)], n, case["chunk"],
                                              FUSIONS[case["fusion"]])
    return bl.blink_make_schedule(trees, OPS[case["op"]], n, case["chunk"], FUSIONS[case["fusion"]])


def _sizes(case):
    return si.bucket_sizes(case["n"]) if case["buckets"] else [case["n"]]


def _input(case, seed, bucket, rank, n):
    """Rank `rank`'s buffer before the call: gradients are small and centred, integers span their whole range."""
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1009 + bucket) * 64 + rank)
    if case["dtype"] == "int32":
        return torch.randint(-2 ** 31, 2 ** 31, (n,), dtype=torch.int32, device="cuda", generator=g)
    return torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, 1e-2, generator=g)


def prepare(case, seed):
    trees = _trees(case["top"])
    k = RANKS[case["top"]]
    calls = []
    for b, n in enumerate(_sizes(case)):
        calls.append((_schedule(case, trees, n), n, [_input(case, seed, b, r, n) for r in range(k)]))
    return {"op": case["op"], "redop": REDOPS[case["redop"]],
            "dtype": bl.BLINK_FP32 if case["dtype"] == "fp32" else bl.BLINK_INT32, "calls": calls,
            "stream": torch.cuda.current_stream().cuda_stream}


def run(state):
    op, redop, dtype, stream = state["op"], state["redop"], state["dtype"], state["stream"]
    out = []
    for schedule, n, bufs in state["calls"]:
        if op == "allreduce":
            if redop == bl.BLINK_SUM:
                bl.blink_allreduce(bufs, n, dtype, schedule, stream)
            else:
                bl.blink_allreduce_op(bufs, n, dtype, redop, schedule, stream)
        elif op == "broadcast":
            bl.blink_broadcast(bufs, n, dtype, schedule, stream)
        elif op == "allgather":
            bl.blink_allgather(bufs, n, dtype, schedule, stream)
        elif op == "reduce":
            bl.blink_reduce(bufs, n, dtype, redop, schedule, stream)
        else:
            bl.blink_gather(bufs, n, dtype, schedule, stream)
        # the ranks that hold the result: the root alone, or all of them (of a
        # whole set of buckets two ranks' worth, the first and the last)
        out.append(bufs[:1] if op in ("reduce", "gather") else bufs if len(state["calls"]) == 1 else [bufs[0], bufs[-1]])
    return out


def work(case):
    k, n = RANKS[case["top"]], case["n"]
    op = case["op"]
    values = {"allreduce": 2 * k * n,            # every rank's buffer read and written
              "broadcast": n + (k - 1) * n,      # the root's read, the others' written
              "reduce": k * n + n,               # every rank's read, the root's written
              "allgather": n + (k - 1) * n,      # every piece read once and written to the other ranks
              "gather": 2 * (n - n // k)}[op]    # every piece but the root's own read and written once
    return {"bytes": 4 * values, "flops": (k - 1) * n if op in ("allreduce", "reduce") else 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    k, op, redop = RANKS[case["top"]], case["op"], case["redop"]
    out = []
    for b, n in enumerate(_sizes(case)):
        wide = torch.int64 if case["dtype"] == "int32" else torch.float64
        if op == "broadcast":
            result = _input(case, seed, b, 0, n).to(wide)
        elif op in ("allgather", "gather"):
            m = n // k
            result = torch.cat([_input(case, seed, b, r, n)[r * m:(r + 1) * m] for r in range(k)]).to(wide)
        else:
            result = _input(case, seed, b, 0, n).to(wide)
            for r in range(1, k):
                x = _input(case, seed, b, r, n).to(wide)
                if redop == "sum":
                    result += x
                elif redop == "prod":
                    result *= x
                else:
                    result = torch.minimum(result, x) if redop == "min" else torch.maximum(result, x)
                if wide == torch.int64 and redop in ("sum", "prod"):   # modulo 2^32, as a signed number
                    result = ((result + 2 ** 31) & (2 ** 32 - 1)) - 2 ** 31
        copies = 1 if op in ("reduce", "gather") else 2 if case["buckets"] else k
        out.append([result.to(torch.int32) if wide == torch.int64 else result] * copies)
    return out
