"""What is measured: one Allreduce call on rank buffers that are in device memory, as programs make it.

Every case is one ``Plan`` call of the Python binding on the current stream, on the path that a plan takes by
default.  The rank buffers are P rows of one tensor; ``pitch`` is the distance between two rows in elements, so a
row either starts on a 256-byte boundary, as a buffer of its own does, or right behind the row before it, on any
element.  A call reduces in place, so the outputs are the buffers; a second pass on the same state reduces the
first one's results.

The fields of a case: ranks ``P``, elements ``n`` of an instance, instances ``batch`` and the distance ``stride``
between two of them, ``dtype``, ``op``, step count ``k`` (a number or "auto"), ``group``, ``schedule`` and
``pitch``.
"""
import math

import torch

from paper_2004_09362_amd import ar

DTYPES = {"float32": torch.float32, "int32": torch.int32}


def _case(name, P, n, *, k, batch=1, stride=None, dtype="float32", op="sum", group="cyclic", schedule="butterfly",
          pitch=None):
    stride = n if stride is None else stride
    c = dict(name=name, P=P, n=n, batch=batch, stride=stride, dtype=dtype, op=op, k=k, group=group,
             schedule=schedule, pitch=-(-batch * stride // 64) * 64 if pitch is None else pitch)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # three ranks and a 4 KB integer vector: the smallest call, all latency
        _case("tiny_p3", 3, 1024, k=4, dtype="int32"),
        # one message of the average size of a production Allreduce, 425 bytes, at the paper's 127 ranks, with the
        # step count left to the library
        _case("message_p127", 127, 106, k="auto"),
        # one 1 MB vector on eight ranks, the ranks of one node, as a power of two: Recursive Halving
        _case("node_p8_1mb", 8, 262144, k=6, group="xor"),
        # the 425-byte message many at a time, with few ranks, latency-optimal
        _case("batch_p12", 12, 106, batch=65536, k=4),
        # and at 127 ranks, where a column's sums no longer fit a lane's registers
        _case("batch_p127", 127, 106, batch=65536, k=7),
        # 9 KB messages many at a time, at a step count between the two ends
        _case("medium_p127", 127, 2304, batch=8192, k=11),
        # the largest element of integer messages that lie in records, with gaps between them
        _case("records_p16_max", 16, 1000, batch=4096, stride=1024, k=6, dtype="int32", op="max"),
        # a gradient of an odd length on a prime number of ranks, the rows one behind the other
        _case("ragged_p13", 13, 3000017, k=8, pitch=3000017),
        # a 64 MB gradient on 24 ranks, bandwidth-optimal
        _case("gradient_p24", 24, 1 << 24, k=10),
        # and on 32 ranks over the XOR group, at a step count between its two ends
        _case("gradient_p32_xor", 32, 1 << 24, k=7, group="xor"),
        # the largest of 37 vectors of 16 MB, at a step count between the two ends
        _case("sweep_p37_max", 37, 1 << 22, k=8, op="max"),
        # the largest vectors that fit the card: 256 MB on 127 ranks, bandwidth-optimal
        _case("large_p127", 127, 1 << 26, k=14),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    group = "xor" if rng.random() < 0.25 else "cyclic"
    P = 1 << rng.randint(1, 7) if group == "xor" else _log_uniform(rng, 2, 128)
    L = (P - 1).bit_length()
    schedule = "ring" if group == "cyclic" and rng.random() < 0.15 else "butterfly"
    if schedule == "ring":
        k = 2 * (P - 1)
    else:  # both ends, the library's choice, or any in between
        k = rng.choice([L, 2 * L, "auto", rng.randint(L, 2 * L)])
    row = _log_uniform(rng, 64, min(1 << 26, (1 << 31) // P))  # elements a rank holds in all
    if rng.random() < 0.4:
        n = min(_log_uniform(rng, 32, 4096), row)
        batch = max(1, row // n)
        stride = n if rng.random() < 0.5 else n + rng.randint(1, 64)
    else:
        n, batch, stride = row, 1, row
    end = batch * stride
    pitch = end if rng.random() < 0.4 else -(-end // 64) * 64
    return _case(None, P, n, k=k, batch=batch, stride=stride, dtype=rng.choice(["float32", "float32", "int32"]),
                 op=rng.choice(["sum", "sum", "max"]), group=group, schedule=schedule, pitch=pitch)


def _rows(case, seed):
    """The rank buffers [P, pitch]: gradients and messages are small normal numbers, integers any of 21 bits."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + case["P"])
    shape = (case["P"], case["pitch"])
    X = torch.empty(shape, dtype=DTYPES[case["dtype"]], device="cuda")
    if case["dtype"] == "int32":
        return X.random_(-1000000, 1000000, generator=g)
    return X.normal_(0.0, 0.01, generator=g)


def prepare(case, seed):
    X = _rows(case, seed)
    plan = ar.Plan(case["P"], case["n"], case["dtype"], case["op"], case["k"], group=case["group"],
                   schedule=case["schedule"], batch=case["batch"])
    return {"X": X, "bufs": list(X.unbind(0)), "plan": plan, "batch": case["batch"], "stride": case["stride"]}


def run(state):
    if state["batch"] == 1:
        state["plan"](state["bufs"])
    else:
        state["plan"].batched(state["bufs"], state["batch"], state["stride"])
    return state["X"]


def work(case):
    elems = case["P"] * case["n"] * case["batch"]
    return {"bytes": 2 * 4 * elems, "flops": (case["P"] - 1) * case["n"] * case["batch"]}


def tolerance(case):
    if case["dtype"] == "int32" or case["op"] == "max":
        return "exact"
    return {"rel": 1e-6, "max": 1e-5}


def exact(case, seed):
    X = _rows(case, seed)
    P, n, batch, stride = case["P"], case["n"], case["batch"], case["stride"]
    end = batch * stride
    acc = X[0].to(torch.int64 if case["dtype"] == "int32" else torch.float64)
    for x in range(1, P):
        if case["op"] == "sum":
            acc += X[x]
        else:
            acc = torch.maximum(acc, X[x].to(acc.dtype))
    if case["dtype"] == "int32":  # sums wrap round
        acc = ((acc + (1 << 31)) % (1 << 32) - (1 << 31)).to(torch.int32)
    if stride == n and case["pitch"] == end:
        del X
        return acc.expand(P, case["pitch"])
    out = X.to(acc.dtype)  # the gaps between instances and behind the last one stay as they were
    del X
    out[:, :end].view(P, batch, stride)[:, :, :n] = acc[:end].view(batch, stride)[:, :n]
    return out
