"""Split calls whose rank buffers share no alignment, on the GPU, bit for bit
against the CPU oracle.

The broadcast of a split plan copies destination by destination in 4 KB
chunks laid on the 128-byte lines of each destination, whatever the rank
buffers' alignment, and element by element at the two ends of a buffer and
beside the gaps between instances.  These cases put the ends of the column
space on both sides of a chunk's and a line's edge, rows on every residue of
a line, and gaps of one element and of many; the elements around the rows and
in the gaps must stay as they were.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2004_09362_amd import ar
from test_gpu_parity import DEV, bits, note

pytestmark = pytest.mark.gpu


def packed_rows(x, lead):
    """x [P, span] on the GPU, each row right behind the one before, the
    first `lead` elements behind a 256-byte boundary; the rows and the whole
    allocation, whose other elements are 77."""
    P, span = x.shape
    dt = torch.int32 if x.dtype == np.int32 else torch.float32
    mem = torch.full((lead + P * span + 64,), 77, dtype=dt, device=DEV)
    rows = mem[lead:lead + P * span].view(P, span)
    rows.copy_(torch.from_numpy(x))
    return mem, rows


def check(P, n, k, B=1, gap=0, lead=0, dtype="float32", op="sum", group="cyclic", schedule="butterfly"):
    rng = np.random.default_rng(P * 7919 + n + 31 * gap + lead)
    stride = n + gap
    span = (B - 1) * stride + n
    x = (rng.integers(-2**31, 2**31, size=(P, span)).astype(np.int32) if dtype == "int32"
         else rng.normal(size=(P, span)).astype(np.float32))
    mem, rows = packed_rows(x, lead)
    plan = ar.Plan(P, n, dtype, op, k, group=group, schedule=schedule)
    note("line grids P=%d n=%d k=%d B=%d gap=%d lead=%d %s %s %s/%s launches %d"
         % (P, n, k, B, gap, lead, dtype, op, group, schedule, plan.stats().fused_launches))
    plan.batched([rows[i] for i in range(P)], B, stride)
    torch.cuda.synchronize()
    got = rows.cpu().numpy()
    inst = np.stack([x[:, j * stride:j * stride + n] for j in range(B)], axis=1)
    want = oracle.allreduce_batched(np.ascontiguousarray(inst), k, op, group=group, schedule=schedule)
    for j in range(B):
        assert np.array_equal(bits(got[:, j * stride:j * stride + n]), bits(want[:, j])), j
        assert np.array_equal(bits(got[:, j * stride + n:(j + 1) * stride]),
                              bits(x[:, j * stride + n:(j + 1) * stride])), j
    m = mem.cpu().numpy()
    assert (m[:lead] == 77).all() and (m[lead + P * span:] == 77).all()
    plan.close()


@pytest.mark.parametrize("order", ["2", "3"])
@pytest.mark.parametrize("P,k,group,schedule", [(2, 2, "cyclic", "butterfly"), (13, 8, "cyclic", "butterfly"),
                                                (37, 12, "cyclic", "butterfly"), (32, 10, "xor", "butterfly"),
                                                (24, 46, "cyclic", "ring"), (127, 14, "cyclic", "butterfly")])
def test_split_calls_on_rows_off_the_lines(P, k, group, schedule, order, monkeypatch):
    monkeypatch.setenv("AR_FUSED_SPLIT", "1")
    monkeypatch.setenv("AR_BCAST_STREAM", order)
    for n, lead in ((1, 3), (31, 0), (993, 31), (1023, 1), (1024, 0), (1025, 5), (4097, 2), (70001, 17)):
        check(P, n, k, lead=lead, group=group, schedule=schedule)


@pytest.mark.parametrize("P,n,B,gap", [(33, 106, 50, 7), (37, 2304, 9, 1), (64, 5, 301, 3), (64, 1, 77, 1),
                                       (127, 1000, 7, 24), (100, 4100, 3, 1000)])
def test_split_batches_with_gaps(P, n, B, gap):
    L = (P - 1).bit_length()
    for lead in (0, 1, 16):
        check(P, n, 2 * L, B=B, gap=gap, lead=lead)
    check(P, n, 2 * L, B=B, gap=gap, lead=3, dtype="int32", op="max")
