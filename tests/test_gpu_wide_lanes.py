"""fp32 plans whose launches choose their lanes and accesses by the layout of
the rank buffers, bit for bit against the oracle.

Few ranks: four columns per lane in the block-tiled, latency-optimal and XOR
kernels, with blocks on both sides of the length from which they are taken,
every residue of a lane's columns at a block's ends, batches with and without
gaps, rows on and off the 128-byte lines.  More ranks: rows off the lines,
which take cached accesses, also where they are nontemporal on them
(AR_FUSED_NT unset, 0 and 1).  Shifted max on batches of short blocks: rank
slots, on values and on signed zeros, whose result shows every combination's
operand order.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2004_09362_amd import ar
from test_gpu_line_grids import check
from test_gpu_parity import DEV, bits, note

pytestmark = pytest.mark.gpu


def L(P):
    return (P - 1).bit_length()


@pytest.mark.parametrize("nt", [None, "0", "1"])
@pytest.mark.parametrize("P", [2, 3, 4, 5, 6, 7, 8, 9])
def test_few_ranks(P, nt, monkeypatch):
    if nt is not None:
        monkeypatch.setenv("AR_FUSED_NT", nt)
    for k in range(L(P), 2 * L(P) + 1):
        for n, B, gap, lead in ((P * 1024 - 1, 1, 0, 0), (P * 1024 + 1, 1, 0, 0), (P * 1030 + P - 1, 1, 0, 3),
                                (P * 2051, 3, 0, 1), (P * 1027 + 2, 2, 5, 2), (P * 5000 + 3, 1, 0, 32), (7, 1, 0, 1)):
            check(P, n, k, B=B, gap=gap, lead=lead, op=("sum", "max")[(n + k) % 2])
    check(P, P * 1100 + 1, 2 * (P - 1), lead=5, schedule="ring")
    if P & (P - 1) == 0:
        for k in range(L(P), 2 * L(P) + 1):
            for n, lead in ((1, 0), (4097, 0), (4098, 7), (P * 1024 + 3, 1)):
                check(P, n, k, lead=lead, group="xor")
            check(P, 1023, k, B=3, lead=1, group="xor")
            check(P, 1023, k, B=3, gap=2, lead=1, group="xor")


@pytest.mark.parametrize("split", ["2", "8"])
@pytest.mark.parametrize("P", [2, 4, 7])
def test_few_ranks_split(P, split, monkeypatch):
    monkeypatch.setenv("AR_FUSED_SPLIT", "1")
    for lead in (0, 3):
        check(P, P * 1024 * int(split) + 5, 2 * L(P), lead=lead)


@pytest.mark.parametrize("nt", [None, "0", "1"])
@pytest.mark.parametrize("P", [13, 24, 37, 48, 100, 127])
def test_more_ranks_off_the_lines(P, nt, monkeypatch):
    if nt is not None:
        monkeypatch.setenv("AR_FUSED_NT", nt)
    for k in sorted({L(P), L(P) + 1, 2 * L(P) - 1, 2 * L(P)}):
        for n, B, gap, lead in ((P * 150 + 3, 1, 0, 1), (106, 41, 7, 0), (106, 41, 0, 5)):
            check(P, n, k, B=B, gap=gap, lead=lead, op=("sum", "max")[(n + k) % 2])
    check(P, P * 100 + 7, 2 * (P - 1), B=2, gap=9, lead=1, schedule="ring")


@pytest.mark.parametrize("P", [3, 5, 8, 16, 23, 24, 49, 64, 127])
def test_shifted_max_on_short_blocks(P):
    for k in range(L(P) + 1, 2 * L(P)):
        for n, B, gap in ((3, 70, 0), (106, 33, 0), (P * 18 + 5, 7, 3)):
            check(P, n, k, B=B, gap=gap, op="max")
        n, B = 5 * P + 3, 9
        rng = np.random.default_rng(P * 100 + k)
        x = np.where(rng.random((P, B, n)) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
        X = torch.from_numpy(x).to(DEV)
        plan = ar.Plan(P, n, "float32", "max", k)
        note("shifted max of signed zeros P=%d k=%d" % (P, k))
        plan.batched([X[i] for i in range(P)], B, n)
        torch.cuda.synchronize()
        assert np.array_equal(bits(X.cpu().numpy()), bits(oracle.allreduce_batched(x, k, "max"))), (P, k)
        plan.close()
