"""int32 plans on the GPU: their fused kernel combines a column's P values in
any order, several columns per lane, and must give the oracle's bits for
every schedule.

P on both sides of every change of the kernel's width and unrolling, n on
every residue of a lane's elements, with and without gaps (below and above
the length from which a lane may hold part of a group), rows on and off the
128-byte lines, cached and nontemporal, in one launch and split.  Values reach
the ends of the type, so sums wrap round.
"""
import pytest
import torch

from paper_2004_09362_amd import ar
from test_gpu_line_grids import check
from test_gpu_parity import DEV, note

pytestmark = pytest.mark.gpu


def L(P):
    return (P - 1).bit_length()


@pytest.mark.parametrize("nt", ["0", "1"])
@pytest.mark.parametrize("split", ["0", "1"])
@pytest.mark.parametrize("P", [2, 3, 7, 16, 17, 18, 33, 34, 49, 50, 65, 66, 81, 82, 97, 98, 113, 114, 127, 128])
def test_any_int32_plan(P, split, nt, monkeypatch):
    monkeypatch.setenv("AR_FUSED_SPLIT", split)
    monkeypatch.setenv("AR_FUSED_NT", nt)
    for i, (n, B, gap, lead) in enumerate(((1, 1, 0, 0), (255, 1, 0, 3), (1026, 1, 0, 0), (4099, 1, 0, 1),
                                           (106, 9, 22, 0), (63, 7, 1, 5), (1000, 3, 24, 0), (4098, 2, 31, 2))):
        k = (L(P), 2 * L(P), (3 * L(P) + 1) // 2)[i % 3]
        check(P, n, k, B=B, gap=gap, lead=lead, dtype="int32", op=("sum", "max")[i % 2])
    check(P, 300, 2 * (P - 1), B=2, gap=4, dtype="int32", schedule="ring")
    if P & (P - 1) == 0:
        check(P, 777, 2 * L(P) - 1, dtype="int32", op="max", group="xor")


def launches(P, n, B, pitch, k):
    """Launches of one call on rows `pitch` elements apart, B instances back to back."""
    X = torch.zeros((P, pitch), dtype=torch.int32, device=DEV)
    plan = ar.Plan(P, n, "int32", "max", k)
    ms = plan.timed(list(X.unbind(0)), B, n)
    plan.close()
    return len(ms)


@pytest.mark.parametrize("P,k", [(16, 4), (17, 5), (24, 10), (100, 14)])
def test_split_by_size_and_one_launch_agree(P, k):
    """Calls just below and at the size from which int32 plans of 17 ranks and
    more split, rows off the lines (144 MiB over all ranks, 128 MiB from 33
    ranks): one instance, and a batch of short ones, whose size is that of all
    its instances."""
    least = ((144 if P < 33 else 128) << 20) // 4 // P
    for n, B in ((least - 1, 1), (least, 1), (106, least // 106), (106, least // 106 + 1)):
        want = 2 if P >= 17 and n * B >= least else 1
        note("int32 split P=%d n=%d B=%d k=%d" % (P, n, B, k))
        assert launches(P, n, B, -(-n * B // 32) * 32 + 1, k) == want, (P, n, B)
        if B > 1 or n == least:
            check(P, n, k, B=B, lead=1, dtype="int32", op="max")


@pytest.mark.parametrize("P,mib", [(24, 144), (33, 128), (127, 128)])
def test_split_size_on_the_lines(P, mib):
    least = (mib << 20) // 4 // P
    for n, B in ((least - 1, 1), (least, 1), (106, least // 106), (106, least // 106 + 1)):
        assert launches(P, n, B, -(-n * B // 32) * 32, L(P)) == (2 if n * B >= least else 1), (P, n, B)
