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

from test_gpu_line_grids import check

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


@pytest.mark.parametrize("P", [5, 24, 100])
def test_split_by_size_and_one_launch_agree(P):
    """Rank instances just below and at the size from which int32 plans of
    12 ranks and more split, rows off the lines."""
    for n in ((1 << 20) - 1, 1 << 20):
        check(P, n, L(P), lead=1, dtype="int32", op="max")
