"""fp32 calls of few columns at many ranks, on the GPU, bit for bit against the
oracle: the kernel that deals the ranks out over a workgroup's waves, at every
step count, on both sides of a workgroup's 16 columns, of the ranks a wave
covers and of the size up to which it is taken; batches with and without
gaps, blocks of no, one and several elements, and signed zeros, whose maximum
shows every combination's operand order."""
import numpy as np
import pytest
import torch

import oracle
from paper_2004_09362_amd import ar
from test_gpu_line_grids import check
from test_gpu_parity import DEV, bits, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [79, 80, 81, 95, 96, 97, 98, 99, 113, 126, 127, 128])
def test_every_step_count(P):
    L = (P - 1).bit_length()
    for k in range(L, 2 * L + 1):
        for n, B, gap, lead in ((1, 1, 0, 0), (15, 1, 0, 1), (16, 1, 0, 0), (17, 1, 0, 2), (31, 1, 0, 3), (106, 1, 0, 1), (P + 1, 3, 0, 0), (33, 5, 7, 2),
                                (4095, 1, 0, 0), (4097, 1, 0, 0), (1024, 4, 1, 0)):
            check(P, n, k, B=B, gap=gap, lead=lead, op=("sum", "max")[(n + k) % 2])


@pytest.mark.parametrize("P", [80, 97, 127])
def test_signed_zeros(P):
    L = (P - 1).bit_length()
    rng = np.random.default_rng(P)
    for k in range(L, 2 * L + 1):
        x = np.where(rng.random((P, 500)) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
        x[rng.integers(P), 7] = np.float32("nan")
        x[rng.integers(P), 9] = np.float32("inf")
        for op in ("sum", "max"):
            X = torch.from_numpy(x).to(DEV)
            plan = ar.Plan(P, 500, "float32", op, k)
            note("small call, signed zeros P=%d k=%d %s" % (P, k, op))
            plan([X[i] for i in range(P)])
            torch.cuda.synchronize()
            got, want = X.cpu().numpy(), oracle.allreduce(x, k, op)
            nan = np.isnan(want)
            assert np.array_equal(np.isnan(got), nan) and np.array_equal(bits(got)[~nan], bits(want)[~nan]), (P, k, op)
            plan.close()
