"""The execute calls' native part (csrc/bind.cpp): what it takes gives the same
results as the Python path, and what it does not take reaches that path, which
accepts or names it.  Every call is checked anew: a tensor that passed once and
changed since is refused."""
import numpy as np
import pytest
import torch

import oracle
from paper_2004_09362_amd import ar

P, N = 5, 64


def test_cpu_tensors_and_odd_arguments_go_to_python():
    plan = ar.Plan(P, N, "float32", "sum", 6)
    info = ar._PLAN_INFO[plan.handle]
    X = [torch.zeros(N) for _ in range(P)]
    call = lambda *a: ar._bind_execute(*a)  # noqa: E731
    assert call(plan.handle, info, X, 1, 0, 0, 0, 0) is None            # not on a GPU
    assert call(plan.handle, info, [4096] * P, 1, 0, 0, 0, 0) is None   # raw addresses
    assert call(plan.handle, info, X[:-1], 1, 0, 0, 0, 0) is None       # too few
    assert call(plan.handle, info, iter(X), 1, 0, 0, 0, 0) is None      # no list or tuple
    assert call(plan.handle, info, X, 0, N, 0, 0, 0) is None            # batch below 1
    assert call(plan.handle, info, X, True, N, 0, 0, 0) is None         # no plain integers
    assert call(plan.handle, info, X, 1 << 62, 1 << 62, 0, 0, 0) is None
    assert call(plan.handle, info, X, 1 << 70, N, 0, 0, 0) is None
    assert call(plan.handle, info, X) is None


class Sub(torch.Tensor):
    pass


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["list", "tuple", "iterator", "parameters", "subclass", "mixed", "stream", "context"])
def test_accepted_forms(form):
    plan = ar.Plan(P, N, "float32", "sum", 4)
    x = np.random.default_rng(7).normal(size=(P, N)).astype(np.float32)
    rows = [torch.from_numpy(x[i].copy()).cuda() for i in range(P)]
    if form == "parameters":
        rows = [torch.nn.Parameter(r, requires_grad=False) for r in rows]
    if form == "subclass":
        rows = [r.as_subclass(Sub) for r in rows]
    bufs = {"tuple": tuple(rows), "iterator": iter(rows),
            "mixed": [r.data_ptr() if i % 2 else r for i, r in enumerate(rows)]}.get(form, rows)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    if form == "stream":
        plan(bufs, stream=s)
    elif form == "context":
        with torch.cuda.stream(s):
            plan(bufs)
    else:
        plan(bufs)
    torch.cuda.synchronize()
    got = np.stack([r.detach().cpu().numpy() for r in rows])
    assert np.array_equal(got.view(np.uint32), oracle.allreduce(x, 4, "sum").view(np.uint32))
    plan.close()


@pytest.mark.gpu
def test_a_stream_handle_takes_the_native_path(monkeypatch):
    """A stream given as its handle is no reason to check every rank in Python."""
    plan = ar.Plan(P, N, "float32", "sum", 4)
    x = np.random.default_rng(8).normal(size=(P, 2, N)).astype(np.float32)
    X = torch.from_numpy(x).cuda()
    rows = list(X.unbind(0))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    monkeypatch.setattr(ar, "_ptr_table", lambda *a, **k: pytest.fail("the Python path ran"))
    plan.batched(rows, 1, N, stream=s.cuda_stream)
    plan.batched([r[1] for r in rows], 1, N, stream=0)
    torch.cuda.synchronize()
    assert np.array_equal(X.cpu().numpy().view(np.uint32), oracle.allreduce_batched(x, 4, "sum").view(np.uint32))
    plan.close()


def test_tables_of_raw_addresses():
    plan = ar.Plan(P, N, "float32", "sum", 4)
    addrs = [4096 * (i + 1) for i in range(P)]
    for form in (addrs, tuple(addrs), iter(addrs), [np.int64(a) for a in addrs], [True] + addrs[1:]):
        want = [int(form[0])] + addrs[1:] if isinstance(form, list) else addrs
        assert list(ar._ptr_table(plan.handle, form)) == want
    for bad in (addrs[:-1], addrs + [4096], []):
        with pytest.raises(ar.ArError, match="P=5 ranks"):
            ar._ptr_table(plan.handle, bad)
    with pytest.raises(ar.ArError, match="batch"):
        ar._ptr_table(plan.handle, addrs, 0, N)
    plan.close()


@pytest.mark.gpu
def test_refused_buffers_name_the_fault_each_time():
    plan = ar.Plan(P, N, "float32", "sum", 4)
    rows = [torch.zeros(N, device="cuda") for _ in range(P)]

    def refused(bufs, what, batch=1, stride=N):
        with pytest.raises(ar.ArError, match=what) as ei:
            plan.batched(bufs, batch, stride)
        assert ei.value.status in (ar.AR_ERR_INVALID_ARG, ar.AR_ERR_ALIAS)

    plan(rows)
    refused(rows[:4], "got 4")
    refused(rows[:4] + [torch.zeros(N)], "not on a GPU")
    refused(rows[:4] + [torch.zeros(N, dtype=torch.int32, device="cuda")], "dtype")
    refused(rows[:4] + [torch.zeros(2 * N, device="cuda")[::2]], "contiguous")
    refused(rows[:4] + [torch.zeros(N - 1, device="cuda")], "holds 63")
    refused(rows, "holds 64", batch=2)
    refused(rows, "batch", batch=0)
    refused(rows[:4] + [rows[0]], "overlap")
    # the same tensor objects at the same addresses, one with a smaller storage
    plan(rows)
    rows[2].untyped_storage().resize_(4 * (N - 1))
    refused(rows, "holds 63")
    torch.cuda.synchronize()
    plan.close()
