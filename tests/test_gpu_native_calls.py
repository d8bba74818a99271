"""The calls that go past ctypes: the same results and refusals as the general code, on the current stream."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import check_c, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


def both(call, monkeypatch, gpu):  # noqa: F811
    """What `call` does with and without the module: its value, or the exception's type and text."""
    import torch

    def outcome():
        try:
            r = call()
            torch.cuda.synchronize()
            return r.clone() if isinstance(r, torch.Tensor) else r
        except Exception as e:
            return type(e), str(e)

    mine = outcome()
    with monkeypatch.context() as m:
        m.setattr(gpu, "_native", gpu._ThroughCtypes)
        return mine, outcome()


def test_refusals_and_forms_are_those_of_the_general_code(gpu, monkeypatch):  # noqa: F811
    import torch
    A = W.clustered_blocks(500, 4, 40, seed=3)
    plan = make_plan(gpu, A)
    gone = make_plan(gpu, A)
    gpu.spmm_plan_destroy(gone)
    N = 48
    B = torch.from_numpy(W.dense_b(A.K, N, 5)).cuda()
    C = torch.empty((A.M, N), device="cuda")
    vals = torch.from_numpy(A.vals).cuda()
    rp, ci = torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(A.colind).cuda()
    like = torch.Tensor._make_subclass(type("Like", (torch.Tensor,), {}), B)
    products = {
        "plain": (plan, B, C), "no C": (plan, B, None), "parameter": (plan, torch.nn.Parameter(B), C),
        "subclass": (plan, like, C), "strided B": (plan, B.t().contiguous().t(), C), "strided C": (plan, B, torch.empty((N, A.M), device="cuda").t()),
        "double B": (plan, B.double(), C), "half C": (plan, B, C.half()), "host B": (plan, B.cpu(), C), "host C": (plan, B, C.cpu()),
        "rows of B": (plan, B[:-1], C), "rows of C": (plan, B, C[:-1]), "width of C": (plan, B, C[:, :-1].contiguous()),
        "flat B": (plan, B.flatten(), C), "three dimensions": (plan, B[None], C), "no columns": (plan, B[:, :0].contiguous(), C[:, :0].contiguous()),
        "destroyed": (gone, B, C), "an array": (plan, B.cpu().numpy(), C), "not a tensor": (plan, None, C),
        "offset": (plan, torch.cat([B.flatten()[:1], B.flatten()])[1:].view(A.K, N), C),
    }
    for name, (p, b, c) in products.items():
        for entry in (gpu.spmm_exec, gpu.spmm_exec_noalloc):
            if c is None and entry is gpu.spmm_exec_noalloc:
                continue
            x, y = both(lambda: entry(p, b, c), monkeypatch, gpu)
            assert type(x) is type(y), (name, x, y)
            assert torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y, (name, x, y)
    updates = {"plain": vals, "short": vals[:-1], "double": vals.double(), "host": vals.cpu(), "strided": torch.stack([vals, vals], 1)[:, 0]}
    for name, v in updates.items():
        x, y = both(lambda: gpu.spmm_plan_update_values(plan, v), monkeypatch, gpu)
        assert x == y, (name, x, y)
    bad = ci.clone()
    bad[0] = -1
    plans = {"plain": (A.M, A.K, rp, ci, vals), "numpy sizes": (np.int64(A.M), np.int64(A.K), rp, ci, vals), "rows": (A.M + 1, A.K, rp, ci, vals),
             "values": (A.M, A.K, rp, ci, vals[:-1]), "long": (A.M, A.K, rp.long(), ci, vals), "host": (A.M, A.K, rp.cpu(), ci, vals),
             "column": (A.M, A.K, rp, bad, vals), "negative": (A.M, -1, rp, ci, vals), "no entries": (3, 5, rp[:1].repeat(4), ci[:0], vals[:0])}
    for name, a in plans.items():
        x, y = both(lambda: gpu.spmm_plan_sizes(gpu.spmm_plan(*a)), monkeypatch, gpu)
        assert x == y, (name, x, y)


def test_wrapped_tensors_are_refused(gpu, monkeypatch):  # noqa: F811
    """Tensors without memory of their own (vmap's): an exception, as before, and no product."""
    import torch
    A = W.clustered_blocks(200, 4, 40, seed=3)
    plan = make_plan(gpu, A)
    B = torch.from_numpy(W.dense_b(A.K, 16, 5)).cuda().repeat(2, 1, 1)
    C = torch.zeros((A.M, 16), device="cuda")
    x, y = both(lambda: torch.vmap(lambda b: gpu.spmm_exec(plan, b, C))(B), monkeypatch, gpu)
    assert x[0] is y[0] and issubclass(x[0], Exception), (x, y)
    assert not C.any()


def test_current_stream_and_capture(gpu):  # noqa: F811
    """The product goes to the stream that is current: behind work of that stream, and into a graph."""
    import torch
    A = W.clustered_blocks(3000, 6, 90, seed=3)
    plan = make_plan(gpu, A)
    N = 64
    host = W.dense_b(A.K, N, 5)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, host)
    good = torch.from_numpy(host).cuda()
    B, C = torch.zeros_like(good), torch.zeros((A.M, N), device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        B.copy_(good)
        gpu.spmm_exec(plan, B, C)
    side.synchronize()
    check_c(C.cpu().numpy(), Cref, S)
    g = torch.cuda.CUDAGraph()
    new_vals = torch.from_numpy(-A.vals).cuda()
    with torch.cuda.graph(g):
        gpu.spmm_plan_update_values(plan, new_vals)
        gpu.spmm_exec_noalloc(plan, B, C)
    for _ in range(3):
        C.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        check_c(-C.cpu().numpy(), Cref, S)
