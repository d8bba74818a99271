"""Device memory that plans let go is kept for the next ones: bounded, given back on request, and
never handed out while anything uses it -- plans made, used and destroyed from several threads on
streams of their own all give the oracle's product."""
import threading

import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import check_c, gpu, make_plan, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_kept_memory_is_bounded_and_given_back(gpu):  # noqa: F811
    A = W.clustered_blocks(120_000, 10, 256, seed=5)          # 3.6 M entries: 40 MB a plan
    make_plan(gpu, A).destroy()
    gpu._lib.spmm_plan_destroy(None)
    dev = to_dev(A)
    base = free_bytes()
    plans = [gpu.spmm_plan(A.M, A.K, *dev) for _ in range(20)]   # 800 MB at once
    held = base - free_bytes()
    for p in plans:
        p.destroy()
    kept = base - free_bytes()
    assert 0 < kept <= 520 << 20 < held
    gpu._lib.spmm_plan_destroy(None)
    assert base - free_bytes() <= 4 << 20


def test_plans_do_not_hold_what_they_were_made_with(gpu):  # noqa: F811
    """Working memory has a byte a column: small matrices of many columns, on each of the three paths."""
    K = 6_000_000
    band = W.csr_from_coo(2000, K, np.repeat(np.arange(2000), 5), np.tile(np.arange(5), 2000) + np.repeat(np.arange(2000), 5))
    for A in (band, W.csr_from_coo(2000, K, np.repeat(np.arange(2000), 5), np.arange(10000) * 599),
              W.csr_from_coo(32, K, np.repeat([3, 20], 9000), np.tile(np.arange(9000) * 666, 2))):
        dev = to_dev(A)
        gpu._lib.spmm_plan_destroy(None)
        base = free_bytes()
        plans = [gpu.spmm_plan(A.M, A.K, *dev) for _ in range(16)]
        gpu._lib.spmm_plan_destroy(None)
        assert base - free_bytes() <= 16 * (2 << 20)
        for p in plans:
            p.destroy()


def test_plans_of_several_threads_and_streams(gpu):  # noqa: F811
    import torch
    mats = [W.clustered_blocks(20_000, 8, 200, seed=1), W.power_law(M=30_000, target_nnz=None, cap=900, seed=2),
            W.brick_sweep(0.4, M=16384, target_nnz=300_000, seed=3), W.tiny_banded(M=25_000, seed=4)]
    N = 40
    cases = []
    for A in mats:
        B = W.dense_b(A.K, N, 9)
        cases.append((A, to_dev(A), torch.from_numpy(B).cuda(), *oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)))
    torch.cuda.synchronize()
    results, errors = [], []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for r in range(6):
                    i = (t + r) % len(cases)
                    A, dev, Bd = cases[i][:3]
                    plan = gpu.spmm_plan(A.M, A.K, *dev)
                    Cd = torch.full((A.M, N), float("nan"), device="cuda")
                    gpu.spmm_exec(plan, Bd, Cd)
                    plan.destroy()
                    stream.synchronize()
                    results.append((i, Cd))
        except Exception as e:   # noqa: BLE001  (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert len(results) == 24
    for i, Cd in results:
        Cg = Cd.cpu().numpy()
        assert not np.isnan(Cg).any()
        check_c(Cg, cases[i][3], cases[i][4])


def test_giving_back_leaves_a_capture_valid(gpu):  # noqa: F811
    import torch
    A = W.clustered_blocks(20_000, 8, 200, seed=6)
    B = W.dense_b(A.K, 40, 9)
    make_plan(gpu, W.clustered_blocks(60_000, 10, 256, seed=5)).destroy()
    plan, Bd, Cd = make_plan(gpu, A), torch.from_numpy(B).cuda(), torch.empty((A.M, 40), device="cuda")
    before = free_bytes()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gpu.spmm_exec(plan, Bd, Cd)
        gpu._lib.spmm_plan_destroy(None)
    assert free_bytes() - before >= 8 << 20
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    for _ in range(2):
        Cd.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        check_c(Cd.cpu().numpy(), Cref, S)
