"""New values for an unchanged pattern where the plan keeps 16-bit steps and where it keeps entries: panels of up to
and more than 32,768 entries, numbers of entries around a workgroup's share, with the CSR copy and without."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import assert_format_equal, check_c, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


def wide_panel(entries):
    """One panel of 16 rows of that many entries in all, over a span that a bitmap holds, and two small ones."""
    rng = np.random.default_rng(entries)
    K = 8192
    keep = np.zeros(16 * K, bool)
    keep[rng.choice(16 * K, size=entries, replace=False)] = True
    r, c = np.nonzero(keep.reshape(16, K))
    more = rng.integers(0, K, size=(20, 3))
    r, c = np.r_[r, 16 + np.repeat(np.arange(20), 3)], np.r_[c, more.ravel()]
    return W.csr_from_coo(36, K, r, c, rng.uniform(-1, 1, len(r)).astype(np.float32))


CASES = {"band 2047": lambda: W.tiny_banded(M=204, per_row=10, half_width=64, seed=1), "blocks": lambda: W.clustered_blocks(3001, 6, 90, seed=2),
         "wide 32768": lambda: wide_panel(32768), "wide 32769": lambda: wide_panel(32769), "wide 2048": lambda: wide_panel(2048),
         "wide 2049": lambda: wide_panel(2049), "wide 70000": lambda: wide_panel(70000),
         "scattered": lambda: W.uniform_random(900, 40000, 0.001, 5), "graph": lambda: W.power_law(M=6000, target_nnz=None, cap=900, alpha=1.8, seed=3),
         "one": lambda: W.uniform_random(1, 1, 1.0, 7)}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("csr", [False, True])
def test_update(gpu, name, csr):  # noqa: F811
    import torch
    A = CASES[name]()
    plan = make_plan(gpu, A)
    if csr:
        gpu.spmm_plan_set_route(plan, gpu.ROUTE_VALU)
    rng = np.random.default_rng(11)
    for _ in range(2):
        vals = rng.uniform(-1, 1, A.nnz).astype(np.float32)
        gpu.spmm_plan_update_values(plan, torch.from_numpy(vals).cuda())
        assert_format_equal(gpu.spmm_plan_export(plan), oracle.build_bricks(A.M, A.rowptr, A.colind, vals))
    B = W.dense_b(A.K, 20, 4)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, vals, B)
    for route in (gpu.ROUTE_VALU, gpu.ROUTE_AUTO):            # (the first from the CSR arrays, restored or kept)
        gpu.spmm_plan_set_route(plan, route)
        C = gpu.spmm_exec(plan, torch.from_numpy(B).cuda())
        torch.cuda.synchronize()
        check_c(C.cpu().numpy(), Cref, S)


@pytest.mark.parametrize("nnz", [1, 3, 4, 2047, 2048, 2049, 4095, 4096, 4097, 6145])
@pytest.mark.parametrize("scattered", [False, True])
def test_numbers_of_entries(gpu, nnz, scattered):  # noqa: F811
    import torch
    rng = np.random.default_rng(nnz)
    M, K = 700, 700 if not scattered else 3_000_000
    cells = rng.choice(M * 40, size=nnz, replace=False)
    r = cells // 40
    c = np.minimum(r + cells % 40, K - 1) if not scattered else (cells * 104729) % K
    A = W.csr_from_coo(M, K, r, c)
    plan = make_plan(gpu, A)
    vals = rng.uniform(-1, 1, A.nnz).astype(np.float32)
    gpu.spmm_plan_update_values(plan, torch.from_numpy(vals).cuda())
    assert_format_equal(gpu.spmm_plan_export(plan), oracle.build_bricks(A.M, A.rowptr, A.colind, vals))
