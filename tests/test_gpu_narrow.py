"""Tiles of 16 and 32 columns: items around whole and half chunks of eight bricks, at the widths where loads
of sixteen bytes end inside a row, on operands at every dword alignment."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import check_c, gpu, make_plan  # noqa: F401
from test_gpu_split_exceptions import panels_of

pytestmark = pytest.mark.gpu

BRICKS = (0, 1, 2, 3, 4, 5, 7, 8, 9, 10, 12, 15, 16, 17, 20, 23, 24, 25, 33)


@pytest.mark.parametrize("N", [4, 5, 7, 8, 13, 15, 16, 17, 18, 22, 31, 32])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_chunks_and_widths(gpu, N, offset):  # noqa: F811
    import torch
    A = panels_of(BRICKS)
    plan = make_plan(gpu, A)
    gpu.spmm_plan_set_split(plan, gpu.SPLIT_NEVER)
    B = W.dense_b(A.K, N, 7)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    Bd = torch.empty(A.K * N + 4, device="cuda")[offset:offset + A.K * N].view(A.K, N)
    Bd.copy_(torch.from_numpy(B))
    whole = torch.full((A.M * N + 8,), 7.0, device="cuda")
    Cd = whole[offset:offset + A.M * N].view(A.M, N)
    Cd.fill_(float("nan"))
    gpu.spmm_exec(plan, Bd, Cd)
    torch.cuda.synchronize()
    check_c(Cd.cpu().numpy(), Cref, S)
    assert bool((whole[:offset] == 7.0).all()) and bool((whole[offset + A.M * N:] == 7.0).all())


@pytest.mark.parametrize("N", [8, 16, 32])
def test_split_panels_on_either_side_of_the_rule(gpu, N):  # noqa: F811
    """Split panels take this kernel at N = 8 and the other at 16 and 32 (B is small)."""
    import torch
    A = panels_of(BRICKS)
    plan = make_plan(gpu, A)
    gpu.spmm_plan_set_split(plan, 3)
    B = W.dense_b(A.K, N, 7)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    C = gpu.spmm_exec(plan, torch.from_numpy(B).cuda())
    torch.cuda.synchronize()
    check_c(C.cpu().numpy(), Cref, S)
