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


def kernels_of(call):
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as seen:
        call()
        torch.cuda.synchronize()
    return " ".join(e.key for e in seen.key_averages())


@pytest.mark.parametrize("listed", ["exceptions", "heavy first", "class route"])
def test_the_rule_sees_split_panels_in_every_list(gpu, listed):  # noqa: F811
    """B is small: split panels take this kernel up to N = 8, whole ones up to 32, however the work is listed."""
    import torch
    A = panels_of(BRICKS)
    plan = make_plan(gpu, A)
    if listed == "heavy first":
        gpu.spmm_plan_set_order(plan, gpu.ORDER_HEAVY_FIRST)
    if listed == "class route":
        gpu.spmm_plan_set_route(plan, gpu.ROUTE_CLASS)
    for parts in (3, gpu.SPLIT_NEVER):
        gpu.spmm_plan_set_split(plan, parts)
        for N in (8, 16, 32, 33):
            B = torch.from_numpy(W.dense_b(A.K, N, 7)).cuda()
            gpu.spmm_exec(plan, B)                            # (the first product uploads its list)
            names = kernels_of(lambda: gpu.spmm_exec(plan, B))
            assert ("k_merge" in names) == (parts == 3), names
            narrow = N <= (8 if parts == 3 else 32)
            assert ("k_spmm_mfma_narrow" in names, "k_spmm_mfma_fast" in names) == (narrow, not narrow), names


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


@pytest.mark.parametrize("N, wide", [(8, 0), (16, 0), (20, 0), (32, 0), (48, 0), (48, 3), (64, 4), (77, 5), (96, 6), (100, 7),
                                     (128, 8), (144, 5)])
def test_infinities_stay_where_the_other_tiles_have_them(gpu, N, wide):  # noqa: F811
    """A panel's rows with an entry in the column of an infinity are infinite, its other rows NaN (0 * inf), and
    no other panel has either, whatever place the column's brick has in a load or chunk, on the narrow tiles of few
    panels and on wide ones."""
    import torch
    A = more = panels_of(BRICKS)
    rows = torch.arange(A.M)
    if wide:
        from test_gpu_widths import among_empty_panels
        more, rows = among_empty_panels(A, 3.6)
    plan = make_plan(gpu, more)
    gpu.spmm_plan_set_split(plan, gpu.SPLIT_NEVER)
    names = kernels_of(lambda: gpu.spmm_exec(plan, torch.zeros((A.K, N), device="cuda")))
    assert ("fast<%d, " % wide if wide else "narrow<") in names, names
    dense = np.zeros((A.M, A.K), np.float32)
    dense[np.repeat(np.arange(A.M), np.diff(A.rowptr)), A.colind] = A.vals
    bricks = np.repeat(BRICKS, 16)[:A.M]
    for n in BRICKS[1:]:
        B = W.dense_b(A.K, N, 7)
        B[4 * n - 1] = np.inf                              # the last column of panels of n bricks
        C = gpu.spmm_exec(plan, torch.from_numpy(B).cuda())
        infinite = int(torch.isfinite(C).logical_not().sum())
        C = C[rows.cuda()].cpu().numpy()
        assert infinite == np.count_nonzero(~np.isfinite(C))
        entry = dense[:, 4 * n - 1]
        expect = np.where(bricks < n, 0.0, np.where(entry != 0, np.copysign(np.inf, entry), np.nan))
        got = np.where(np.isfinite(C), 0.0, C)
        np.testing.assert_array_equal(got, np.repeat(expect[:, None], N, 1).astype(np.float32))


@pytest.mark.parametrize("N, log2_k", [(9, 21), (13, 21), (16, 21), (17, 20), (22, 20), (31, 20), (32, 20)])
@pytest.mark.parametrize("heavy_first", [False, True])
def test_partial_tiles_where_b_is_large(gpu, N, log2_k, heavy_first):  # noqa: F811
    """Split panels beyond N = 8 take this kernel where B has 64 MiB and more: the columns of a small matrix,
    far apart."""
    import torch
    A = panels_of(BRICKS)
    K = 1 << log2_k
    at = (np.arange(A.K) * (K // A.K) + N).astype(np.int32)
    assert at[-1] < K and K * N * 4 >= 64 << 20
    plan = gpu.spmm_plan(A.M, K, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(at[A.colind]).cuda(),
                         torch.from_numpy(A.vals).cuda())
    gpu.spmm_plan_set_split(plan, 3)
    if heavy_first:
        gpu.spmm_plan_set_order(plan, gpu.ORDER_HEAVY_FIRST)
    B = W.dense_b(A.K, N, 7)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    Bd = torch.zeros((K, N), device="cuda")
    Bd[torch.from_numpy(at).long().cuda()] = torch.from_numpy(B).cuda()
    names = kernels_of(lambda: gpu.spmm_exec(plan, Bd))
    assert "k_spmm_mfma_narrow" in names and "k_merge" in names, names
    for product in (gpu.spmm_exec, gpu.spmm_exec_noalloc):
        Cd = torch.full((A.M, N), float("nan"), device="cuda")
        product(plan, Bd, Cd)
        torch.cuda.synchronize()
        check_c(Cd.cpu().numpy(), Cref, S)
