"""Split panels beside whole ones: the brick kernels take whole panels from panel_ptr and the parts of the
others from a list, told apart by one number of bricks."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import INT_KEYS, check_c, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


def panels_of(bricks):
    """A matrix whose panel p has bricks[p] bricks; the last panel has five rows."""
    M, K = 16 * len(bricks) - 11, 4 * max(bricks)
    keep = np.zeros((M, K), bool)
    rng = np.random.default_rng(len(bricks) + max(bricks))
    for p, n in enumerate(bricks):
        rows = keep[16 * p:16 * p + 16]
        rows[:, :4 * n] = rng.random((len(rows), 4 * n)) < 0.3
        rows[p % len(rows), :4 * n] = True              # every column occurs
    r, c = np.nonzero(keep)
    return W.csr_from_coo(M, K, r, c, rng.uniform(-1, 1, len(r)).astype(np.float32))


@pytest.mark.parametrize("mode", ["fp32", "bf16x6", "shared"])
@pytest.mark.parametrize("parts", [2, 3, 5])
def test_panels_around_the_smallest_that_is_split(gpu, mode, parts):  # noqa: F811
    import torch
    edge = 4 * (parts - 1)                              # bricks of the largest panel that stays whole
    A = panels_of([edge + 1, 0, edge, 1, edge + 1, edge + 2, edge, 40, 0, edge - 1, edge + 1])
    N = 256 if mode == "shared" else 48
    plan = make_plan(gpu, A)
    if mode == "bf16x6":
        gpu.spmm_plan_set_precision(plan, gpu.PRECISION_BF16X6)
    if mode == "shared":
        gpu.spmm_plan_set_tile_sharing(plan, gpu.SHARE_WORKGROUP)
    gpu.spmm_plan_set_split(plan, parts)
    ptr = gpu.spmm_plan_export(plan)["panel_ptr"].astype(np.int64)
    items = [[int(x) for x in i] for i in gpu.spmm_plan_worklist(plan, N)["items"]]
    at = 0
    for p in range(len(ptr) - 1):                       # in panel order, every brick once
        mine = [i for i in items if i[0] == p]
        assert items[at:at + len(mine)] == mine
        at += len(mine)
        assert (len(mine) > 1) == (ptr[p + 1] - ptr[p] > edge)
        assert [i[1] for i in mine] + [ptr[p + 1]] == [ptr[p]] + [i[2] for i in mine]
    assert at == len(items)
    B = W.dense_b(A.K, N, 5)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    for product in (gpu.spmm_exec, gpu.spmm_exec_noalloc):
        Cd = torch.full((A.M, N), float("nan"), device="cuda")
        product(plan, torch.from_numpy(B).cuda(), Cd)
        torch.cuda.synchronize()
        check_c(Cd.cpu().numpy(), Cref, S)


@pytest.mark.parametrize("panels", [261758, 261759, 261760, 262200])
@pytest.mark.parametrize("scattered", [False, True])
def test_split_panels_around_what_pinned_memory_holds(gpu, panels, scattered):  # noqa: F811
    """A megabyte of pinned memory holds the counters and panel_ptr of 261,759 panels; more are copied another
    way.  Mostly empty rows, a few heavy panels at both ends and in the middle."""
    M, K = 16 * panels - 3, 1 << 20
    rng = np.random.default_rng(panels)
    rows, cols = [], []
    for p, n in ((0, 400), (1, 30), (777, 90), (panels // 2, 801), (panels - 2, 3), (panels - 1, 500)):
        c = rng.choice(K, n, replace=False) if scattered else 5 * p + np.arange(n)
        r = 16 * p + rng.integers(0, 13, n)
        rows.append(r)
        cols.append(c)
    light = np.setdiff1d(rng.integers(0, panels, 4000), [0, 1, 777, panels // 2, panels - 2, panels - 1])
    rows.append(16 * light)
    cols.append(light % K)
    r, c = np.concatenate(rows), np.concatenate(cols) % K
    A = W.csr_from_coo(M, K, r, c, rng.uniform(-1, 1, len(r)).astype(np.float32))
    ref = oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals)
    other = make_plan(gpu, panels_of([40, 7]))          # its words are not this plan's
    gpu.spmm_plan_destroy(other)
    plan = make_plan(gpu, A)
    got, exp = gpu.spmm_synergy(plan, 48), oracle.synergy(A.M, A.K, 48, A.rowptr, A.colind, ref)
    for k in INT_KEYS:
        assert got[k] == exp[k], (k, got[k], exp[k])
    wl = gpu.spmm_plan_worklist(plan, 48)
    items = np.array([[int(x) for x in i] for i in wl["items"]], np.int64)
    ptr = gpu.spmm_plan_export(plan)["panel_ptr"].astype(np.int64)
    np.testing.assert_array_equal(ptr, ref["panel_ptr"])
    first = np.flatnonzero(np.diff(items[:, 0], prepend=-1))      # a panel's first part
    np.testing.assert_array_equal(items[first, 0], np.arange(panels))
    np.testing.assert_array_equal(items[first, 1], ptr[:-1])
    np.testing.assert_array_equal(items[np.append(first[1:], len(items)) - 1, 2], ptr[1:])
    inner = np.setdiff1d(np.arange(len(items)), first)            # further parts begin where the one before ends
    np.testing.assert_array_equal(items[inner, 1], items[inner - 1, 2])
    assert len(inner) >= 4
