"""Plans whose counts are at the upper end of what is accepted, where a launch of a wavefront a brick
or a panel would hold 2^32 threads, or 32-bit byte offsets end.  The matrices are regular or nearly
empty, so that C and the format follow from the construction."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def test_csr_route_with_2_to_26_bricks(gpu):  # noqa: F811
    """Row r of every panel holds columns 256 r .. 256 r + 255: 1024 bricks a panel, one row each.
    Columns, values and a later update all reach the CSR kernel."""
    import torch
    P, K, N = 1 << 16, 4096, 4
    M = 16 * P
    rowptr = torch.arange(M + 1, dtype=torch.int64, device="cuda").mul_(256).to(torch.int32)
    colind = torch.arange(K, dtype=torch.int32, device="cuda").repeat(P)
    gen = torch.Generator(device="cuda").manual_seed(3)

    def fresh():
        return torch.randint(-4, 5, (M * 256,), generator=gen, device="cuda").to(torch.float32)

    B = torch.randint(-4, 5, (K, N), generator=gen, device="cuda").to(torch.float32)

    def expected(vals):   # whole numbers: every order of summation gives the same
        return torch.bmm(vals.view(P, 16, 256).transpose(0, 1).contiguous(), B.view(16, 256, N)).transpose(0, 1)

    vals = fresh()
    plan = gpu.spmm_plan(M, K, rowptr, colind, vals)
    assert gpu.spmm_plan_sizes(plan)["n_bricks"] == 1 << 26
    print("planned 2^26 bricks", flush=True)
    gpu.spmm_plan_set_route(plan, gpu.ROUTE_VALU)
    assert torch.equal(gpu.spmm_exec(plan, B).view(P, 16, N), expected(vals))
    vals = fresh()
    gpu.spmm_plan_update_values(plan, vals)
    assert torch.equal(gpu.spmm_exec(plan, B).view(P, 16, N), expected(vals))


def test_plan_of_2_to_30_rows(gpu):  # noqa: F811
    """2^26 panels, nearly all empty: the bricks are those of the few others by themselves."""
    import torch
    M, K = 1 << 30, 1000
    panels = np.array([0, 1, 5, 1 << 22, (1 << 25) + 3, (1 << 26) - 1])
    A = W.uniform_random(16 * len(panels), K, 0.05, 7)
    ref = oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals)
    length = torch.zeros(M, dtype=torch.int32, device="cuda")
    rows = (panels[:, None] * 16 + np.arange(16)).ravel()
    length[torch.from_numpy(rows).cuda()] = torch.from_numpy(np.diff(A.rowptr).astype(np.int32)).cuda()
    rowptr = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    torch.cumsum(length, 0, dtype=torch.int32, out=rowptr[1:])
    del length
    assert int(rowptr[-1]) == A.nnz
    print("planning 2^30 rows", flush=True)
    plan = gpu.spmm_plan(M, K, rowptr, torch.from_numpy(A.colind).cuda(), torch.from_numpy(A.vals).cuda())
    got = gpu.spmm_plan_export(plan)
    for k in ("brick_cols", "brick_mask", "brick_valptr", "vals"):
        assert np.array_equal(got[k], ref[k]), k
    bricks = np.diff(got["panel_ptr"])
    assert np.array_equal(bricks[panels], np.diff(ref["panel_ptr"]))
    assert int(bricks.sum()) == len(ref["brick_mask"]) and got["panel_ptr"][0] == 0


def test_tile_reported_where_values_are_beyond_32bit_offsets(gpu):  # noqa: F811
    """2^30 stored entries: the general kernel runs, on tiles of a power of two columns, and the work
    list says so."""
    import torch
    M = K = 1 << 15
    rowptr = torch.arange(M + 1, dtype=torch.int64, device="cuda").mul_(K).to(torch.int32)
    colind = torch.arange(K, dtype=torch.int32, device="cuda").repeat(M)
    gen = torch.Generator(device="cuda").manual_seed(3)
    vals = torch.randint(-1, 2, (M, K), generator=gen, device="cuda", dtype=torch.int8).to(torch.float32)
    plan = gpu.spmm_plan(M, K, rowptr, colind, vals.flatten())
    del rowptr, colind
    print(f"planned {M} x {K}, every entry stored", flush=True)
    B = torch.randint(-3, 4, (K, 48), generator=gen, device="cuda").to(torch.float32)
    assert torch.equal(gpu.spmm_exec(plan, B), vals @ B)      # whole numbers below 2^24
    assert gpu.spmm_plan_worklist(plan, 48)["n_tile"] == 64
