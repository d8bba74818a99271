"""Values read by index from a uniform byte offset (tiles of up to 64 columns), and workgroups of one wavefront."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_narrow import kernels_of
from test_gpu_parity import check_c, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


def simds():
    import torch
    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


def test_values_beyond_two_gib(gpu):  # noqa: F811
    """599 M stored entries: byte offsets of values with the top bit of 32 set, by index at every width that has it."""
    import torch
    M, K = 16 * (7 * simds() // 2 + 16), 10400
    assert 4 * M * K > 1 << 31
    gen = torch.Generator(device="cuda").manual_seed(3)
    rowptr = torch.arange(M + 1, dtype=torch.int64, device="cuda").mul_(K).to(torch.int32)
    colind = torch.arange(K, dtype=torch.int32, device="cuda").repeat(M)
    vals = torch.randint(-1, 2, (M, K), generator=gen, device="cuda", dtype=torch.int8).to(torch.float32)
    plan = gpu.spmm_plan(M, K, rowptr, colind, vals.flatten())
    del rowptr, colind
    print(f"planned {M} x {K}, every entry stored", flush=True)
    for N in (16, 32, 48, 64):
        B = torch.randint(-3, 4, (K, N), generator=gen, device="cuda").to(torch.float32)
        got = gpu.spmm_exec(plan, B)
        print(f"N={N}", flush=True)
        assert torch.equal(got, vals @ B)                     # whole numbers below 2^24
        names = kernels_of(lambda: gpu.spmm_exec(plan, B))
        assert ("narrow<%d, true" if N <= 32 else "fast<%d, false, true") % (N // 16) in names, names


@pytest.mark.parametrize("N", [17, 32, 64, 100, 128, 256])
@pytest.mark.parametrize("large", [False, True])
def test_split_panels_over_a_large_b(gpu, N, large):  # noqa: F811
    """Split panels over a B of 64 MiB and more run in workgroups of one wavefront; a number of items that is no
    multiple of four or of the XCDs, and parts behind whole panels."""
    import torch
    A = W.power_law(M=16 * 1003 - 5, target_nnz=None, cap=1500, alpha=1.7, seed=N)
    K = -(-(64 << 20) // (4 * N)) if large else A.K
    col = (A.colind.astype(np.int64) * (K // A.K) + K % A.K).astype(np.int32)   # the last column is reached
    plan = gpu.spmm_plan(A.M, K, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(col).cuda(),
                         torch.from_numpy(A.vals).cuda())
    B = W.dense_b(A.K, N, 7)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    Bd = torch.zeros((K, N), device="cuda")
    Bd[torch.arange(A.K, device="cuda") * (K // A.K) + K % A.K] = torch.from_numpy(B).cuda()
    names = kernels_of(lambda: gpu.spmm_exec(plan, Bd))
    assert "k_merge" in names and (", 1>" in names) == large, names
    for product in (gpu.spmm_exec, gpu.spmm_exec_noalloc):
        Cd = torch.full((A.M, N), float("nan"), device="cuda")
        product(plan, Bd, Cd)
        torch.cuda.synchronize()
        check_c(Cd.cpu().numpy(), Cref, S)


RULES = [(16, 64, 3.5, None), (16, 44, 5, None), (31, 20, 3.5, None), (32, 20, 3.5, None), (48, 64, 3.5, None),
         (61, 64, 3.5, 6), (64, 64, 3.5, 6)]


@pytest.mark.parametrize("N, least, fewest, most, outside", [
    rule + (outside,) for rule in RULES for outside in ("", "bricks", "panels", "many") if rule[3] or outside != "many"])
def test_values_by_index_from_a_mean_of_bricks(gpu, N, least, fewest, most, outside):  # noqa: F811
    """Panels of 3 and of 2m - 3 bricks: m on average as each width wants it, or one less; as many panels a SIMD as it
    wants, or one less, and as many as it may have, or one more."""
    import torch
    P = int(fewest * simds()) + (fewest == 5) - (outside == "panels")
    if most is not None and outside != "panels":
        P = most * simds() + (outside == "many")
    rng = np.random.default_rng(N)
    m = least - (outside == "bricks")
    bricks = np.where(np.arange(P) % 2, 3, 2 * m - 3)
    if P % 2:
        bricks[-1] = m
    K = 8 * least + 9
    cols = np.concatenate([np.arange(4 * b) * 2 % K for b in bricks])   # (K is odd)
    panel = np.repeat(np.arange(P), 4 * bricks)
    rows = 16 * panel + rng.integers(0, 16, size=len(cols))
    A = W.csr_from_coo(16 * P, K, rows, cols, rng.uniform(-1, 1, len(cols)).astype(np.float32))
    plan = make_plan(gpu, A)
    assert gpu.spmm_plan_export(plan)["brick_mask"].shape[0] // P == m
    B = W.dense_b(A.K, N, 3)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    got = []
    names = kernels_of(lambda: got.append(gpu.spmm_exec(plan, torch.from_numpy(B).cuda())))
    kernel = "narrow<%d, %s, false, 4>" if N <= 32 else "fast<%d, false, %s, 4>"
    assert kernel % ((N + 15) // 16, "false" if outside else "true") in names, names
    check_c(got[0].cpu().numpy(), Cref, S)


def test_values_by_index_in_several_tiles_of_a_panel(gpu):  # noqa: F811
    """Scattered panels on tiles of 64 columns, more than ten wavefronts a SIMD."""
    import torch
    P, bricks, N, rng = 5 * simds() + 1, 64, 128, np.random.default_rng(3)
    K = 16 * P
    cols = (rng.integers(0, K // 4, P * bricks)[:, None] * 4 + np.arange(4)).ravel()
    rows = 16 * np.repeat(np.arange(P), 4 * bricks) + rng.integers(0, 16, len(cols))
    rows[::4 * bricks], rows[1::4 * bricks] = 16 * np.arange(P), 16 * np.arange(P)
    cols[::4 * bricks], cols[1::4 * bricks] = 0, K - 1      # (so that no panel has fewer)
    extra = 16 * np.arange(P) + 1, np.full(P, 8)
    A = W.csr_from_coo(K, K, np.concatenate([rows] + [extra[0]] * 12), np.concatenate([cols] + [extra[1] + 40 * i for i in range(12)]),
                       rng.uniform(-1, 1, len(rows) + 12 * P).astype(np.float32))
    plan = make_plan(gpu, A)
    assert gpu.spmm_plan_export(plan)["brick_mask"].shape[0] >= 64 * P
    B = W.dense_b(A.K, N, 3)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    got = []
    names = kernels_of(lambda: got.append(gpu.spmm_exec(plan, torch.from_numpy(B).cuda())))
    assert "fast<4, false, true, 4>" in names, names
    check_c(got[0].cpu().numpy(), Cref, S)
