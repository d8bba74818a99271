"""Few panels are multiplied on narrower tiles than many: widths around every tile, ragged and whole, on either
side of the counts where the tile changes, with and without split panels."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_narrow import kernels_of
from test_gpu_parity import check_c, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu

WIDTHS = (20, 31, 32, 47, 48, 50, 64, 65, 77, 80, 96, 97, 112, 113, 127, 128, 129, 144, 160, 191, 192, 200, 223, 255,
          256, 257, 300)


def simds():
    import torch
    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


# the tile that even panels run on, by panels a SIMD (2.5: one panel more)
TILES = {0.02: {20: 16, 32: 16, 64: 16, 96: 16, 128: 16, 256: 16}, 0.5: {31: 16, 32: 16},
         0.6: {31: 32, 32: 32, 64: 16, 96: 32, 128: 32, 256: 64}, 1.5: {32: 32, 64: 32, 96: 96, 128: 64, 256: 128},
         1.6: {64: 64, 96: 96, 128: 128, 256: 128}, 2.4: {64: 64, 96: 96, 128: 64, 256: 128}, 2.5: {64: 64, 128: 128, 256: 128},
         2.6: {64: 64, 128: 128, 256: 128}}


@pytest.mark.parametrize("per_simd", sorted(TILES))
@pytest.mark.parametrize("split", [0, 2])
@pytest.mark.parametrize("scattered", [False, True])
def test_every_width_on_either_side_of_the_rule(gpu, per_simd, split, scattered):  # noqa: F811
    import torch
    panels = int(per_simd * simds()) + (per_simd == 2.5)
    rows = 16 * panels - 11                                 # a ragged last panel
    A = W.uniform_random(rows, rows, 0.02, 3) if scattered and panels < 100 else \
        W.brick_sweep(0.1, M=16 * panels, target_nnz=100 * panels, seed=5) if scattered else \
        W.clustered_blocks(rows, 2, 40, seed=7)
    plan = make_plan(gpu, A)
    gpu.spmm_plan_set_split(plan, split)
    Ball = W.dense_b(A.K, max(WIDTHS), 11)
    Call, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, Ball)
    for N in WIDTHS:
        print(f"{panels} panels, N={N} split={split} scattered={scattered}", flush=True)
        offset = (N + WIDTHS.index(N)) % 4                  # operands at every dword alignment
        Bd = torch.empty(A.K * N + 4, device="cuda")[offset:offset + A.K * N].view(A.K, N)
        Bd.copy_(torch.from_numpy(Ball[:, :N].copy()))
        whole = torch.full((A.M * N + 8,), 7.0, device="cuda")
        Cd = whole[offset:offset + A.M * N].view(A.M, N)
        Cd.fill_(float("nan"))
        gpu.spmm_exec(plan, Bd, Cd)
        torch.cuda.synchronize()
        check_c(Cd.cpu().numpy(), Call[:, :N], S[:, :N])
        assert bool((whole[:offset] == 7.0).all()) and bool((whole[offset + A.M * N:] == 7.0).all())
        if split == 0 and not scattered and N in TILES[per_simd]:
            names = kernels_of(lambda: gpu.spmm_exec(plan, Bd, Cd))
            tile = TILES[per_simd][N]
            assert ("narrow<%d, " if tile <= 32 else "fast<%d, ") % (tile // 16) in names, (N, names)


@pytest.mark.parametrize("N", [48, 64, 128])
def test_split_panels_and_lists_do_not_depend_on_the_tile(gpu, N):  # noqa: F811
    """Eq. 7 goes by the wide tiles, and the few panels here run on narrow ones."""
    import torch
    A = W.power_law(M=4000, target_nnz=None, cap=2000, alpha=1.6, seed=41)
    plan = make_plan(gpu, A)
    wl = gpu.spmm_plan_worklist(plan, N)
    assert wl["n_tile"] == min(N, 128) and wl["n_tiles"] == -(-N // 128) and wl["n_split_panels"] > 0
    B = W.dense_b(A.K, N, 42)
    Bd = torch.from_numpy(B).cuda()
    C = gpu.spmm_exec(plan, Bd)
    names = kernels_of(lambda: gpu.spmm_exec(plan, Bd))
    assert "k_spmm_mfma_narrow" in names and "k_merge" in names, names
    again = torch.full_like(C, float("nan"))
    gpu.spmm_exec_noalloc(plan, Bd, again)
    torch.cuda.synchronize()
    assert torch.equal(C, again)
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    check_c(C.cpu().numpy(), Cref, S)


@pytest.mark.parametrize("N", [32, 64, 96, 200])
def test_infinities_stay_in_their_panels(gpu, N):  # noqa: F811
    """Tiles that read bricks in pairs or fours multiply none that is not there, in any column tile."""
    import torch
    from test_gpu_narrow import BRICKS
    from test_gpu_split_exceptions import panels_of
    A = panels_of(BRICKS)
    plan = make_plan(gpu, A)
    gpu.spmm_plan_set_split(plan, gpu.SPLIT_NEVER)
    bricks = np.repeat(BRICKS, 16)[:A.M]
    for n in BRICKS[1:]:
        B = W.dense_b(A.K, N, 7)
        B[4 * n - 1] = np.inf
        C = gpu.spmm_exec(plan, torch.from_numpy(B).cuda()).cpu().numpy()
        np.testing.assert_array_equal(np.isfinite(C), np.repeat((bricks < n)[:, None], N, 1))


def with_long_rows(A, rows, entries):
    """A with `rows` of its rows stored in `entries` columns spread over all of them."""
    at = (np.arange(rows) + 1) * A.M // (rows + 1)
    old = np.repeat(np.arange(A.M), np.diff(A.rowptr))
    keep = ~np.isin(old, at)
    row = np.concatenate([old[keep], np.repeat(at, entries)])
    col = np.concatenate([A.colind[keep], np.tile(np.arange(entries) * A.K // entries, rows)])
    return W.csr_from_coo(A.M, A.K, row, col, np.random.default_rng(rows).uniform(-1, 1, len(row)).astype(np.float32))


@pytest.mark.parametrize("per_simd, rows, entries, tiles", [
    (0.4, 1, 600, {24: 16, 32: 16}),            # half as wide as 32 while each wavefront has a SIMD
    (0.5, 1, 600, {24: 32, 32: 32}),
    (2.0, "wide", 0, {64: 64}),                  # scattered and split, but of many bricks
    (3.66, 0, 0, {64: 64, 128: 128}),            # even panels, more than narrow tiles are for,
    (3.66, 1, 1000, {64: 64, 96: 96, 128: 128, 160: 96}),     # and the same with a long row: neither a graph
    (1.2, 0, 0, {96: 96, 160: 64}),
    (1.2, 1, 1000, {96: 32, 160: 32}),           # three or five for one or two wide ones
    (2.3, 1, 1000, {96: 96, 160: 32}),
    (4.4, 1, 1000, {64: 64, 128: 64}),           # but just over what the device holds
    (6.1, 1, 1000, {64: 64, 128: 128}),
    (6.1, 30, 2000, {64: 64, 128: 64}),          # or with much of the matrix in long rows
    (2.0, "graph", 0, {64: 32, 96: 32, 128: 32}),
    (6.1, "graph", 0, {64: 64, 96: 96, 128: 64})])
def test_a_few_long_rows_do_not_make_a_graph(gpu, per_simd, rows, entries, tiles):  # noqa: F811
    import torch
    M = 16 * int(per_simd * simds())
    if rows == "graph":
        A = W.power_law(M, target_nnz=int(2.854 * M), seed=3)
    elif rows == "wide":
        A = with_long_rows(W.uniform_random(M, M, 6 / M, 3), M // 16 // 40 + 1, 1500)
    else:
        A = W.clustered_blocks(M, 4, 60, seed=7)
        if rows:
            A = with_long_rows(A, rows, entries)
    plan = make_plan(gpu, A)
    Ball = W.dense_b(A.K, max(tiles), 11)
    Call, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, Ball)
    for N, tile in tiles.items():
        assert (gpu.spmm_plan_worklist(plan, N)["n_split_panels"] > 0) == (rows != 0)
        B = torch.from_numpy(Ball[:, :N].copy()).cuda()
        C = gpu.spmm_exec(plan, B)
        names = kernels_of(lambda: gpu.spmm_exec(plan, B))
        assert "fast<%d," % (tile // 16) in names or "narrow<%d," % (tile // 16) in names, (N, names)
        check_c(C.cpu().numpy(), Call[:, :N], S[:, :N])


@pytest.mark.parametrize("N", [32, 48, 64, 80, 128])
@pytest.mark.parametrize("rows, waves", [(1, 4), (9, 4), ("graph", 1)])
def test_long_rows_over_a_large_b(gpu, N, rows, waves):  # noqa: F811
    """Workgroups of one wavefront are for graphs, not for a band with a few long rows, and not for tiles of 48 and 80."""
    import torch
    M = 16 * 4133 - 3
    A = W.power_law(M, target_nnz=int(2.854 * M), seed=3) if rows == "graph" else \
        with_long_rows(W.clustered_blocks(M, 3, 40, seed=7), rows, 3000)
    step = -(-(64 << 20) // (4 * N * A.K))
    K = step * A.K + 5                                      # 64 MiB of B
    col = (A.colind.astype(np.int64) * step + 5).astype(np.int32)
    plan = gpu.spmm_plan(A.M, K, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(col).cuda(),
                         torch.from_numpy(A.vals).cuda())
    assert gpu.spmm_plan_worklist(plan, N)["n_split_panels"] > 0
    B = W.dense_b(A.K, N, 11)
    Bd = torch.zeros((K, N), device="cuda")
    Bd[torch.arange(A.K, device="cuda") * step + 5] = torch.from_numpy(B).cuda()
    C = gpu.spmm_exec(plan, Bd)
    names = kernels_of(lambda: gpu.spmm_exec(plan, Bd))
    assert ", %d>" % (4 if N in (48, 80) else waves) in names, names
    Cref, S = oracle.spmm_f64(A.rowptr, A.colind, A.vals, B)
    check_c(C.cpu().numpy(), Cref, S)
