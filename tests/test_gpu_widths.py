"""Every width of C from one column up, on operands that are only dword-aligned: the tiles of
16..128 columns in steps of 16, their remainders, and the vectors that end a row."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_narrow import kernels_of
from test_gpu_parity import check_c, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu

# each tile width T*16 at its first, an odd and its last column; two and three tiles
WIDTHS = (2, 3, 4, 5, 15, 17, 18, 31, 34, 47, 48, 49, 63, 65, 66, 77, 80, 81, 95, 96, 97, 98, 99, 111,
          112, 113, 114, 127, 128, 129, 144, 145, 191, 223, 255, 256, 257, 300)
GUARD = 7.0


def among_empty_panels(A, per_simd):
    """A with empty panels between its tenth and eleventh until there are `per_simd` a SIMD, as many as the wide tiles
    are for, and A's rows in it."""
    import torch
    n = 16 * int(per_simd * 4 * torch.cuda.get_device_properties(0).multi_processor_count)
    rp = A.rowptr
    more = W.CSR(A.M + n, A.K, np.concatenate([rp[:161], np.full(n, rp[160], rp.dtype), rp[161:]]), A.colind, A.vals)
    return more, torch.cat([torch.arange(160), torch.arange(160 + n, A.M + n)])


def wide_tile(N):
    tiles = -(-N // 128)
    t = -(-(-(-N // 16)) // tiles)
    return (t + 1) // 2 * 2 if tiles > 1 and N % 32 == 0 else t


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("split", [0, 2])
@pytest.mark.parametrize("wide", [False, True])
def test_any_width_any_dword_alignment(gpu, offset, split, wide):  # noqa: F811
    """`wide`: with so many panels that every width runs on its wide tile (at 256 columns not if some are split)."""
    import torch
    A = few = W.clustered_blocks(331, 6, 90, seed=3)    # a ragged last panel
    rows = torch.arange(A.M)
    if wide:
        A, rows = among_empty_panels(A, 3.6)
    plan = make_plan(gpu, A)
    gpu.spmm_plan_set_split(plan, split)
    for N in WIDTHS:
        print(f"width N={N} offset={offset} split={split}", flush=True)
        B = W.dense_b(A.K, N, 41)
        Cref, S = oracle.spmm_f64(few.rowptr, few.colind, few.vals, B)
        Bd = torch.empty(A.K * N + 4, device="cuda")[offset:offset + A.K * N].view(A.K, N)
        Bd.copy_(torch.from_numpy(B))
        whole = torch.full((A.M * N + 8,), GUARD, device="cuda")
        Cd = whole[offset:offset + A.M * N].view(A.M, N)
        Cd.fill_(float("nan"))
        gpu.spmm_exec(plan, Bd, Cd)
        torch.cuda.synchronize()
        assert not bool(torch.isnan(Cd).any()), "every element of C must be written"
        check_c(Cd[rows.cuda()].cpu().numpy(), Cref, S)
        assert int(torch.count_nonzero(Cd)) == int(torch.count_nonzero(Cd[rows.cuda()]))
        assert bool((whole[:offset] == GUARD).all()) and bool((whole[offset + A.M * N:] == GUARD).all())
        if wide and offset == 0 and not (split and N == 256):
            names = kernels_of(lambda: gpu.spmm_exec(plan, Bd, Cd))
            narrow = 4 <= N <= (8 if split else 32)
            assert ("narrow<%d, " if narrow else "fast<%d, ") % wide_tile(N) in names, (N, names)
            assert ("fast<8, true, " in names) == (N % 128 == 0), (N, names)


@pytest.mark.parametrize("N,as_wide_as", [(48, 64), (44, 64), (80, 128), (96, 128), (144, 128), (400, 128)])
def test_narrow_tiles_do_not_split_more(gpu, N, as_wide_as):  # noqa: F811
    """Eq. 7's capacity is that of the power-of-two tile, so a panel is cut into no more parts (and
    takes no more of the static scratch of spmm_exec_noalloc) because a narrower tile runs."""
    A = W.power_law(M=120000, target_nnz=None, cap=2000, alpha=1.6, seed=41)
    plan = make_plan(gpu, A)
    mine, wide = gpu.spmm_plan_worklist(plan, N), gpu.spmm_plan_worklist(plan, as_wide_as)
    assert mine["n_tile"] not in (16, 32, 64, 128)
    assert mine["resident_waves_per_cu"] == wide["resident_waves_per_cu"]
    if N <= as_wide_as:   # the same number of tiles, hence the same list
        assert mine["n_mfma_items"] == wide["n_mfma_items"]
        assert mine["num_waves"] == wide["num_waves"]


def test_tile_reported_under_32_row_panels_and_tile_sharing(gpu):  # noqa: F811
    """Both modes run tiles of a power of two columns; the reported tile follows them, set and unset,
    though the list of that width was made before.  Widths that a mode does not serve keep theirs."""
    A = W.paired_panels(1000, cols_per_group=60, half_width=200, seed=73)
    plan = make_plan(gpu, A)
    widths = {44: 48, 48: 48, 77: 80, 388: 112, 389: 112, 260: 96}

    def reported():
        lists = {N: gpu.spmm_plan_worklist(plan, N) for N in widths}
        for N, wl in lists.items():
            assert wl["n_tiles"] == -(-N // wl["n_tile"]) == -(-N // 128)
        return {N: wl["n_tile"] for N, wl in lists.items()}

    assert reported() == widths
    gpu.spmm_plan_set_tile_sharing(plan, gpu.SHARE_WORKGROUP)    # 388: four tiles; 260: three; 389 is odd
    assert reported() == widths | {388: 128}
    gpu.spmm_plan_set_tile_sharing(plan, gpu.SHARE_NONE)
    assert reported() == widths
    gpu.spmm_plan_set_panel_height(plan, 32)                     # N a multiple of four
    assert reported() == widths | {44: 64, 48: 64, 388: 128, 260: 128}
    gpu.spmm_plan_set_panel_height(plan, 16)
    assert reported() == widths
