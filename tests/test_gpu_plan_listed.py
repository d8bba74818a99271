"""Heavy panels among light, scattered ones: ranked by a bitmap of all columns or sorted, by their size and number and
the number of columns, and panel_ptr by one launch or two."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_narrow import kernels_of
from test_gpu_parity import INT_KEYS, assert_format_equal, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu

HEAVY = (513, 600, 1024, 2048, 2049, 4097, 8191, 8192)


def heavy_panel(n, K, rng):
    """Rows and columns of n entries, half of them in columns that the rows share, columns 0 and K - 1 among them."""
    shared = rng.choice(K, n // 16 + 8, replace=False)
    at = rng.choice(16 * len(shared), n // 2, replace=False)
    key = np.union1d(at % 16 * K + shared[at // 16], [0, 9 * K - 1])
    while len(key) < n:
        key = np.union1d(key, rng.integers(0, 16 * K, n - len(key)))
    return key // K, key % K


def matrix(P, K, light, heavy, seed):
    """P panels of `light` entries each but for the heavy ones, far apart, which have exactly theirs; a last panel of five
    rows."""
    rng = np.random.default_rng(seed)
    at = np.linspace(0, P - 2, len(heavy)).astype(int)
    panel = np.repeat(np.setdiff1d(np.arange(P), at), light)
    row = np.minimum(16 * panel + rng.integers(0, 16, len(panel)), 16 * P - 12)
    col = rng.integers(0, K, len(panel))
    edge = np.r_[True, panel[1:] != panel[:-1]]             # a panel's ends reached, so that the span is wide
    col[edge] = K - 1
    col[np.r_[False, edge[:-1]]] = 0
    parts = [heavy_panel(n, K, rng) for n in heavy]
    row = np.concatenate([row] + [16 * p + r for p, (r, _) in zip(at, parts)])
    col = np.concatenate([col] + [c for _, c in parts])
    A = W.csr_from_coo(16 * P - 11, K, row, col, rng.uniform(-1, 1, len(row)).astype(np.float32))
    sizes = A.rowptr[np.minimum(16 * np.arange(P + 1), A.M)]
    assert np.array_equal(np.diff(sizes)[at], heavy)
    return A


def same_as_the_oracle(gpu, A):  # noqa: F811
    plan = make_plan(gpu, A)
    ref = oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals)
    assert_format_equal(gpu.spmm_plan_export(plan), ref)
    got, exp = gpu.spmm_synergy(plan, 8), oracle.synergy(A.M, A.K, 8, A.rowptr, A.colind, ref)
    for k in INT_KEYS:
        assert got[k] == exp[k], (k, got[k], exp[k])


# 2^19 columns are the last that the bitmap takes; more light panels than one workgroup of the scan
@pytest.mark.parametrize("K", [50_001, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("P", [300, 4097])
@pytest.mark.parametrize("heavy", [HEAVY, (513,), (2049,) * 3, (700,) * 40])
def test_heavy_panels_among_light_ones(gpu, K, P, heavy):  # noqa: F811
    same_as_the_oracle(gpu, matrix(P, K, 20, heavy, seed=P + len(heavy)))


@pytest.mark.parametrize("light", [20, 140])
@pytest.mark.parametrize("heavy, bitmap, mid_sorted", [
    ((600,) * 3, False, True),                  # the middle class alone,
    ((2048,) + (513,) * 511, False, True),
    ((2049,), True, False),                     # with the largest as one round of workgroups,
    ((2049,) + (513,) * 511, True, False),
    ((2049,) + (513,) * 512, True, True),       # and as more than one
    ((8192, 2049) * 8 + (600,) * 900, True, True)])
def test_which_panels_a_bitmap_ranks(gpu, light, heavy, bitmap, mid_sorted):  # noqa: F811
    """A workgroup goes through a whole bitmap however few entries it has."""
    A = matrix(1500, 300_000, light, heavy, seed=light)
    names = kernels_of(lambda: make_plan(gpu, A))
    assert ("k_panel_bitmap_census" in names) == bitmap, names
    assert ("k_panel_sort_census<unsigned int, 11, true>" in names) == mid_sorted, names
    assert ("k_panel_sort_census<unsigned int, 11, false>" in names) != mid_sorted, names
    assert "k_panel_sort_census_big" not in names, names
    same_as_the_oracle(gpu, A)


def test_more_columns_than_a_bitmap_has(gpu):  # noqa: F811
    A = matrix(600, (1 << 19) + 1, 20, (8192, 2049) * 4 + (600,) * 40, seed=5)
    names = kernels_of(lambda: make_plan(gpu, A))
    assert "k_panel_sort_census_big" in names and "k_panel_bitmap_census" not in names, names
    same_as_the_oracle(gpu, A)


@pytest.mark.parametrize("P", [1 << 16, (1 << 16) + 1])
def test_panels_of_one_scan_launch(gpu, P):  # noqa: F811
    same_as_the_oracle(gpu, matrix(P, 400_000, 6, (600, 3000), seed=7))


@pytest.mark.parametrize("n", [700, 5000])
@pytest.mark.parametrize("fault", ["swapped", "duplicate", "beyond", "negative"])
def test_invalid_columns_in_heavy_panels(gpu, n, fault):  # noqa: F811
    import torch
    A = matrix(300, 90_000, 20, (600, n, 600), seed=n)
    panel = int(np.argmax(np.diff(A.rowptr[::16]) == np.diff(A.rowptr[::16])[1:-1].max()))
    lengths = np.diff(A.rowptr)
    row = 16 * panel + int(np.argmax(lengths[16 * panel:16 * panel + 16] >= 3))
    ci, at, end = A.colind.copy(), int(A.rowptr[row]), int(A.rowptr[row + 1])
    assert end - at >= 3
    if fault == "swapped":
        ci[at], ci[at + 1] = ci[at + 1], ci[at]
    elif fault == "duplicate":
        ci[at + 1] = ci[at]
    elif fault == "beyond":
        ci[end - 1] = A.K
    else:
        ci[at] = -1
    with pytest.raises(gpu.SpmmError) as e:
        gpu.spmm_plan(A.M, A.K, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(ci).cuda(),
                      torch.from_numpy(A.vals).cuda())
    assert e.value.code == gpu.SPMM_EFORMAT
